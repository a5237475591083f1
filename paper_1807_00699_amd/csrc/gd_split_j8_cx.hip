// Split-FP32 coupling kernels (gd_split.h): FP8-stored couplings, complex amplitudes.
#include "gd_split.h"

namespace gd {

hipError_t launch_split_j8_cx(int idx, int mode, const DenseStepArgs &a, hipStream_t st) {
#define GD_CASE(id, bm, bn, bk, wm, wn, ks, jd) \
    case id: return split::launch_modes<bm, bn, bk, wm, wn, ks, jd, true, split::J_FP8>(mode, a, st);
    switch (idx) { GD_SPLIT_J8_VARIANTS(GD_CASE) }
#undef GD_CASE
    return hipErrorInvalidValue;
}

}  // namespace gd

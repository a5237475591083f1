// Split-FP32 coupling kernels (gd_split.h): split couplings, real amplitudes.
#include "gd_split.h"

namespace gd {

hipError_t launch_split_j3_re(int idx, int mode, const DenseStepArgs &a, hipStream_t st) {
#define GD_CASE(id, bm, bn, bk, wm, wn, ks, jd) \
    case id: return split::launch_modes<bm, bn, bk, wm, wn, ks, jd, false, split::J_PIECES>(mode, a, st);
    switch (idx) { GD_SPLIT_J3_VARIANTS(GD_CASE) }
#undef GD_CASE
    return hipErrorInvalidValue;
}

}  // namespace gd

// Ising energies from the signs of the amplitudes (gd_split.h): FP8 couplings,
// one BF16 product, FP32 sums, FP64 terms.
#include "gd_split.h"

namespace gd {

hipError_t launch_split_sign(int idx, const DenseStepArgs &a, hipStream_t st) {
#define GD_CASE(id, bm, bn, bk, wm, wn, ks, jd) \
    case id: return split::launch_energy<bm, bn, bk, wm, wn, ks, jd, false, split::J_FP8_SIGN>(a, st);
    switch (idx) { GD_SPLIT_SIGN_VARIANTS(GD_CASE) }
#undef GD_CASE
    return hipErrorInvalidValue;
}

}  // namespace gd

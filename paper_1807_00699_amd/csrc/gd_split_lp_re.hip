// Reduced-precision coupling kernels on FP8-stored couplings (gd_split.h),
// real amplitudes.
#include "gd_split.h"

namespace gd {

hipError_t launch_split_lp_re(int idx, int mode, int op, const DenseStepArgs &a, hipStream_t st) {
#define GD_CASE(id, bm, bn, bk, wm, wn, ks, jd)                                                                     \
    case id:                                                                                                        \
        return op == OP_F16 ? split::launch_modes<bm, bn, bk, wm, wn, ks, jd, false, split::J_FP8, OP_F16>(mode, a, st) \
                            : split::launch_modes<bm, bn, bk, wm, wn, ks, jd, false, split::J_FP8, OP_BF16>(mode, a, st);
    switch (idx) { GD_SPLIT_LP_VARIANTS(GD_CASE) }
#undef GD_CASE
    return hipErrorInvalidValue;
}

}  // namespace gd

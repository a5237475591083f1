// Readout of one amplitude onto the spin domains of Eq. (h), in FP64: shared by
// the discretisation and energy kernels and the fused small-problem kernel.
#pragma once
#include "gd_internal.h"

namespace gd {

constexpr double kTwoPi = 6.283185307179586476925286766559;   // nearest double to 2 pi

// q-state clock readout in FP64: theta = arg Psi in [0, 2pi) (Psi = 0 ->
// theta = 0), k = floor(q theta / 2pi + 1/2) mod q.
__device__ inline int clock_state(double x, double y, int q) {
    double th = (x == 0.0 && y == 0.0) ? 0.0 : atan2(y, x);
    if (th < 0.0) th += kTwoPi;
    const long long c = (long long)floor((double)q * th / kTwoPi + 0.5);
    return (int)(((c % q) + q) % q);
}

// Planes of clock state k: d0 = cos(2 pi k / q); d1 = sin(2 pi k / q), held
// as sin / (sqrt(3)/2) in {0, +-1} for q = 3 and 6 so that both planes are
// exact (their product then carries the weight 3/4).
__device__ inline void clock_planes(int k, int q, double &d0, double &d1) {
    switch (q) {
    case 2: d0 = k ? -1.0 : 1.0; d1 = 0.0; return;
    case 3: d0 = k ? -0.5 : 1.0; d1 = k == 0 ? 0.0 : (k == 1 ? 1.0 : -1.0); return;
    case 4: d0 = k == 0 ? 1.0 : (k == 2 ? -1.0 : 0.0); d1 = k == 1 ? 1.0 : (k == 3 ? -1.0 : 0.0); return;
    case 6:   // cos: 1, 1/2, -1/2, -1, -1/2, 1/2; sin / (sqrt(3)/2): 0, 1, 1, 0, -1, -1
        d0 = k == 0 ? 1.0 : (k == 3 ? -1.0 : ((k == 1 || k == 5) ? 0.5 : -0.5));
        d1 = (k == 0 || k == 3) ? 0.0 : (k < 3 ? 1.0 : -1.0);
        return;
    default: sincospi(2.0 * k / q, &d1, &d0); return;
    }
}

// Discretised planes (d0, d1) of one amplitude in FP64 for readout `ro`;
// `k` receives the clock state (RO_CLOCK) or 0/1 for the sign readouts.
__device__ inline void readout_planes(double x, double y, int ro, int q, double &d0, double &d1,
                                      int &k) {
    d1 = 0.0;
    k = 0;
    switch (ro) {
    case RO_SIGN:
    case RO_SIGN_RE:
        d0 = (x < 0.0) ? -1.0 : 1.0;   // sign(+-0) = +1
        k = x < 0.0;
        return;
    case RO_PHASOR: {
        if (x == 0.0 && y == 0.0) {
            d0 = 1.0;
            return;
        }
        const double m = sqrt(x * x + y * y);
        d0 = x / m;
        d1 = y / m;
        return;
    }
    default:
        k = clock_state(x, y, q);
        clock_planes(k, q, d0, d1);
        return;
    }
}

}  // namespace gd

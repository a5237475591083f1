// Fused small-problem kernel (Np 64 or 128, FP32): many integration steps of a
// dense problem in one launch, and the energy check that ends them.
//
// What bounds it is the latency of dependent steps: the paper's small
// workload (N = 64, R = 100) is 100 independent chains of steps on a chip with
// 1024 SIMDs.  So one trajectory gets one wave (Np = 64) or one wave per 64
// spins and, for complex amplitudes, plane (Np = 128), a lane owns one spin,
// and the lane's row of J stays in registers for all steps.  The amplitudes
// reach the multiply-adds without LDS: two permlane swaps broadcast each row
// of 16 lanes to all four rows, and the multiply-adds read them rotated within
// the row (DPP), against couplings laid out in that order.  A coupling
// evaluation at Np = 64 is 64 multiply-adds in four chains and three swaps; at
// Np = 128 the waves of a trajectory exchange amplitudes through LDS, with one
// barrier.  Ising N = 64, R = 100: 0.26 us per step (0.66 with J and the
// amplitudes read from LDS by 256-thread workgroups).
#include "gd_check.h"
#include "gd_epilogue.h"
#include "gd_readout.h"

namespace gd {

namespace {

// Couplings in the order the lanes multiply them: word e / 4 of column block
// b for the rows of half h is out[((h NB + b) 16 + e / 4) 64 + lane], element
// e % 4: J[64 h + lane][64 b + 16 (e / 16) + (lane - e) % 16].
__global__ void small_couplings_k(const float *__restrict__ J, float *__restrict__ out, int Np) {
    const int nb = Np / 64;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < Np * Np; t += gridDim.x * blockDim.x) {
        const int e = (t & 3) + 4 * (t >> 8 & 15), lane = t >> 2 & 63, hb = t >> 12;
        const int row = 64 * (hb / nb) + lane, col = 64 * (hb % nb) + 16 * (e >> 4) + ((lane - e) & 15);
        out[t] = J[(long long)row * Np + col];
    }
}

// s[v] += w[v] * (r[v] of lane (l - N) mod 16 of l's row of 16 lanes), v < 4.
// One instruction each (the compiler leaves the rotation a move of its own).
// A DPP read needs two wait states after the vector instruction that wrote
// its register: the first block after the swaps (N = 1) waits for them.
#define GD_FMAC4                                                              \
    "v_fmac_f32_dpp %0, %4, %8 row_ror:%c12 row_mask:0xf bank_mask:0xf\n\t"   \
    "v_fmac_f32_dpp %1, %5, %9 row_ror:%c12 row_mask:0xf bank_mask:0xf\n\t"   \
    "v_fmac_f32_dpp %2, %6, %10 row_ror:%c12 row_mask:0xf bank_mask:0xf\n\t"  \
    "v_fmac_f32_dpp %3, %7, %11 row_ror:%c12 row_mask:0xf bank_mask:0xf"
#define GD_FMAC4_ARGS                                                         \
    "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3])                            \
    : "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(r[3]), "v"(w0), "v"(w1), "v"(w2), "v"(w3), "n"(N)
template <int N>
__device__ inline void fmac4_ror(float (&s)[4], const float (&r)[4], float w0, float w1, float w2, float w3) {
    if constexpr (N == 1) __asm__("s_nop 1\n\t" GD_FMAC4 : GD_FMAC4_ARGS);
    else __asm__(GD_FMAC4 : GD_FMAC4_ARGS);
}

// sum_j J_ij x_j over one column block: x_j in lane j, the lane's 64 couplings in w
__device__ inline float dot64(const float (&w)[64], float x) {
    const auto half = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const auto r01 = __builtin_amdgcn_permlane16_swap(half[0], half[0], false, false);
    const auto r23 = __builtin_amdgcn_permlane16_swap(half[1], half[1], false, false);
    const float r[4] = {__uint_as_float(r01[0]), __uint_as_float(r01[1]), __uint_as_float(r23[0]),
                        __uint_as_float(r23[1])};
    float s[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = r[v] * w[16 * v];
    seq_apply(
        [&](auto n) {
            constexpr int N = decltype(n)::value + 1;
            fmac4_ror<N>(s, r, w[N], w[16 + N], w[32 + N], w[48 + N]);
        },
        std::make_integer_sequence<int, 15>{});
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// `steps` Euler or RK4 steps (Eq. (main, gamma), as in gd_epilogue.h) of
// trajectory blockIdx.x, then the noise increment of step t0 + k after step k
// (key derived from `seed` as on the host).  With ce.E: the Eq. (h) energy of the
// final state's readout (ro, clock order q), E_r = sum_i [-(d0_i T0_i + w d1_i
// T1_i) + g_i d0_i], T = J d in FP32, the terms in FP64 in a fixed tree.
template <bool CPLX, int NPX, bool RK4>
__global__ void __launch_bounds__(64 * (NPX / 64) * (CPLX && NPX == 128 ? 2 : 1))
small_step_k(DenseStepArgs a, int steps, unsigned long long seed, long long t0, int ro, int q, CheckEnd ce) {
    constexpr int NB = NPX / 64;
    constexpr bool SPLIT = CPLX && NPX == 128;   // a wave holds one plane of its spins
    constexpr int NC = CPLX && !SPLIT ? 2 : 1;   // amplitude components held by a lane
    constexpr int W = NB * (SPLIT ? 2 : 1);
    __shared__ float xs[2][SPLIT ? 2 : 1][NPX];
    __shared__ double red[W];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = wave % NB, p = SPLIT ? wave / NB : 0;
    const int i = 64 * h + lane, r = blockIdx.x;
    const long long idx = (long long)r * NPX + i, ps = a.plane_stride;

    float w[NB][64];
    const f32x4 *jw = static_cast<const f32x4 *>(a.J) + h * NB * 16 * 64 + lane;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const f32x4 v = jw[(b * 16 + u) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[b][4 * u + e] = v[e];
        }
    float v[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = a.psi_in[(p + c) * ps + idx];
    float oth = SPLIT ? a.psi_in[(1 - p) * ps + idx] : 0.0f;   // the other plane's amplitude
    float g = a.gam_in[idx];
    const float ep = a.eps[i], hh = p == 0 ? a.h1[i] : 0.0f;
    const bool valid = i < a.n;
    float xh[NC];                                              // the other half's amplitudes
    int buf = 0;
    // exchange (s) between the waves of the trajectory: xh and `so`.  Two
    // buffers: a wave writes one again only after the barrier that follows
    // every wave's reads of it.
    auto publish = [&](const float (&s)[NC], float &so) {
        if constexpr (W > 1) {
            xs[buf][p][i] = s[0];
            __syncthreads();
            xh[0] = xs[buf][p][64 * (1 - h) + lane];
            if constexpr (SPLIT) so = xs[buf][1 - p][i];
            buf ^= 1;
        }
    };
    auto dot = [&](int c, float x) {
        float s = dot64(w[0], NB == 2 && h ? xh[c] : x);
        if constexpr (NB == 2) s += dot64(w[NB - 1], h ? x : xh[c]);
        return s;
    };
    // right-hand side at the stage (s, so, sg)
    auto rhs = [&](const float (&s)[NC], float so, float sg, float (&f)[NC], float &fg) {
        const float sx = SPLIT && p ? so : s[0];
        const float sy = CPLX ? (SPLIT ? (p ? s[0] : so) : s[NC - 1]) : 0.0f;
        const float rho = CPLX ? sx * sx + sy * sy : sx * sx;
        const float lin = sg - a.gamma_c - rho;
#pragma unroll
        for (int c = 0; c < NC; ++c) f[c] = s[c] * lin + dot(c, s[c]) * a.inv_s;
        f[0] += hh;
        fg = ep * (a.rho_th - rho);
        if (CPLX && a.q >= 2) {
            // resonant term h_q conj(Psi)^(q-1), as in the dense kernels
            float pr = sx, pi = -sy;
            for (int k = 2; k < a.q; ++k) {
                const float tr = pr * sx + pi * sy;
                const float ti = pi * sx - pr * sy;
                pr = tr;
                pi = ti;
            }
            f[0] += a.hq * (SPLIT && p ? pi : pr);
            if constexpr (NC == 2) f[NC - 1] += a.hq * pi;
        }
    };
    const float dt = a.dt;
    publish(v, oth);
    for (int st = 0; st < steps; ++st) {
        float f[NC], fg;
        if constexpr (!RK4) {
            rhs(v, oth, g, f, fg);
            if (valid) {
#pragma unroll
                for (int c = 0; c < NC; ++c) v[c] = v[c] + dt * f[c];
                g = g + dt * fg;
            }
        } else {
            // stage inputs y + c k with c = dt/2, dt/2, dt; accumulator
            // k1 + 2 k2 + 2 k3 (rows outside n keep their state)
            float acc[NC], s[NC], ag, sg = g, so = oth;
#pragma unroll
            for (int c = 0; c < NC; ++c) s[c] = v[c];
#pragma unroll
            for (int k = 1; k <= 3; ++k) {
                rhs(s, so, sg, f, fg);
                const float m = k == 1 ? 1.0f : 2.0f, ck = k == 3 ? dt : 0.5f * dt;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    acc[c] = k == 1 ? f[c] : acc[c] + m * f[c];
                    s[c] = valid ? v[c] + ck * f[c] : v[c];
                }
                ag = k == 1 ? fg : ag + m * fg;
                sg = valid ? g + ck * fg : g;
                publish(s, so);
            }
            rhs(s, so, sg, f, fg);
            const float c6 = dt * (1.0f / 6.0f);
            if (valid) {
#pragma unroll
                for (int c = 0; c < NC; ++c) v[c] = v[c] + c6 * (acc[c] + f[c]);
                g = g + c6 * (ag + fg);
            }
        }
        if (a.noise_amp != 0.0f && valid) {
            float g0, g1;
            noise_pair(mix64(seed ^ mix64((unsigned long long)(t0 + st))), r, i, g0, g1);
            v[0] += a.noise_amp * (SPLIT && p ? g1 : g0);
            if constexpr (NC == 2) v[NC - 1] += a.noise_amp * g1;
        }
        publish(v, oth);
    }
    bool bad = !__builtin_isfinite(g);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        a.psi_out[(p + c) * ps + idx] = v[c];
        if (tiny_number(v[c])) store_agent(a.tiny, 1);
        bad |= !__builtin_isfinite(v[c]);
    }
    if (p == 0) a.gam_out[idx] = g;
    // non-finite values persist once they appear, so the final state tells
    if (bad) store_agent(a.flags + r, 1);
    if (ce.E) {
        double d0 = 0.0, d1 = 0.0;
        int k;
        const float x = SPLIT && p ? oth : v[0], y = CPLX ? (SPLIT ? (p ? v[0] : oth) : v[NC - 1]) : 0.0f;
        if (valid) readout_planes(x, y, ro, q, d0, d1, k);
        float d[NC], unused = 0.0f;
        d[0] = float(SPLIT && p ? d1 : d0);
        if constexpr (NC == 2) d[NC - 1] = float(d1);
        publish(d, unused);
        double term = p == 0 ? (double)a.g[i] * (double)d[0] : 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double t = (double)d[c] * (double)dot(c, d[c]);
            term -= p + c == 0 ? t : (double)a.im_weight * t;
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) term += __shfl_xor(term, m);
        if constexpr (W == 1) {
            if (lane == 0) store_agent(ce.E + r, term);
        } else {
            if (lane == 0) red[wave] = term;
            __syncthreads();
            if (threadIdx.x == 0) {
                double s = red[0];
#pragma unroll
                for (int u = 1; u < W; ++u) s += red[u];
                store_agent(ce.E + r, s);
            }
        }
    }
    // the end of a check or a run: by the last trajectory, unless a launch follows for it
    if (ce.count && last_arrival(ce.count, gridDim.x)) check_end(ce);
}

#undef GD_FMAC4
#undef GD_FMAC4_ARGS

}  // namespace

hipError_t launch_small_couplings(const float *J, float *out, int Np, hipStream_t st) {
    if (Np != 64 && Np != 128) return hipErrorInvalidValue;
    small_couplings_k<<<Np * Np / 256, 256, 0, st>>>(J, out, Np);
    return hipGetLastError();
}

hipError_t launch_small_steps(bool complex_mode, bool rk4, const DenseStepArgs &a, int steps,
                              unsigned long long seed, long long t0, int readout, int q, const CheckEnd &c,
                              hipStream_t st) {
    if (!a.J || steps < 1 || (a.Np != 64 && a.Np != 128) || a.R < 1 || a.R > a.Rp) return hipErrorInvalidValue;
    if (c.E && readout == RO_CLOCK && (q < 2 || q > 8)) return hipErrorInvalidValue;
    if ((c.E || c.out) && (c.R != a.R || !c.count)) return hipErrorInvalidValue;
    const int waves = a.Np / 64 * (complex_mode && a.Np == 128 ? 2 : 1);
    CheckEnd z = c;
    const bool own_end = (c.E || c.out) && a.R > kEndRows;
    if (own_end || !(c.E || c.out)) z.count = nullptr;
#define GD_SMALL(C, N, K) small_step_k<C, N, K><<<a.R, 64 * waves, 0, st>>>(a, steps, seed, t0, readout, q, z)
    if (a.Np == 64) {
        if (complex_mode) { if (rk4) GD_SMALL(true, 64, true); else GD_SMALL(true, 64, false); }
        else { if (rk4) GD_SMALL(false, 64, true); else GD_SMALL(false, 64, false); }
    } else {
        if (complex_mode) { if (rk4) GD_SMALL(true, 128, true); else GD_SMALL(true, 128, false); }
        else { if (rk4) GD_SMALL(false, 128, true); else GD_SMALL(false, 128, false); }
    }
#undef GD_SMALL
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && own_end ? launch_check_end(c, st) : e;
}

}  // namespace gd

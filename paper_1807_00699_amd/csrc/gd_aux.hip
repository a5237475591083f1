// Auxiliary kernels of libgd.so: layout conversion, readout (discretisation)
// of the amplitudes onto the spin domains of Eq. (h), deterministic energy
// reductions and the FP64 re-scoring of Eq. (h).
#include "gd_check.h"
#include "gd_epilogue.h"
#include "gd_readout.h"

#include <algorithm>

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

namespace gd {

namespace {

// user [R][n] or [R][n][2] <-> planes [P][Rp][Np] (zero padded)
__global__ void pack_planes_k(const float *__restrict__ user, float *__restrict__ planes, int n,
                              int R, int Np, int Rp, int P, int *tiny) {
    const long long total = (long long)Rp * Np;
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total;
         t += (long long)gridDim.x * blockDim.x) {
        const int r = int(t / Np), i = int(t % Np);
        const bool in = (r < R) && (i < n);
        for (int p = 0; p < P; ++p) {
            float v = 0.0f;
            if (in) v = (P == 1) ? user[(long long)r * n + i] : user[((long long)r * n + i) * 2 + p];
            planes[p * total + t] = v;
            if (tiny && tiny_number(v)) *tiny = 1;
        }
    }
}

// Four spins of one trajectory per thread; `vec`: rows of the user's array are
// 16-byte aligned (n a multiple of 4).  Bound by HBM.
template <int P>
__device__ inline void unpack_rows(const float *__restrict__ planes, float *__restrict__ user, int n, int R, int Np,
                                   long long ps, bool vec) {
    const int i = 4 * (blockIdx.x * 256 + threadIdx.x);
    if (i >= n) return;
    for (int r = blockIdx.y; r < R; r += gridDim.y) {
        const float *src = planes + (long long)r * Np + i;
        float *dst = user + ((long long)r * n + i) * P;
        f32x4 v[P];
#pragma unroll
        for (int p = 0; p < P; ++p) v[p] = *reinterpret_cast<const f32x4 *>(src + p * ps);
        f32x4 o[P];
#pragma unroll
        for (int e = 0; e < 4 * P; ++e) o[e / 4][e % 4] = v[e % P][e / P];
        if (vec) {
#pragma unroll
            for (int p = 0; p < P; ++p) *reinterpret_cast<f32x4 *>(dst + 4 * p) = o[p];
        } else {
#pragma unroll
            for (int e = 0; e < 4 * P; ++e)
                if (i + e / P < n) dst[e] = o[e / 4][e % 4];
        }
    }
}

template <int P>
__global__ void __launch_bounds__(256) unpack_planes_k(const float *__restrict__ planes, float *__restrict__ user,
                                                       int n, int R, int Np, long long ps, bool vec) {
    unpack_rows<P>(planes, user, n, R, Np, ps, vec);
}

template <int P>
__global__ void __launch_bounds__(256)
unpack_state_k(const float *__restrict__ psi, float *__restrict__ upsi, const float *__restrict__ gam,
               float *__restrict__ ugam, int n, int R, int Np, long long ps, bool vec) {
    if (blockIdx.z == 0) unpack_rows<P>(psi, upsi, n, R, Np, ps, vec);
    else unpack_rows<1>(gam, ugam, n, R, Np, ps, vec);
}

__device__ inline void store_shadow(void *dst, long long k, float v, int op) {
    if (op == OP_BF16) static_cast<__hip_bfloat16 *>(dst)[k] = __float2bfloat16(v);
    else if (op == OP_F16) static_cast<__half *>(dst)[k] = __float2half(v);
}

// Readout onto the spin domains of Eq. (h).
__global__ void __launch_bounds__(256)
discretise_k(const float *__restrict__ psi, float *__restrict__ D, void *shadowD,
             int op, int ro, int q, int8_t *__restrict__ spins8,
             float *__restrict__ angle, int32_t *__restrict__ states,
             int *__restrict__ flags, int n, int R, int Np, int Rp, int P,
             long long ps) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    // 2-D grid: trajectories along y, groups of 4 consecutive spins along x
    // (Np is a multiple of 4: 16-byte plane loads and stores)
    const int nq = Np / 4;
    for (int r = blockIdx.y; r < Rp; r += gridDim.y)
    for (int iq = blockIdx.x * blockDim.x + threadIdx.x; iq < nq; iq += gridDim.x * blockDim.x) {
        const int i0 = iq * 4;
        const long long t = (long long)r * Np + i0;
        const f32x4 xv = *reinterpret_cast<const f32x4 *>(psi + t);
        const f32x4 yv = P == 2 ? *reinterpret_cast<const f32x4 *>(psi + ps + t) : f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 d0v = {0.f, 0.f, 0.f, 0.f}, d1v = {0.f, 0.f, 0.f, 0.f};
        bool nan = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + e;
            if (r >= R || i >= n) continue;
            const float x = xv[e], y = yv[e];
            double e0, e1;
            int k;
            readout_planes(x, y, ro, q, e0, e1, k);
            d0v[e] = float(e0);
            d1v[e] = float(e1);
            float th;
            if (ro == RO_PHASOR) {
                th = 0.0f;
                if (!(x == 0.0f && y == 0.0f)) {
                    th = atan2f(y, x);
                    if (th < 0.0f) th += 6.28318530717958647692f;
                    if (th >= 6.28318530717958647692f) th = 0.0f;
                }
            } else if (ro == RO_CLOCK) {
                th = float(kTwoPi * k / q);
            } else {
                th = k ? 3.14159265358979323846f : 0.0f;
            }
            const long long o = (long long)r * n + i;
            if (spins8) spins8[o] = k ? int8_t(-1) : int8_t(1);
            if (angle) angle[o] = th;
            if (states) states[o] = k;
            nan |= __builtin_isnan(x) || __builtin_isnan(y);
        }
        if (nan) flags[r] = 1;
        if (D) *reinterpret_cast<f32x4 *>(D + t) = d0v;
        if (D && P == 2) *reinterpret_cast<f32x4 *>(D + ps + t) = d1v;
        if (shadowD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                store_shadow(shadowD, t + e, d0v[e], op);
                if (P == 2) store_shadow(shadowD, ps + t + e, d1v[e], op);
            }
        }
    }
}

// int8 spins of real amplitudes alone, n a multiple of 4: four spins per load
// and store, four of those in flight per thread.  Bound by HBM: N = R = 4096
// 14 us (discretise_k 36, one load per thread).
__global__ void __launch_bounds__(256)
sign_spins_k(const float *__restrict__ psi, unsigned *__restrict__ spins, int *__restrict__ flags, int n, int R, int Np) {
    const unsigned nq = n / 4, total = nq * (unsigned)R;   // (the launcher's limit: below 2^31)
    constexpr int U = 4;
    const unsigned q0 = blockIdx.x * (256u * U) + threadIdx.x;
    f32x4 x[U];
    unsigned r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const unsigned q = min(q0 + u * 256u, total - 1);
        r[u] = q / nq;
        x[u] = *reinterpret_cast<const f32x4 *>(psi + (long long)r[u] * Np + 4 * (q - r[u] * nq));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (q0 + u * 256u >= total) break;
        unsigned w = 0;
        bool nan = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            w |= (x[u][e] < 0.0f ? 0xFFu : 1u) << 8 * e;
            nan |= __builtin_isnan(x[u][e]);
        }
        spins[q0 + u * 256u] = w;
        if (nan) flags[r[u]] = 1;
    }
}

// E[r] = sum over row tiles in fixed order (one thread per trajectory).
__global__ void energy_sum_k(const double *__restrict__ partial, int ntiles, int Rp, int R,
                             double *__restrict__ E) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    double s = 0.0;
    for (int t = 0; t < ntiles; ++t) s += partial[(long long)t * Rp + r];
    E[r] = s;
}

// The same sums for few trajectories and many row tiles: one wave per
// trajectory, lane l adds tiles l, l + 64, ... in order, then a butterfly
// over the wave (a fixed order, so repeated checks give the same sums).
__global__ void __launch_bounds__(64) energy_sum_wide_k(const double *__restrict__ partial, int ntiles, int Rp,
                                                        CheckEnd c) {
    const int r = blockIdx.x, lane = threadIdx.x;
    double s = 0.0;
    for (int t = lane; t < ntiles; t += 64) s += partial[(long long)t * Rp + r];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m);
    if (lane == 0) store_agent(c.E + r, s);
    if (c.count && last_arrival(c.count, c.R)) check_end(c);
}

__global__ void __launch_bounds__(1024) check_end_k(CheckEnd c) { check_end<4>(c); }

// FP64 re-score of Eq. (h) for the discretised state, formed in FP64 from
// the FP32 amplitudes by the readout of the model.  The readout planes are
// written once in FP64 ([P][Rp][Np], zero outside n x R); then per workgroup
// (row tile t of 64 spins, column tile of 64 trajectories): T = J d over K
// through LDS in FP64, and partial[t][r] = sum_{i in tile} [ -(d0_i T0_i +
// w d1_i T1_i) + g_i d0_i ] (w: weight of the second plane).
constexpr int E64_T = 64;
constexpr int E64_K = 16;

__global__ void __launch_bounds__(256)
planes64_k(const float *__restrict__ psi, double *__restrict__ D64, int n, int R, int Np, int Rp, int P,
           long long ps, int ro, int q) {
    for (int r = blockIdx.y; r < Rp; r += gridDim.y)
        for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < Np; i += gridDim.x * blockDim.x) {
            const long long t = (long long)r * Np + i;
            double d0 = 0.0, d1 = 0.0;
            if (r < R && i < n) {
                int k;
                readout_planes(psi[t], P == 2 ? psi[ps + t] : 0.0f, ro, q, d0, d1, k);
            }
            D64[t] = d0;
            if (P == 2) D64[ps + t] = d1;
        }
}

// T = J d on the FP64 matrix cores (v_mfma_f64_16x16x4_f64): workgroup tile
// 64 rows x 64 trajectories, 2 x 2 waves of 32 x 32 (2 x 2 blocks of 16 x 16),
// K chunks of 16 staged in LDS as [row][k] doubles with a one-double pad (the
// 8-byte operand reads of 16 rows at one k then hit distinct banks).  MFMA
// operands: A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k; result
// D[l / 16 + 4 e][l % 16] in element e of lane l (rows interleaved, unlike
// the FP32 16x16x4 layout).
template <int P>
__global__ void __launch_bounds__(256)
energy_fp64_k(const float *__restrict__ J, const double *__restrict__ D64, const float *__restrict__ g,
              double *__restrict__ partial, int Np, int Rp, long long ps, double w) {
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    constexpr int KP = E64_K + 1;
    __shared__ double sJ[E64_T][KP];
    __shared__ double sD[P][E64_T][KP];
    __shared__ double red[2][E64_T];
    const int mt = blockIdx.x, ct = blockIdx.y;
    const int i0 = mt * E64_T, r0 = ct * E64_T;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int l16 = lane & 15, lq = lane >> 4;
    f64x4 acc[P][2][2];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc[p][mb][nb] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < Np; k0 += E64_K) {
        // 64 rows x 16 k of J and of each plane: 4 elements per thread
#pragma unroll
        for (int u = 0; u < E64_K * E64_T / 256; ++u) {
            const int e = tid + u * 256;
            const int row = e / E64_K, kk = e % E64_K;
            sJ[row][kk] = (double)J[(long long)(i0 + row) * Np + k0 + kk];
#pragma unroll
            for (int p = 0; p < P; ++p) sD[p][row][kk] = D64[p * ps + (long long)(r0 + row) * Np + k0 + kk];
        }
        __syncthreads();
#pragma unroll
        for (int k4 = 0; k4 < E64_K / 4; ++k4) {
            const int k = 4 * k4 + lq;
            double av[2], bv[P][2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) av[mb] = sJ[wm * 32 + mb * 16 + l16][k];
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) bv[p][nb] = sD[p][wn * 32 + nb * 16 + l16][k];
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        acc[p][mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[mb], bv[p][nb], acc[p][mb][nb],
                                                                             0, 0, 0);
        }
        __syncthreads();
    }
    // per trajectory column: sum over this wave's rows, then over the lanes
    // that hold the same column, then over the two row waves
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int rl = wn * 32 + nb * 16 + l16;
        const long long rb = (long long)(r0 + rl) * Np;
        double s = 0.0;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = i0 + wm * 32 + mb * 16 + lq + 4 * e;
                const double d0 = D64[rb + i];
                double t = d0 * acc[0][mb][nb][e];
                if (P == 2) t += w * (D64[ps + rb + i] * acc[P - 1][mb][nb][e]);
                s += -t + (double)g[i] * d0;
            }
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lq == 0) red[wm][rl] = s;
    }
    __syncthreads();
    if (tid < E64_T) partial[(long long)mt * Rp + r0 + tid] = red[0][tid] + red[1][tid];
}

__global__ void make_shadow_k(const float *__restrict__ src, void *dst, long long count, int op) {
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < count;
         t += (long long)gridDim.x * blockDim.x)
        store_shadow(dst, t, src[t], op);
}

inline int grid_for(long long total) {
    long long b = (total + 255) / 256;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return int(b);
}

}  // namespace

hipError_t launch_pack_planes(const float *user, float *planes, int n, int R, int Np, int Rp,
                              int nplanes, int *tiny, hipStream_t st) {
    pack_planes_k<<<grid_for((long long)Rp * Np), 256, 0, st>>>(user, planes, n, R, Np, Rp, nplanes, tiny);
    return hipGetLastError();
}

hipError_t launch_unpack_planes(const float *planes, float *user, int n, int R, int Np, int Rp,
                                int nplanes, hipStream_t st) {
    const dim3 grid(unsigned((n + 1023) / 1024), unsigned(std::min(R, 65535)));
    const long long ps = (long long)Rp * Np;
    const bool vec = n % 4 == 0 && reinterpret_cast<uintptr_t>(user) % 16 == 0;
    if (nplanes == 2) unpack_planes_k<2><<<grid, 256, 0, st>>>(planes, user, n, R, Np, ps, vec);
    else unpack_planes_k<1><<<grid, 256, 0, st>>>(planes, user, n, R, Np, ps, vec);
    return hipGetLastError();
}

hipError_t launch_unpack_state(const float *psi, float *upsi, const float *gam, float *ugam, int n, int R, int Np, int Rp,
                               int nplanes, hipStream_t st) {
    const dim3 grid(unsigned((n + 1023) / 1024), unsigned(std::min(R, 65535)), 2);
    const long long ps = (long long)Rp * Np;
    const bool vec =
        n % 4 == 0 && (reinterpret_cast<uintptr_t>(upsi) | reinterpret_cast<uintptr_t>(ugam)) % 16 == 0;
    if (nplanes == 2) unpack_state_k<2><<<grid, 256, 0, st>>>(psi, upsi, gam, ugam, n, R, Np, ps, vec);
    else unpack_state_k<1><<<grid, 256, 0, st>>>(psi, upsi, gam, ugam, n, R, Np, ps, vec);
    return hipGetLastError();
}

float clock_im_weight(int q) { return (q == 3 || q == 6) ? 0.75f : 1.0f; }

hipError_t launch_discretise(const float *psi, float *D, void *shadowD, int op, int readout, int q,
                             int8_t *spins8, float *angle, int32_t *states, int *flags, int n, int R,
                             int Np, int Rp, int nplanes, long long plane_stride, hipStream_t st) {
    if (readout == RO_CLOCK && (q < 2 || q > 8)) return hipErrorInvalidValue;
    if (Np % 4) return hipErrorInvalidValue;
    const long long quads = (long long)(n / 4) * R;
    if (spins8 && !D && !shadowD && !angle && !states && readout == RO_SIGN && nplanes == 1 && n % 4 == 0 &&
        reinterpret_cast<uintptr_t>(spins8) % 4 == 0 && quads < (1ll << 31)) {
        sign_spins_k<<<unsigned((quads + 1023) / 1024), 256, 0, st>>>(psi, reinterpret_cast<unsigned *>(spins8), flags, n, R,
                                                                     Np);
        return hipGetLastError();
    }
    const dim3 grid(unsigned(std::min(64, (Np / 4 + 255) / 256)), unsigned(std::min(Rp, 65535)));
    discretise_k<<<grid, 256, 0, st>>>(psi, D, shadowD, op, readout, q, spins8,
                                                              angle, states, flags, n, R, Np, Rp,
                                                              nplanes, plane_stride);
    return hipGetLastError();
}

hipError_t launch_energy_reduce(const double *partial, int ntiles, int Rp, const CheckEnd &c, hipStream_t st) {
    if (c.R < 1 || c.R > Rp || !c.E || !c.count) return hipErrorInvalidValue;
    // one thread per trajectory reads its tiles one after the other: N = 800,
    // R = 100 (26 tiles) 7.3 us
    if (c.R <= 512 && ntiles >= 8) {
        CheckEnd z = c;
        if (c.R > kEndRows) z.count = nullptr;
        energy_sum_wide_k<<<c.R, 64, 0, st>>>(partial, ntiles, Rp, z);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess && !z.count ? launch_check_end(c, st) : e;
    }
    energy_sum_k<<<(c.R + 255) / 256, 256, 0, st>>>(partial, ntiles, Rp, c.R, c.E);
    return launch_check_end(c, st);
}

hipError_t launch_check_end(const CheckEnd &c, hipStream_t st) {
    if (c.R < 1 || (c.out && !c.flags)) return hipErrorInvalidValue;
    check_end_k<<<1, c.R > 512 ? 1024 : c.R > 64 ? 256 : 64, 0, st>>>(c);
    return hipGetLastError();
}

hipError_t launch_energy_fp64(const float *J, const float *psi, const float *g, double *D64,
                              double *partial, int Np, int Rp, int n, int R, int nplanes,
                              long long plane_stride, int readout, int q, hipStream_t st) {
    if (Np % E64_T || Rp % E64_T) return hipErrorInvalidValue;
    if (readout == RO_CLOCK && (q < 2 || q > 8)) return hipErrorInvalidValue;
    if (nplanes != 1 && nplanes != 2) return hipErrorInvalidValue;
    const double w = readout == RO_CLOCK ? (double)clock_im_weight(q) : 1.0;
    const dim3 pgrid(unsigned(std::min(64, (Np + 255) / 256)), unsigned(std::min(Rp, 65535)));
    planes64_k<<<pgrid, 256, 0, st>>>(psi, D64, n, R, Np, Rp, nplanes, plane_stride, readout, q);
    const dim3 grid(Np / E64_T, Rp / E64_T);
    if (nplanes == 2)
        energy_fp64_k<2><<<grid, 256, 0, st>>>(J, D64, g, partial, Np, Rp, plane_stride, w);
    else
        energy_fp64_k<1><<<grid, 256, 0, st>>>(J, D64, g, partial, Np, Rp, plane_stride, w);
    return hipGetLastError();
}

hipError_t launch_make_shadow(const float *src, void *dst, long long count, int op, hipStream_t st) {
    make_shadow_k<<<grid_for(count), 256, 0, st>>>(src, dst, count, op);
    return hipGetLastError();
}

}  // namespace gd

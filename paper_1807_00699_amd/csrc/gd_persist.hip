// Persistent steps: all steps of a run in one launch, J in registers, the
// amplitudes exchanged between workgroups through device memory.
//
// What bounds small dense problems is the latency of a step: its launch, the
// loads of J and of the amplitudes and their reduction, 5-8 us for microseconds
// of work.  Here a workgroup keeps its rows of J in registers (FP8, or the
// three BF16 pieces of gd_split.h) and its spins' state, and a step is: wait
// for the amplitudes of its trajectories, split and multiply (as gd_split.h:
// the same exact products, sums in FP32), add the waves' sums in LDS, update,
// publish (2^24 Psi, gd_split.h).  Trajectories are independent, so only the
// workgroups of one group of trajectories wait for each other.
//
// Exchange: an amplitude is its own arrival mark.  Slots hold kEmpty (a NaN
// pattern that is never published) until the new value is stored; readers poll
// the values themselves, so a step costs one store and one load through the
// memory side (1.5-2.4 us measured for 4 KB to 50 KB per group).  Amplitude
// set k goes through buffer k % 4.  A workgroup that has read set k - 1 knows
// that every other one has read set k - 2 (they published k - 1 after it), so
// it marks its slots of that buffer empty again; those stores have arrived
// (waited for one evaluation later) before it publishes set k + 1, which every
// reader of the next values of that buffer has seen.  The set counter goes on
// from launch to launch, which makes the first marks of a launch those of the
// last sets of the one before.  A poll that comes too early costs a whole
// round trip, so every wave sleeps first: with hardly any pause N = 4096, R = 1
// takes 2.7 us per step instead of 1.9, XY N = 1000, R = 128 24.3 instead of
// 17.7 (16.5 now).
//
// All workgroups have to be resident at once: at most one per CU, launched
// cooperatively.  A wait longer than `patience` ends the kernel in every
// workgroup that waits for the others, and sets *stalled; launches that find it
// set end at their first missing amplitude.  No launch writes the state it
// reads, so the state at the start of the first of them is there for the host
// to go on from.
//
// Per step in long runs, one launch per step -> persistent: Ising Euler N =
// 4096, R = 1 5.6 -> 1.9 us (FP8 couplings), 13.2 -> 2.4 (split couplings); N =
// 300, R = 64 4.2 -> 1.9; N = 800, R = 100 5.5 -> 3.1; N = 2000, R = 64 8.4 ->
// 5.6; XY RK4 (four evaluations) N = 1000, R = 128 30.5 -> 16.5, N = 1500, R =
// 48 with FP8 couplings 30.1 -> 23.4.  Each cooperative launch adds about 20 us.
#include "gd_check.h"
#include "gd_split.h"

namespace gd {

namespace {

using split::bf16x8;
using split::kAmpScale;
using split::ldexp4;
using split::split8;
using split::u32x4;
using split::widen8;

constexpr unsigned kEmpty = 0xFFFFFFFFu;   // a slot not yet published
constexpr int kWaves = 8;
// pauses before the first poll, in sleeps of 64 cycles: the time that the
// published amplitudes take to arrive.  N = 800, R = 100 3.54, 3.20 and 3.30 us
// per step for 6, 10 and 16; XY N = 1000, R = 128 16.8 per RK4 step for 6 to 10,
// 17.5 for 16.  Few trajectories, 5 and 24: N = 200 1.4-1.7 and 1.7-2.2; N = 1000,
// R = 1 to 4, FP8 couplings 1.77, 2.57, 3.18, 3.16 and 1.64, 1.92, 2.46, 2.55,
// split couplings 2.07, 2.55, 3.65, 3.22 and 1.86, 2.56, 3.71, 3.71; N = 1100
// 1.89-3.68, 2.11-4.13 and 1.76-3.20, 1.93-4.03; N = 4096, R = 1 2.82 and 2.00
constexpr int kPause = 10, kPauseFew = 5, kPauseFewLarge = 24;

__device__ inline f32x4 mfma16(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
}

__device__ inline bool empty2(unsigned long long v) {
    return (unsigned)v == kEmpty || (unsigned)(v >> 32) == kEmpty;
}

__device__ inline unsigned long long load2(const unsigned long long *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline void store1(unsigned *p, unsigned v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A group of 16 real or 8 complex trajectories (one 16-column operand: the
// real parts, then the imaginary parts).  A workgroup has 16 RB rows; its
// eight waves take the fragments w, w + 8, ... of 32 columns of J (FR each, Np
// <= 256 FR), poll the amplitudes in operand order and need no LDS for them.
// Fewer rows spread the matrix work, more rows read the exchange less often:
// with two workgroups of 16 rows per CU N = 800, R = 100 took 4.4 us per step
// instead of 3.5.
template <int FR, int RB, bool CPLX, bool RK4, bool J8>
__global__ void __launch_bounds__(64 * kWaves)
persist_step_k(DenseStepArgs a, PersistArgs p) {
    constexpr int TR = CPLX ? 8 : 16;            // trajectories of a group
    constexpr int ROWS = 16 * RB, RS = ROWS + 4;
    // third pieces of J kept in LDS, as many as fit, where the registers do not
    // hold them (spilled ones cost XY N = 1000, R = 128 10%); the waves' sums
    // then have one buffer and a barrier more
    constexpr int JL = !J8 && FR * RB > 12 ? (RB == 4 ? 15 : FR * RB) : 0;
    __shared__ __attribute__((aligned(16))) float red[JL ? 1 : 2][kWaves][16][RS];
    __shared__ __attribute__((aligned(16))) u32x4 jlds[JL ? JL * kWaves * 64 : 1];
    __shared__ int stalled, gone;   // gone: thread 0's, here to take no register
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const int g = blockIdx.x % p.groups, m0 = blockIdx.x / p.groups * ROWS;
    const int nf = a.Np / 32;
    const long long ps = a.plane_stride;
    long long before = 0;   // (looked at once the first amplitudes are on their way)
    if (tid == 0) {
        before = __hip_atomic_load(p.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stalled = 0;
    }

    // this wave's couplings: fragments w, w + 8, ... of 32 columns, RB blocks of 16 rows
    u32x4 j[J8 ? 1 : FR][J8 ? 1 : RB][3];
    uint2 j8[J8 ? FR : 1][J8 ? RB : 1];
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        const int kf = f * kWaves + wave;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = min(m0 + 16 * rb + col, a.Np - 1);
            const long long at = (long long)row * a.Np + min(kf, nf - 1) * 32 + 8 * kq;
            if constexpr (J8) {
                j8[f][rb] = *reinterpret_cast<const uint2 *>(static_cast<const unsigned char *>(a.J) + at);
            } else {
                const f32x4 *q = reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.J) + at);
                u32x4 t;
                split8(ldexp4(q[0], -a.j_exp), ldexp4(q[1], -a.j_exp), j[f][rb][0], j[f][rb][1], t);
                if (f * RB + rb < JL) jlds[((f * RB + rb) * kWaves + wave) * 64 + lane] = t;
                else j[f][rb][2] = t;
            }
        }
    }

    // this thread's spins (rows lr + 32 k) and trajectory
    constexpr int IT = ROWS * TR > 64 * kWaves ? ROWS * TR / (64 * kWaves) : 1;
    const bool item = tid < ROWS * TR;
    const int lr = 2 * (tid / (2 * TR)) + (tid & 1), tr = (tid >> 1) & (TR - 1), r = g * TR + tr;
    constexpr int LSTEP = 64 * kWaves / TR;
    float xr[IT], xi[IT], gm[IT], ep[IT], hh[IT], yr[IT], yi[IT], yg[IT], ar[IT], ai[IT], ag[IT];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int i = m0 + lr + k * LSTEP;
        xr[k] = xi[k] = gm[k] = ep[k] = hh[k] = ar[k] = ai[k] = ag[k] = 0.0f;
        if (item && i < a.n && r < a.R) {
            xr[k] = a.psi_in[(long long)r * a.Np + i];
            if (CPLX) xi[k] = a.psi_in[ps + (long long)r * a.Np + i];
            gm[k] = a.gam_in[(long long)r * a.Np + i];
            ep[k] = a.eps[i];
            hh[k] = a.h1[i];
        }
        yr[k] = xr[k];
        yi[k] = xi[k];
        yg[k] = gm[k];
    }
    // exchange: four buffers of [group][fragment][k pair][lane][2]
    const long long gsz = (long long)nf * 512, bsz = gsz * p.groups;
    unsigned *const xg = p.x + g * gsz;
    auto slot = [&](long long set, int k) {
        const int i = m0 + lr + k * LSTEP;
        return xg + (set & 3) * bsz + ((((i >> 5) * 4 + ((i >> 1) & 3)) * 64 + ((i >> 3) & 3) * 16 + tr) * 2 + (i & 1));
    };
    auto publish = [&](long long set) {   // (a NaN of the empty pattern becomes another NaN)
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            if (!(item && m0 + lr + k * LSTEP < a.Np)) continue;
            unsigned *out = slot(set, k);
            const unsigned ur = __float_as_uint(xr[k] * kAmpScale), ui = __float_as_uint(xi[k] * kAmpScale);
            store1(out, ur == kEmpty ? 0x7FC00000u : ur);
            if (CPLX) store1(out + 16, ui == kEmpty ? 0x7FC00000u : ui);
        }
    };

    publish(p.base);
    __syncthreads();
    if (tid == 0) {
        gone = before != 0;
        if (gone || p.patience < 0) stalled = 1;
    }
    const int evals = p.steps * (RK4 ? 4 : 1);
    for (int ev = 1; ev <= evals; ++ev) {
        f32x4 hi[RB], lo[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) hi[rb] = lo[rb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(
                                            p.x + ((p.base + ev - 1) & 3) * bsz + g * gsz) + lane;
        unsigned long long v[FR][4];
        auto fetch = [&](int f) {
            const unsigned long long *q = src + (f * kWaves + wave) * 256;
            v[f][0] = load2(q);
            v[f][1] = load2(q + 64);
            v[f][2] = load2(q + 128);
            v[f][3] = load2(q + 192);
        };
        auto missing = [&](int f) {
            return __any(empty2(v[f][0]) || empty2(v[f][1]) || empty2(v[f][2]) || empty2(v[f][3]));
        };
        for (int q = 0; q < p.pause; ++q) __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int f = 0; f < FR; ++f)
            if (f * kWaves + wave < nf) fetch(f);
#pragma unroll
        for (int f = 0; f < FR; ++f) {
            const int kf = f * kWaves + wave;
            if (kf < nf) {
                long long since = 0;
                while (missing(f)) {
                    const long long now = wall_clock64();
                    if (since == 0) since = now;
                    if (now - since > p.patience || *(volatile int *)&stalled) {
                        stalled = 1;
                        break;
                    }
                    fetch(f);
                }
                f32x4 b0, b1;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    (u < 2 ? b0 : b1)[2 * (u & 1)] = __uint_as_float((unsigned)v[f][u]);
                    (u < 2 ? b0 : b1)[2 * (u & 1) + 1] = __uint_as_float((unsigned)(v[f][u] >> 32));
                }
                u32x4 x0, x1, x2;
                split8(b0, b1, x0, x1, x2);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    if constexpr (J8) {
                        const u32x4 j0 = widen8<OP_F32>(j8[f][rb].x, j8[f][rb].y);
                        lo[rb] = mfma16(j0, x2, lo[rb]);
                        lo[rb] = mfma16(j0, x1, lo[rb]);
                        hi[rb] = mfma16(j0, x0, hi[rb]);
                    } else {
                        const u32x4 &j0 = j[f][rb][0], &j1 = j[f][rb][1];
                        const u32x4 j2 = f * RB + rb < JL ? jlds[((f * RB + rb) * kWaves + wave) * 64 + lane] : j[f][rb][2];
                        lo[rb] = mfma16(j0, x2, lo[rb]);
                        lo[rb] = mfma16(j2, x0, lo[rb]);
                        lo[rb] = mfma16(j1, x1, lo[rb]);
                        lo[rb] = mfma16(j0, x1, lo[rb]);
                        lo[rb] = mfma16(j1, x0, lo[rb]);
                        hi[rb] = mfma16(j0, x0, hi[rb]);
                    }
                }
            }
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            *reinterpret_cast<f32x4 *>(&red[JL ? 0 : ev & 1][wave][col][16 * rb + 4 * kq]) = hi[rb] + lo[rb];
        // (also: the empty marks this wave stored in the last evaluation have arrived)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (stalled) break;
        float cr[IT], ci[IT];
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            cr[k] = ci[k] = 0.0f;
            if (item) {
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    cr[k] += red[JL ? 0 : ev & 1][w][tr][lr + k * LSTEP];
                    if (CPLX) ci[k] += red[JL ? 0 : ev & 1][w][(8 + tr) & 15][lr + k * LSTEP];
                }
            }
        }
        if constexpr (JL != 0) __syncthreads();
        const int stage = RK4 ? (ev - 1) & 3 : 0;
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            const int i = m0 + lr + k * LSTEP;
            const float x = xr[k], z = xi[k];
            const float rho = CPLX ? x * x + z * z : x * x;
            const float lin = gm[k] - a.gamma_c - rho;
            float fr = x * lin + cr[k] * a.inv_s + hh[k];
            float fi = CPLX ? z * lin + ci[k] * a.inv_s : 0.0f;
            const float fg = ep[k] * (a.rho_th - rho);
            if (CPLX && a.q >= 2) {
                float pr = x, pi = -z;
                for (int m = 2; m < a.q; ++m) {
                    const float u = pr * x + pi * z;
                    pi = pi * x - pr * z;
                    pr = u;
                }
                fr += a.hq * pr;
                fi += a.hq * pi;
            }
            if (!RK4) {
                xr[k] = x + a.dt * fr;
                xi[k] = z + a.dt * fi;
                gm[k] += a.dt * fg;
            } else if (stage == 3) {
                const float c6 = a.dt * (1.0f / 6.0f);
                xr[k] = yr[k] + c6 * (ar[k] + fr);
                xi[k] = yi[k] + c6 * (ai[k] + fi);
                gm[k] = yg[k] + c6 * (ag[k] + fg);
            } else {
                ar[k] = stage ? ar[k] + 2.0f * fr : fr;
                ai[k] = stage ? ai[k] + 2.0f * fi : fi;
                ag[k] = stage ? ag[k] + 2.0f * fg : fg;
                const float c = stage == 2 ? a.dt : 0.5f * a.dt;
                xr[k] = yr[k] + c * fr;
                xi[k] = yi[k] + c * fi;
                gm[k] = yg[k] + c * fg;
            }
            if (!RK4 || stage == 3) {
                if (a.noise_amp != 0.0f) {
                    float g0, g1;
                    noise_pair(mix64(p.seed ^ mix64((unsigned long long)(p.t0 + (RK4 ? (ev - 1) / 4 : ev - 1)))), r, i, g0,
                               g1);
                    xr[k] += a.noise_amp * g0;
                    if (CPLX) xi[k] += a.noise_amp * g1;
                }
                yr[k] = xr[k];
                yi[k] = xi[k];
                yg[k] = gm[k];
            }
            if (!(item && i < a.n && r < a.R)) xr[k] = xi[k] = gm[k] = yr[k] = yi[k] = yg[k] = 0.0f;
        }
        if (ev < evals) publish(p.base + ev);
#pragma unroll
        for (int k = 0; k < IT; ++k) {
            if (!(item && m0 + lr + k * LSTEP < a.Np)) continue;
            unsigned *mark = slot(p.base + ev + 2, k);
            store1(mark, kEmpty);
            if (CPLX) store1(mark + 16, kEmpty);
        }
    }
    if (stalled && tid == 0 && !gone) store_agent(p.stalled, p.tag);
#pragma unroll
    for (int k = 0; k < IT && !stalled; ++k) {
        const int i = m0 + lr + k * LSTEP;
        if (!(item && i < a.n && r < a.R)) continue;
        a.psi_out[(long long)r * a.Np + i] = xr[k];
        if (tiny_number(xr[k]) || (CPLX && tiny_number(xi[k]))) store_agent(a.tiny, 1);
        if (CPLX) a.psi_out[ps + (long long)r * a.Np + i] = xi[k];
        a.gam_out[(long long)r * a.Np + i] = gm[k];
        if (!(gd_finite(xr[k]) && gd_finite(gm[k]) && gd_finite(xi[k]))) store_agent(a.flags + r, 1);
    }
}

// Few trajectories: R <= NR <= 4 real ones, Np <= 4096.  A workgroup has 16
// rows, a wave 256 columns of them.  The pieces of the amplitudes are columns
// of the matrix product (3 r + piece), so one matrix instruction per 32
// couplings (three with split couplings) takes all trajectories; every lane
// polls and splits four amplitudes of each, and the operands are transposed
// through LDS within the wave.
template <int NR, bool J8>
__global__ void __launch_bounds__(1024)
persist_few_k(DenseStepArgs a, PersistArgs p, CheckEnd ce) {
    constexpr int NC = 3 * NR, PB = 528, RS = 20;   // LDS bytes of one piece's 256 values, floats of 16 rows (both padded)
    __shared__ __attribute__((aligned(16))) unsigned char xl[16][NC][PB];
    __shared__ __attribute__((aligned(16))) float red[2][16][NC][RS];
    __shared__ int stalled, gone;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nw = blockDim.x / 64;
    const int col = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.x * 16, Np = a.Np, R = a.R;
    long long before = 0;   // (looked at once the first amplitudes are on their way)
    if (tid == 0) {
        before = __hip_atomic_load(p.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stalled = 0;
    }

    uint2 j8[8];
    u32x4 j[J8 ? 1 : 8][3];
#pragma unroll
    for (int f = 0; f < 8; ++f) {
        const int k = 256 * wave + 32 * f + 8 * kq;
        const long long at = (long long)(m0 + col) * Np + k;
        if constexpr (J8) {
            j8[f] = make_uint2(0u, 0u);
            if (k < Np) j8[f] = *reinterpret_cast<const uint2 *>(static_cast<const unsigned char *>(a.J) + at);
        } else {
            f32x4 q[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
            if (k < Np) {
                q[0] = reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.J) + at)[0];
                q[1] = reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.J) + at)[1];
            }
            split8(ldexp4(q[0], -a.j_exp), ldexp4(q[1], -a.j_exp), j[f][0], j[f][1], j[f][2]);
        }
    }

    // wave r < R: trajectory r, its 16 rows in the lanes of each quarter
    const int r = wave, i = m0 + (lane & 15);
    const bool updates = wave < R, inside = updates && i < a.n;
    float x = 0.0f, gm = 0.0f, ep = 0.0f, hh = 0.0f;
    if (inside) {
        x = a.psi_in[(long long)r * Np + i];
        gm = a.gam_in[(long long)r * Np + i];
        ep = a.eps[i];
        hh = a.h1[i];
    }
    const long long bsz = (long long)R * Np;
    unsigned *const own = p.x + (long long)r * Np + i;
    auto publish = [&](long long set) {   // (a NaN of the empty pattern becomes another NaN)
        if (!updates || lane >= 16) return;
        const unsigned u = __float_as_uint(x * kAmpScale);
        store1(own + (set & 3) * bsz, u == kEmpty ? 0x7FC00000u : u);
    };
    publish(p.base);
    __syncthreads();
    if (tid == 0) {
        gone = before != 0;
        if (gone || p.patience < 0) stalled = 1;
    }
    const int k4 = 256 * wave + 4 * lane;   // this lane polls columns k4 .. k4 + 3
    for (int ev = 1; ev <= p.steps; ++ev) {
        const unsigned *src = p.x + ((p.base + ev - 1) & 3) * bsz + k4;
        unsigned long long v[NR][2];
        auto fetch = [&](int q) {
            const unsigned long long *s = reinterpret_cast<const unsigned long long *>(src + (long long)q * Np);
            v[q][0] = load2(s);
            v[q][1] = load2(s + 1);
        };
        for (int q = 0; q < p.pause; ++q) __builtin_amdgcn_s_sleep(1);
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            v[q][0] = v[q][1] = 0ull;
            if (q < R && k4 < Np) fetch(q);
        }
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            long long since = 0;
            while (__any(empty2(v[q][0]) || empty2(v[q][1]))) {
                const long long now = wall_clock64();
                if (since == 0) since = now;
                if (now - since > p.patience || *(volatile int *)&stalled) {
                    stalled = 1;
                    break;
                }
                if (k4 < Np) fetch(q);
            }
            if (q < R) {
                const f32x4 b = {__uint_as_float((unsigned)v[q][0]), __uint_as_float((unsigned)(v[q][0] >> 32)),
                                 __uint_as_float((unsigned)v[q][1]), __uint_as_float((unsigned)(v[q][1] >> 32))};
                u32x4 x0, x1, x2;
                split8(b, f32x4{0.0f, 0.0f, 0.0f, 0.0f}, x0, x1, x2);
                *reinterpret_cast<uint2 *>(&xl[wave][3 * q][8 * lane]) = make_uint2(x0[0], x0[1]);
                *reinterpret_cast<uint2 *>(&xl[wave][3 * q + 1][8 * lane]) = make_uint2(x1[0], x1[1]);
                *reinterpret_cast<uint2 *>(&xl[wave][3 * q + 2][8 * lane]) = make_uint2(x2[0], x2[1]);
            }
        }
        // the wave's own LDS writes, read by its other lanes (LDS operations
        // of a wave complete in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // (the same order of the sums for both forms of J: the smaller pieces of
        // couplings that are exact in FP8 are zero)
        f32x4 c0 = {0.0f, 0.0f, 0.0f, 0.0f}, c1 = c0, c2 = c0;
        const bool has = col < 3 * R;
        const unsigned char *xp = xl[wave][has ? col : 0] + 16 * kq;
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            u32x4 b = *reinterpret_cast<const u32x4 *>(xp + 64 * f);
            if (!has) b = u32x4{0u, 0u, 0u, 0u};
            f32x4 &c = f & 1 ? c1 : c0;
            if constexpr (J8) {
                c = mfma16(widen8<OP_F32>(j8[f].x, j8[f].y), b, c);
            } else {
                c2 = mfma16(j[f][2], b, c2);
                c2 = mfma16(j[f][1], b, c2);
                c = mfma16(j[f][0], b, c);
            }
        }
        if (has) *reinterpret_cast<f32x4 *>(&red[ev & 1][wave][has ? col : 0][4 * kq]) = J8 ? c0 + c1 : (c0 + c1) + c2;
        // (also: the empty marks this wave stored in the last step have arrived)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (stalled) break;
        if (updates) {
            float hi = 0.0f, lo = 0.0f;
            for (int w = kq; w < nw; w += 4) {
                hi += red[ev & 1][w][3 * r][col];
                lo += red[ev & 1][w][3 * r + 1][col] + red[ev & 1][w][3 * r + 2][col];
            }
            hi += __shfl_xor(hi, 16);
            lo += __shfl_xor(lo, 16);
            hi += __shfl_xor(hi, 32);
            lo += __shfl_xor(lo, 32);
            const float c = hi + lo, rho = x * x;
            const float f = x * (gm - a.gamma_c - rho) + c * a.inv_s + hh;
            gm += a.dt * (ep * (a.rho_th - rho));
            x += a.dt * f;
            if (a.noise_amp != 0.0f) {
                float g0, g1;
                noise_pair(mix64(p.seed ^ mix64((unsigned long long)(p.t0 + ev - 1))), r, i, g0, g1);
                x += a.noise_amp * g0;
            }
            if (!inside) x = gm = 0.0f;
            if (ev < p.steps) publish(p.base + ev);
            if (lane < 16) store1(own + ((p.base + ev + 2) & 3) * bsz, kEmpty);
        }
    }
    if (stalled && tid == 0 && !gone) store_agent(p.stalled, p.tag);
    if (inside && lane < 16 && !stalled) {
        a.psi_out[(long long)r * Np + i] = x;
        if (tiny_number(x)) store_agent(a.tiny, 1);
        a.gam_out[(long long)r * Np + i] = gm;
        if (!(gd_finite(x) && gd_finite(gm))) store_agent(a.flags + r, 1);
    }
    if (ce.out && last_arrival(ce.count, gridDim.x)) check_end(ce);   // the end of a run
}

}  // namespace

// {FR, RB}: fragments of 32 couplings per wave (Np <= 256 FR), blocks of 16
// rows (8, 4 with FP8 couplings only)
#define GD_PERSIST_VARIANTS(X) X(0, 4, 1) X(1, 4, 2) X(2, 4, 4) X(3, 8, 1) X(4, 8, 2) X(5, 8, 4)

namespace {
constexpr int kCfg[][2] = {
#define GD_ROW(id, fr, rb) {fr, rb},
    GD_PERSIST_VARIANTS(GD_ROW)
#undef GD_ROW
};

template <int FR, int RB>
const void *kernel_of(bool cplx, bool rk4, bool j8) {
    if constexpr (FR * RB > 16) {   // the pieces of J do not fit the registers
        if (!j8) return nullptr;
        if (cplx)
            return rk4 ? (const void *)&persist_step_k<FR, RB, true, true, true>
                       : (const void *)&persist_step_k<FR, RB, true, false, true>;
        return rk4 ? (const void *)&persist_step_k<FR, RB, false, true, true>
                   : (const void *)&persist_step_k<FR, RB, false, false, true>;
    } else {
    if (cplx)
        return rk4 ? (j8 ? (const void *)&persist_step_k<FR, RB, true, true, true>
                         : (const void *)&persist_step_k<FR, RB, true, true, false>)
                   : (j8 ? (const void *)&persist_step_k<FR, RB, true, false, true>
                         : (const void *)&persist_step_k<FR, RB, true, false, false>);
    return rk4 ? (j8 ? (const void *)&persist_step_k<FR, RB, false, true, true>
                     : (const void *)&persist_step_k<FR, RB, false, true, false>)
               : (j8 ? (const void *)&persist_step_k<FR, RB, false, false, true>
                     : (const void *)&persist_step_k<FR, RB, false, false, false>);
    }
}

// ids from kFew on: few trajectories, NR 1, 2, 4
constexpr int kFew = 8;

const void *few_kernel(int id, bool j8) {
    switch (id - kFew) {
    case 0: return j8 ? (const void *)&persist_few_k<1, true> : (const void *)&persist_few_k<1, false>;
    case 1: return j8 ? (const void *)&persist_few_k<2, true> : (const void *)&persist_few_k<2, false>;
    case 2: return j8 ? (const void *)&persist_few_k<4, true> : (const void *)&persist_few_k<4, false>;
    }
    return nullptr;
}

const void *kernel_id(int id, bool cplx, bool rk4, bool j8) {
    switch (id) {
#define GD_CASE(id, fr, rb) \
    case id: return kernel_of<fr, rb>(cplx, rk4, j8);
        GD_PERSIST_VARIANTS(GD_CASE)
#undef GD_CASE
    }
    return nullptr;
}
}  // namespace

int persist_groups(int id, bool cplx, int R) { return id >= kFew ? 1 : (R + (cplx ? 7 : 15)) / (cplx ? 8 : 16); }

long long persist_words(int id, bool cplx, int Np, int R) {
    return id >= kFew ? 4ll * R * Np : 4ll * persist_groups(id, cplx, R) * (Np / 32) * 512;
}

// The variant for a problem, or -1.  Few trajectories take the kernel that
// reads no empty columns (N = 1000, R = 1 2.25 us per step, 3.5 in a group of
// 16); a wave updates one trajectory, so R is at most the number of waves.
// Otherwise the fewest rows per workgroup with at most one workgroup per CU.
// In runs of 40 steps every problem that fits is faster this way than with one
// launch per step (from 1.04 times, N = 2000, R = 100: 359 us against 375; N = 300,
// R = 64 102 against 184); larger ones have enough work per step to hide its
// latency.  A call of one step takes 25-46 us against 18-25 (XY RK4 N = 1000 53
// against 48), and 3 to 5 steps the same, but a trajectory does not depend on how
// its steps are cut into calls.  Runs cut by frequent checks: choose_persist.
int persist_variant(bool cplx, bool rk4, bool j8, int Np, int R) {
    int dev = 0, cus = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop)
        return -1;
    auto resident = [&](const void *k, int threads, long long blocks) {
        int occ = 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, threads, 0) == hipSuccess && occ >= 1 && blocks <= cus;
    };
    if (!cplx && !rk4 && R <= 4 && Np <= 4096 && 256 * (R - 1) < Np) {
        const int id = kFew + (R > 2 ? 2 : R - 1);
        if (resident(few_kernel(id, j8), (Np + 255) / 256 * 64, Np / 16)) return id;
    }
    for (int id = 0; id < int(sizeof(kCfg) / sizeof(kCfg[0])); ++id) {
        const void *k = kernel_id(id, cplx, rk4, j8);
        if (!k || Np > 256 * kCfg[id][0]) continue;
        const long long rows = 16 * kCfg[id][1];
        if (resident(k, 64 * kWaves, (Np + rows - 1) / rows * persist_groups(id, cplx, R))) return id;
    }
    return -1;
}

// The kernel for few trajectories also ends a run (gd_check.h); in the other one
// the code for it costs registers: XY N = 1000, R = 128 388 us per 80
// evaluations, 416 with it
bool persist_ends_run(int id) { return id >= kFew; }

hipError_t launch_persist(int id, bool cplx, bool rk4, bool j8, const DenseStepArgs &a, const PersistArgs &p,
                          const CheckEnd &ce, hipStream_t st) {
    if (a.Np % 64 || a.R < 1 || p.steps < 1 || !p.tag || a.sum_exp != 0 || a.psi_out == a.psi_in || a.gam_out == a.gam_in || ce.E ||
        (ce.out && (!persist_ends_run(id) || ce.R != a.R || !ce.count || !ce.flags)))
        return hipErrorInvalidValue;
    DenseStepArgs x = a;
    PersistArgs y = p;
    y.groups = persist_groups(id, cplx, a.R);
    y.pause = id < kFew ? kPause : a.Np > 1024 ? kPauseFewLarge : kPauseFew;
    CheckEnd z = ce;
    void *args[] = {&x, &y, &z};   // (the last for few trajectories only)
    if (id >= kFew) {
        const void *k = few_kernel(id, j8);
        if (!k || cplx || rk4 || a.Np > 4096 || a.R > (1 << (id - kFew)) || 256 * (a.R - 1) >= a.Np)
            return hipErrorInvalidValue;
        return hipLaunchCooperativeKernel(k, dim3(a.Np / 16), dim3((a.Np + 255) / 256 * 64), args, 0, st);
    }
    const void *k = kernel_id(id, cplx, rk4, j8);
    if (!k || a.Np > 256 * kCfg[id][0]) return hipErrorInvalidValue;
    const int rows = 16 * kCfg[id][1];
    return hipLaunchCooperativeKernel(k, dim3((a.Np + rows - 1) / rows * y.groups), dim3(64 * kWaves), args, 0, st);
}

}  // namespace gd

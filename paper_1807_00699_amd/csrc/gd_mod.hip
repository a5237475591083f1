// GD-mod step (Sec. 1): the coupling of Eq. (main) is Delta_ij K_ij with
// Delta_ij = gamma_i + gamma_j, and every trajectory carries its own coupling
// matrix K that follows Eq. (gamma2), dK_ij/dt = eps_hat (J_ij - Delta_ij K_ij).
//
// One explicit Euler step, all right-hand sides at the old state:
//   c_i   = sum_j (gamma_i + gamma_j) K_ij Psi_j          (raw sum; 1/s in the epilogue)
//   K_ij += dt eps_hat (J_ij - (gamma_i + gamma_j) K_ij)
// followed by the pointwise update of Eq. (main, gamma) shared with the dense
// kernels (gd_epilogue.h).  The diagonal needs no test: J_ii = 0 and K_ii(0)
// = 0, so K_ii stays 0 and adds nothing.
//
// Every K element is read and written once per step: a batched matrix-vector
// product bound by K's traffic (J rows are shared by all trajectories and come
// from L2), not a GEMM.  Sets of K past the last-level cache keep one triangle
// of each (gdmod_sym_k below), which halves that traffic: XY N = 1024, R = 128
// 192 -> 122 us per step (570 MB at 5.0 TB/s; a copy reaches 5.2), R = 256
// 382 -> 235, N = 512, R = 128 51 -> 41.  Its second launch costs more than that
// saves where K stays in the cache: N = 1000, R = 16 27 us full, 29 packed; N =
// 500, R = 16 9.4 and 16; equal at N = 500, R = 64 (67 MB).
//
// Full K: grid (Np / 16 row blocks, R trajectories), 256 threads.  The
// workgroup stages its trajectory's amplitudes and gains in LDS, each wave
// sweeps 4 consecutive rows with 16-byte loads (64 lanes x 4 columns per
// instruction, fully coalesced), reduces each row across the wave, and lane 0
// applies the epilogue to the 4 rows.
#include "gd_epilogue.h"

namespace gd {

namespace {

constexpr int kModRowsPerWave = 4;
constexpr int kModWaves = 4;
constexpr int kModRows = kModRowsPerWave * kModWaves;

template <bool CPLX>
__global__ void __launch_bounds__(64 * kModWaves)
gdmod_euler_k(DenseStepArgs a, const float *__restrict__ J, float *__restrict__ K, float c_hat) {
    extern __shared__ float sh[];   // [Np] gamma, [Np] Re Psi, [Np] Im Psi (complex)
    const int Np = a.Np;
    const int r = blockIdx.y;
    const long long ps = a.plane_stride;
    float *sg = sh, *sx = sh + Np, *sy = sh + 2 * Np;
    for (int j = threadIdx.x * 4; j < Np; j += 64 * kModWaves * 4) {
        const long long o = (long long)r * Np + j;
        *reinterpret_cast<f32x4 *>(sg + j) = *reinterpret_cast<const f32x4 *>(a.gam_in + o);
        *reinterpret_cast<f32x4 *>(sx + j) = *reinterpret_cast<const f32x4 *>(a.psi_in + o);
        if (CPLX) *reinterpret_cast<f32x4 *>(sy + j) = *reinterpret_cast<const f32x4 *>(a.psi_in + ps + o);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i0 = blockIdx.x * kModRows + wave * kModRowsPerWave;
    f32x4 cr = {0.f, 0.f, 0.f, 0.f}, ci = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < kModRowsPerWave; ++q) {
        const int i = i0 + q;
        const float gi = sg[i];
        float *Kr = K + ((long long)r * Np + i) * Np;
        const float *Jr = J + (long long)i * Np;
        float sre = 0.0f, sim = 0.0f;
        // KU chunks of 256 columns per pass: all their K and J loads are in
        // flight together (K is streamed: non-temporal loads and stores)
        constexpr int KU = 4;
        for (int j0 = lane * 4; j0 < Np; j0 += 256 * KU) {
            f32x4 k[KU], jj[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int j = j0 + 256 * u;
                if (j < Np) {
                    k[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Kr + j));
                    jj[u] = *reinterpret_cast<const f32x4 *>(Jr + j);
                }
            }
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int j = j0 + 256 * u;
                if (j >= Np) break;
                const f32x4 gj = *reinterpret_cast<const f32x4 *>(sg + j);
                const f32x4 xj = *reinterpret_cast<const f32x4 *>(sx + j);
                f32x4 yj = {0.f, 0.f, 0.f, 0.f};
                if (CPLX) yj = *reinterpret_cast<const f32x4 *>(sy + j);
                f32x4 kn;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d = gi + gj[e];
                    const float dk = d * k[u][e];
                    sre += dk * xj[e];
                    if (CPLX) sim += dk * yj[e];
                    kn[e] = k[u][e] + c_hat * (jj[u][e] - dk);
                }
                __builtin_nontemporal_store(kn, reinterpret_cast<f32x4 *>(Kr + j));
            }
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            sre += __shfl_xor(sre, m);
            if (CPLX) sim += __shfl_xor(sim, m);
        }
        cr[q] = sre;
        ci[q] = sim;
    }
    if (lane == 0) {
        const bool bad = step_epilogue4<MODE_EULER, CPLX, OP_F32>(a, i0, r, true, cr, ci);
        if (bad) a.flags[r] = 1;
    }
}

// K in packed form: J is exactly symmetric, and with it K for good (both
// triangles follow the same operations), so one triangle is kept: 64 x 64 tiles
// (I, J >= I), tile rows one after the other, each tile row-major.
__host__ __device__ inline long long tiles_before(int strip, int nt) {
    return (long long)strip * nt - (long long)strip * (strip - 1) / 2;
}

__global__ void mod_pack_k(const float *__restrict__ J, float *__restrict__ K, int Np, int R) {
    const int nt = Np / 64;
    const long long per = tiles_before(nt, nt) * 4096, total = per * R / 4;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total; q += (long long)gridDim.x * blockDim.x) {
        const long long at = q * 4 % per;
        const long long tile = at / 4096;
        int strip = 0;
        while (tiles_before(strip + 1, nt) <= tile) ++strip;
        const int e = int(at % 4096);
        const long long row = strip * 64 + e / 64, col = (strip + (tile - tiles_before(strip, nt))) * 64 + e % 64;
        *reinterpret_cast<f32x4 *>(K + q * 4) = *reinterpret_cast<const f32x4 *>(J + row * Np + col);
    }
}

__global__ void mod_unpack_k(const float *__restrict__ K, float *__restrict__ out, int Np, int n) {
    const int nt = Np / 64;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < (long long)n * n;
         q += (long long)gridDim.x * blockDim.x) {
        int i = int(q / n), j = int(q % n);
        if (i / 64 > j / 64) {
            const int h = i;
            i = j;
            j = h;
        }
        out[q] = K[(tiles_before(i / 64, nt) + (j / 64 - i / 64)) * 4096 + i % 64 * 64 + j % 64];
    }
}

// Sum over the 16 lanes of a row of lanes of v[0 .. 15]; lane l gets that of v[l % 16]
__device__ inline float row_transpose_sum(float (&v)[16], int lane) {
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) {
        const bool up = lane & m;
#pragma unroll
        for (int q = 0; q < m; ++q) {
            const float keep = up ? v[q + m] : v[q], send = up ? v[q] : v[q + m];
            v[q] = keep + __shfl_xor(send, m);
        }
    }
    return v[0];
}

// One tile row of one trajectory: its tiles updated in place, and their
// products: part[r][strip][plane][j] gets, for j in the strip's own rows, the
// sums along the tile row, and for j beyond them the sums down the tiles
// (the products of the other triangle).  A wave takes every fourth tile, all 64
// rows of it: 16-byte loads, four tile rows each.
template <bool CPLX>
__global__ void __launch_bounds__(256)
gdmod_sym_k(DenseStepArgs a, const float *__restrict__ J, float *__restrict__ K, float *__restrict__ part, float c_hat) {
    extern __shared__ float sh[];   // [Np] gamma, [Np] Re Psi, [Np] Im Psi (complex)
    __shared__ float red[CPLX ? 2 : 1][4][64];
    const int Np = a.Np, nt = Np / 64;
    const int strip = blockIdx.x / a.R, r = blockIdx.x % a.R;   // the longest first
    const long long ps = a.plane_stride;
    float *sg = sh, *sx = sh + Np, *sy = sh + 2 * Np;
    for (int j = strip * 64 + threadIdx.x * 4; j < Np; j += 1024) {
        const long long o = (long long)r * Np + j;
        *reinterpret_cast<f32x4 *>(sg + j) = *reinterpret_cast<const f32x4 *>(a.gam_in + o);
        *reinterpret_cast<f32x4 *>(sx + j) = *reinterpret_cast<const f32x4 *>(a.psi_in + o);
        if (CPLX) *reinterpret_cast<f32x4 *>(sy + j) = *reinterpret_cast<const f32x4 *>(a.psi_in + ps + o);
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane >> 4, lc = (lane & 15) * 4;
    const int row0 = strip * 64 + lr;      // this lane's rows: row0 + 4 u
    float gi[16], xi[16], yi[16], sr[16], si[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        gi[u] = sg[row0 + 4 * u];
        xi[u] = sx[row0 + 4 * u];
        yi[u] = CPLX ? sy[row0 + 4 * u] : 0.0f;
        sr[u] = si[u] = 0.0f;
    }
    float *Ks = K + ((long long)r * tiles_before(nt, nt) + tiles_before(strip, nt)) * 4096 + lane * 4;
    float *out = part + ((long long)r * nt + strip) * (CPLX ? 2 : 1) * Np;
    for (int t = wave; t < nt - strip; t += 4) {
        float *Kt = Ks + (long long)t * 4096;
        const int col = (strip + t) * 64 + lc;
        const float *Jt = J + (long long)row0 * Np + col;
        const f32x4 gj = *reinterpret_cast<const f32x4 *>(sg + col);
        const f32x4 xj = *reinterpret_cast<const f32x4 *>(sx + col);
        f32x4 yj = {0.f, 0.f, 0.f, 0.f};
        if (CPLX) yj = *reinterpret_cast<const f32x4 *>(sy + col);
        f32x4 cr = {0.f, 0.f, 0.f, 0.f}, ci = cr;
        constexpr int KU = 8;
#pragma unroll
        for (int u0 = 0; u0 < 16; u0 += KU) {
            f32x4 k[KU], jj[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                k[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(Kt + (u0 + u) * 256));
                jj[u] = *reinterpret_cast<const f32x4 *>(Jt + (long long)(u0 + u) * 4 * Np);
            }
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                f32x4 kn;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float dk = (gi[u0 + u] + gj[e]) * k[u][e];
                    sr[u0 + u] += dk * xj[e];
                    cr[e] += dk * xi[u0 + u];
                    if (CPLX) {
                        si[u0 + u] += dk * yj[e];
                        ci[e] += dk * yi[u0 + u];
                    }
                    kn[e] = k[u][e] + c_hat * (jj[u][e] - dk);
                }
                __builtin_nontemporal_store(kn, reinterpret_cast<f32x4 *>(Kt + (u0 + u) * 256));
            }
        }
        if (t > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                cr[e] += __shfl_xor(cr[e], 16);
                cr[e] += __shfl_xor(cr[e], 32);
                if (CPLX) {
                    ci[e] += __shfl_xor(ci[e], 16);
                    ci[e] += __shfl_xor(ci[e], 32);
                }
            }
            if (lr == 0) *reinterpret_cast<f32x4 *>(out + col) = cr;
            if (CPLX && lr == 0) *reinterpret_cast<f32x4 *>(out + Np + col) = ci;
        }
    }
    // lane: row 4 (lane % 16) + lr of the strip
    red[0][wave][4 * (lane & 15) + lr] = row_transpose_sum(sr, lane);
    if (CPLX) red[CPLX][wave][4 * (lane & 15) + lr] = row_transpose_sum(si, lane);
    __syncthreads();
    if (threadIdx.x < (CPLX ? 128 : 64)) {
        const int p = threadIdx.x >> 6, q = threadIdx.x & 63;
        out[p * Np + strip * 64 + q] = (red[p][0][q] + red[p][1][q]) + (red[p][2][q] + red[p][3][q]);
    }
}

// Adds the partial sums of the strips up to each row's own, in order, and
// updates amplitudes and gains
template <bool CPLX>
__global__ void __launch_bounds__(256) gdmod_sum_k(DenseStepArgs a, const float *__restrict__ part) {
    const int Np = a.Np, nt = Np / 64;
    const long long q = blockIdx.x * 256ll + threadIdx.x;
    if (q >= (long long)a.R * (Np / 4)) return;
    const int r = int(q / (Np / 4)), i0 = int(q % (Np / 4)) * 4;
    constexpr int PL = CPLX ? 2 : 1, U = 8;
    const float *p = part + (long long)r * nt * PL * Np + i0;
    EpiIn in;
    epi_load<MODE_EULER, CPLX>(a, i0, r, in);
    f32x4 cr = {0.f, 0.f, 0.f, 0.f}, ci = cr;
    const int last = i0 / 64;
    for (int s0 = 0; s0 <= last; s0 += U) {   // U loads in flight
        f32x4 vr[U], vi[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float *q = p + (long long)min(s0 + u, last) * PL * Np;
            vr[u] = *reinterpret_cast<const f32x4 *>(q);
            if (CPLX) vi[u] = *reinterpret_cast<const f32x4 *>(q + Np);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u <= last) {
                cr += vr[u];
                if (CPLX) ci += vi[u];
            }
    }
    if (epi_apply<MODE_EULER, CPLX, OP_F32>(a, i0, r, true, in, cr, ci)) a.flags[r] = 1;
}

}  // namespace

long long gdmod_packed_floats(int Np) { return tiles_before(Np / 64, Np / 64) * 4096; }
long long gdmod_part_floats(bool cplx, int Np, int R) { return (long long)R * (Np / 64) * (cplx ? 2 : 1) * Np; }

hipError_t launch_gdmod_pack(const float *J, float *K, int Np, int R, hipStream_t st) {
    mod_pack_k<<<2048, 256, 0, st>>>(J, K, Np, R);
    return hipGetLastError();
}

hipError_t launch_gdmod_unpack(const float *K, float *out, int Np, int n, hipStream_t st) {
    mod_unpack_k<<<1024, 256, 0, st>>>(K, out, Np, n);
    return hipGetLastError();
}

hipError_t launch_gdmod_sym(bool complex_mode, const DenseStepArgs &a, const float *J, float *K, float *part, float c_hat,
                            hipStream_t st) {
    if (a.Np % 64 || a.R < 1) return hipErrorInvalidValue;
    const size_t lds = gdmod_lds_bytes(complex_mode, a.Np);
    if (lds > 65536) return hipErrorInvalidValue;
    const unsigned grid = unsigned(a.Np / 64) * a.R, tail = unsigned(((long long)a.R * (a.Np / 4) + 255) / 256);
    if (complex_mode) {
        gdmod_sym_k<true><<<grid, 256, lds, st>>>(a, J, K, part, c_hat);
        gdmod_sum_k<true><<<tail, 256, 0, st>>>(a, part);
    } else {
        gdmod_sym_k<false><<<grid, 256, lds, st>>>(a, J, K, part, c_hat);
        gdmod_sum_k<false><<<tail, 256, 0, st>>>(a, part);
    }
    return hipGetLastError();
}

size_t gdmod_lds_bytes(bool complex_mode, int Np) { return size_t(complex_mode ? 3 : 2) * Np * sizeof(float); }

hipError_t launch_gdmod(bool complex_mode, const DenseStepArgs &a, const float *J, float *K, float c_hat,
                        hipStream_t st) {
    if (a.Np % kModRows || a.R < 1) return hipErrorInvalidValue;
    const size_t lds = gdmod_lds_bytes(complex_mode, a.Np);
    if (lds > 65536) return hipErrorInvalidValue;
    const dim3 grid(a.Np / kModRows, a.R), block(64 * kModWaves);
    if (complex_mode)
        gdmod_euler_k<true><<<grid, block, lds, st>>>(a, J, K, c_hat);
    else
        gdmod_euler_k<false><<<grid, block, lds, st>>>(a, J, K, c_hat);
    return hipGetLastError();
}

}  // namespace gd

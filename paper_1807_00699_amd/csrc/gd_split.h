// FP32 coupling step on the BF16 matrix cores: the coupling product of
// Eq. (main) with every FP32 amplitude split into three BF16 pieces,
//   x = x0 + x1 + x2   (x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1),
// exactly: 3 x 8 significant bits hold the 24 of an FP32 number, both
// differences are exact, and so is each product of two pieces in the FP32
// accumulators of v_mfma_f32_32x32x16_bf16.  The pieces of small numbers would
// leave BF16's range (the last bit of 2^-110 is 2^-133), so J is split in units
// of a power of two next to its largest magnitude, and amplitudes times 2^24
// once a step has written one below 2^-100 (*a.tiny): the last bit of any FP32
// number is a normal BF16 then.  The sums are scaled back.  That is a simple
// loop of its own before the pipelined one: a multiplication before every split
// cost 2% (N = R = 4096) to 12% (N = 3001, R = 1500), one of each chunk in LDS,
// where it is not even executed, 4% (the compiler's schedule).  Couplings that are exact in FP8
// (E4M3) are one BF16 piece and take three products per amplitude; any other
// J is split the same way and takes six (j0 x0, j0 x1, j1 x0, j1 x1, j0 x2,
// j2 x0; the three left out are below 2^-24 of j x).
//
// Error of the sums against 64 bits, relative to the sums (2-norm; with
// v_mfma_f32_16x16x4_f32 in brackets): couplings {-1, 0, 1} N = 1000 5-8e-8,
// N = 4096 6-8e-8 (5.6e-7 in the 256-row tiles, which have no registers for a
// second accumulator) [4.0e-7, 8.1e-7]; U[-10, 10] N = 1000 0.9-4.7e-7
// [5.7e-7]; N(0, 1/N) N = 4096 0.12-1.0e-6 [1.15e-6].
//
// BF16 and FP16 operands (FP8 couplings) take one product; the amplitudes are
// then the 16-bit copies that the previous step wrote.
//
// What bounds it: at N = R = 4096 the matrix cores.  One launch is 3 x 137
// GFLOP; it takes 322 us (1.28 PFLOP/s; a large BF16 matrix product runs at
// 1.28 on this card), against 1016 us on the FP32 matrix cores (135 TFLOP/s,
// 86% of their peak); with BF16 operands, one product, 126 us, where the matrix
// work (108 us) and the state update of all workgroups at once follow each
// other.  XY N = R = 1024 31-32 us per stage (45 before): eight K chunks take 20
// us, at the matrix rate, the state update and the start of the launch 11.
// Smaller problems are bound by the latency of the first loads and by the LDS
// reads and the splitting (5.5 vector instructions per amplitude) around each
// matrix instruction: Ising N = 800, R = 100 7.0 us per step (20.2 before), XY
// N = 1000, R = 128 8.6 us per stage (23.5); where J fits the registers of the
// chip they run gd_persist.hip instead.
#pragma once
#include "gd_epilogue.h"

#include <type_traits>
#include <utility>

namespace gd {
namespace split {

// Storage of J: FP8 (E4M3, exact) or its three BF16 pieces; J_FP8_SIGN: FP8
// couplings against the signs of the amplitudes (energies of Ising readouts),
// one product
enum JKind : int { J_FP8 = 0, J_PIECES = 1, J_FP8_SIGN = 2 };

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lvoid_t;

// s_waitcnt immediate: at most n vector-memory operations of this wave
// outstanding, all its LDS operations complete (expcnt at its maximum)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// the 16-byte slot of an LDS row that holds logical slot 0 (XOR swizzle): 16
// consecutive rows read at one logical slot then cover all 64 banks
template <int ROWB>
__device__ inline int row_swz(int row) {
    static_assert(ROWB == 64 || ROWB == 128 || ROWB == 256, "rows of 4, 8 or 16 slots");
    return ROWB == 64 ? (row >> 2) & 3 : ROWB == 128 ? (row >> 1) & 7 : row & 15;
}

// 2^e v
__device__ inline f32x4 ldexp4(f32x4 v, int e) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __builtin_ldexpf(v[q], e);
    return v;
}

constexpr float kAmpScale = float(1 << kAmpExp);

// the three BF16 pieces of eight consecutive FP32 values
__device__ inline void split8(const f32x4 &lo, const f32x4 &hi, u32x4 &p0, u32x4 &p1, u32x4 &p2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float a = q < 2 ? lo[2 * q] : hi[2 * q - 4];
        const float b = q < 2 ? lo[2 * q + 1] : hi[2 * q - 3];
        const unsigned int w0 = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{a, b}, bf16x2));
        const float ra = a - __uint_as_float(w0 << 16), rb = b - __uint_as_float(w0 & 0xFFFF0000u);
        const unsigned int w1 = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{ra, rb}, bf16x2));
        const float sa = ra - __uint_as_float(w1 << 16), sb = rb - __uint_as_float(w1 & 0xFFFF0000u);
        p0[q] = w0;
        p1[q] = w1;
        p2[q] = __builtin_bit_cast(unsigned int, __builtin_convertvector(f32x2{sa, sb}, bf16x2));
    }
}

// the signs (+-1 as BF16, sign(+-0) = +1) of eight consecutive values
__device__ inline u32x4 sign8(const f32x4 &lo, const f32x4 &hi) {
    u32x4 p;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float a = q < 2 ? lo[2 * q] : hi[2 * q - 4];
        const float b = q < 2 ? lo[2 * q + 1] : hi[2 * q - 3];
        p[q] = (a < 0.0f ? 0xBF80u : 0x3F80u) | (b < 0.0f ? 0xBF800000u : 0x3F800000u);
    }
    return p;
}

// eight FP8 (E4M3) values in two dwords -> eight BF16 or FP16 values (exact)
template <int OPT>
__device__ inline u32x4 widen8(unsigned int w0, unsigned int w1) {
    u32x4 r;
    if constexpr (OPT == OP_F16) {
        r[0] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, 1.0f, false));
        r[1] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, 1.0f, true));
        r[2] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, 1.0f, false));
        r[3] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, 1.0f, true));
    } else {
        r[0] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, false));
        r[1] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w0, 1.0f, true));
        r[2] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, false));
        r[3] = __builtin_bit_cast(unsigned int, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w1, 1.0f, true));
    }
    return r;
}

template <int OPT = OP_F32>
__device__ inline f32x16 mfma(const u32x4 &a, const u32x4 &b, const f32x16 &c) {
    if constexpr (OPT == OP_F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                      0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                       0, 0);
}

// Workgroup -> (row tile, column tile): one contiguous range of tiles per XCD
// (consecutive workgroup ids go to the XCDs in turn), in groups of 8 row
// tiles, so that an XCD's L2 keeps its rows of J and its amplitudes.
__device__ inline void tile_of(int b, int nblk, int n_mt, int n_ct, int &mt, int &ct) {
    int t = b;
    if ((nblk & 7) == 0) t = (b & 7) * (nblk >> 3) + (b >> 3);
    const int gm = 8, width = gm * n_ct, first = t / width * gm;
    const int gsz = min(gm, n_mt - first), in = t % width;
    mt = first + in % gsz;
    ct = in / gsz;
}

// Tile BM rows x BN GEMM columns (complex: BN / 2 trajectories; the TN
// columns of a wave are the real parts of TN / 2 trajectories, then their
// imaginary parts).  KS groups of WM x WN waves take the K chunks g, g + KS,
// ... of the same tile, and the groups' sums are added in a fixed order
// through LDS.  A group of one wave needs no barrier in its K loop: it waits
// for its own copies only.
//
// Amplitudes: each group keeps NSTG chunks of its columns in LDS as FP32 rows
// of BK, copied from global memory straight to LDS with the
// 16-byte slots XOR-swizzled by row, and splits them after the LDS read.
// Couplings: loaded straight into registers, JD chunks ahead, from a copy
// laid out in the lane order of the matrix instruction (every load of a wave
// is one contiguous KiB); through LDS, as the amplitudes, XY N = R = 1024 took
// 39 us per stage and N = 800 7.7 us per step:
//   J_FP8:    [Np / 32][Np / 32][lane][16 bytes], lane l holds row l % 32,
//             k = 16 (l / 32) .. + 15 of the 32-wide block: its first eight
//             are operands of one slice, the others of the next;
//   J_PIECES: [Np / 32][Np / 16][piece][lane][8 BF16], k = 8 (l / 32) + e.
template <int BM, int BN, int BK, int WM, int WN, int KS, int JD, bool CPLX, int MODE, int JK,
          int OPT = OP_F32>
__global__ void __launch_bounds__(64 * WM * WN * KS) dense_step_split(DenseStepArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass has no buffer resources; it needs the kernel's stub only
    constexpr int NWG = WM * WN, NT = 64 * NWG * KS;
    constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
    constexpr int PL = CPLX ? 2 : 1, TRAJ = BN / PL, TRW = TN / PL;   // trajectories per tile / wave column
    constexpr int NSL = BK / 16;                                      // 16-wide K slices per chunk
    constexpr bool F32 = OPT == OP_F32;
    constexpr bool J8 = JK != J_PIECES, SIGN = JK == J_FP8_SIGN;
    static_assert(!SIGN || (MODE == MODE_ENERGY && !CPLX && F32), "signs: energies of one plane");
    static_assert(F32 || J8, "16-bit operands: FP8 couplings");
    constexpr int EB = F32 ? 4 : 2;                                   // bytes per amplitude of the operand
    constexpr int RB = EB * BK, TILEB = BN * RB, NI = TILEB / 1024;   // bytes per LDS row; 1 KiB copies per chunk
    constexpr int NCW = NI / NWG;                                     // copies per wave and chunk
    constexpr int JPC = J8 ? NSL / 2 : 3 * NSL, NJ = MB * JPC;        // coupling loads per row block / wave and chunk
    static_assert(BK % 32 == 0 && NI % NWG == 0 && (NI / NWG) * NWG * 1024 == TILEB, "chunks of whole 32-wide blocks");
    static_assert((JD - 1) * NCW + JD * NJ < 64, "outstanding operations fit the wait counter");
    // the update: passes over wave columns when the tile's sums do not fit LDS at once
    constexpr int TP = BM + 4;                                        // LDS pitch of one trajectory's rows
    constexpr int LOOPB = (JD + 1) * KS * TILEB;
    constexpr bool ONE_PASS = KS * PL * TRAJ * TP * 4 <= (LOOPB > 81920 ? LOOPB : 81920);
    constexpr int NPASS = ONE_PASS ? 1 : WN;
    constexpr int TRP = TRAJ / NPASS;
    constexpr int STB = KS * PL * TRP * TP * 4;
    constexpr int LDSB = LOOPB > STB ? LOOPB : STB;
    static_assert(LDSB <= 160 * 1024, "LDS of one workgroup");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[LDSB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int grp = __builtin_amdgcn_readfirstlane(tid / (64 * NWG));
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) % NWG);
    const int wm = wave % WM, wn = wave / WM;
    const int l32 = lane & 31, lh = lane >> 5;
    const int n_mt = (a.Np + BM - 1) / BM, n_ct = (a.R + TRAJ - 1) / TRAJ;
    int tiny = 0;
    if constexpr (F32 && MODE != MODE_ENERGY) tiny = *(const __attribute__((address_space(4))) int *)a.tiny;
    int mt, ct;
    tile_of(blockIdx.x, gridDim.x, n_mt, n_ct, mt, ct);
    const int m0 = mt * BM, r0 = ct * TRAJ;
    const long long Np = a.Np;

    // update groups (trajectory, 4 rows) of this thread; when they are few
    // their state operands are loaded first, under the whole K loop
    constexpr int RG = BM / 4, NGRP = TRP * RG;
    constexpr int NU = (NGRP + NT - 1) / NT;
    static_assert(NGRP % 64 == 0 && RG <= 64, "whole waves update whole trajectories' row groups");
    constexpr bool EARLY = NPASS == 1 && MODE != MODE_ENERGY &&
                           NU * 4 * (epi_fields<MODE, CPLX>() + 2) + MB * NB * 16 + JD * NJ * 4 <= 140;
    EpiIn pre[EARLY ? NU : 1];
    if constexpr (EARLY) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int g = tid + u * NT, i0 = m0 + (g % RG) * 4, r = r0 + g / RG;
            if (g < NGRP && i0 < a.Np && r < a.R) epi_load<MODE, CPLX>(a, i0, r, pre[u]);
        }
    }

    // Copies: row group u of this wave starts at a wave-uniform trajectory
    // and plane (one buffer resource each: buffer loads, unlike global ones to
    // LDS, leave the waits of other loads and LDS reads exact); this lane adds
    // its row and slot.  Trajectories past the planes read the last one; their
    // sums are not used.
    constexpr int LPR = RB / 16, RPC = 64 / LPR;       // lanes per row, rows per copy
    static_assert(TRW % RPC == 0, "a copy stays in one plane");
    const unsigned char *Bb = static_cast<const unsigned char *>(a.B);
    __amdgpu_buffer_rsrc_t rsrc[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p)
        rsrc[p] = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char *>(Bb + (p * a.plane_stride + r0 * Np) * EB), 0, -1, 0x00027000);
    int voff[NCW];
#pragma unroll
    for (int u = 0; u < NCW; ++u) {
        const int row = (wave + u * NWG) * RPC + lane / LPR;
        const int ls = (lane % LPR) ^ row_swz<RB>(row);
        const int tr = row / TN * TRW + row % TN % TRW;
        voff[u] = min(tr, a.Rp - 1 - r0) * (a.Np * EB) + ls * 16;
    }
    unsigned char *gl = lds + grp * (JD + 1) * TILEB;
    auto copy_chunk = [&](int k0, int buf) {
#pragma unroll
        for (int u = 0; u < NCW; ++u) {
            const int j = wave + u * NWG;
            const bool im = CPLX && j * RPC % TN >= TRW;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(im ? rsrc[PL - 1] : rsrc[0], (lvoid_t *)(gl + buf * TILEB + j * 1024),
                                                     16, voff[u], k0 * EB, 0, 0);
        }
    };
    // the couplings of each of this wave's row blocks (blocks past the matrix
    // read its last one)
    const u32x4 *jsrc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const long long rb = min(m0 / 32 + wm * MB + mb, a.Np / 32 - 1);
        jsrc[mb] = static_cast<const u32x4 *>(a.J) + rb * (Np / BK) * (JPC * 64);
    }
    u32x4 jw[JD][MB][JPC];
    auto load_j = [&](int kc, int set, int sl) {   // J_PIECES: of slice sl; J_FP8: of the pair that ends at odd sl
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int q = 0; q < JPC; ++q)
                if (J8 ? q == sl / 2 : q / 3 == sl) jw[set][mb][q] = (jsrc[mb] + (long long)(kc * JPC + q) * 64)[lane];
    };

    // the products of the smaller pieces have accumulators of their own where
    // those fit: the large ones then add to sums of their own size only
    constexpr bool LOWACC = F32 && !SIGN && MB * NB <= (J8 ? 4 : 2);
    // split couplings in 32 x 32 tiles: the large products of odd slices too
    constexpr bool ODDACC = !J8 && MB * NB == 1;
    f32x16 acc[MB][NB], low[LOWACC ? MB : 1][LOWACC ? NB : 1], odd;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                acc[mb][nb][v] = 0.0f;
                if constexpr (LOWACC) low[mb][nb][v] = 0.0f;
            }
        if constexpr (ODDACC) odd[v] = 0.0f;
    }

    // the products of slice sl: jword(mb, q) is word q of the chunk's couplings
    auto products = [&](int sl, const u32x4 (&x0)[NB], const u32x4 (&x1)[NB], const u32x4 (&x2)[NB],
                        auto jword) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if constexpr (J8) {
                const u32x4 w = jword(mb, sl / 2);
                const u32x4 j0 = (sl & 1) == 0 ? widen8<OPT>(w[0], w[1]) : widen8<OPT>(w[2], w[3]);
                if constexpr (F32 && !SIGN) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        f32x16 &lo = LOWACC ? low[LOWACC ? mb : 0][LOWACC ? nb : 0] : acc[mb][nb];
                        lo = mfma(j0, x2[nb], lo);
                    }
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        f32x16 &lo = LOWACC ? low[LOWACC ? mb : 0][LOWACC ? nb : 0] : acc[mb][nb];
                        lo = mfma(j0, x1[nb], lo);
                    }
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma<OPT>(j0, x0[nb], acc[mb][nb]);
            } else {
                const u32x4 j0 = jword(mb, 3 * sl), j1 = jword(mb, 3 * sl + 1), j2 = jword(mb, 3 * sl + 2);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    f32x16 &lo = LOWACC ? low[LOWACC ? mb : 0][LOWACC ? nb : 0] : acc[mb][nb];
                    lo = mfma(j0, x2[nb], lo);
                    lo = mfma(j2, x0[nb], lo);
                    lo = mfma(j1, x1[nb], lo);
                    lo = mfma(j0, x1[nb], lo);
                    lo = mfma(j1, x0[nb], lo);
                    f32x16 &hi = ODDACC && (sl & 1) ? odd : acc[mb][nb];
                    hi = mfma(j0, x0[nb], hi);
                }
            }
        }
    };

    // the sums (of 2^amp_exp times the amplitudes) and the update
    auto finish = [&](int amp_exp) __attribute__((always_inline)) {
        if constexpr (ODDACC) acc[0][0] += odd;
        if constexpr (LOWACC) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[mb][nb] += low[mb][nb];
        }

        // ---------------------------------------------------------------- epilogue
        // acc[mb][nb][4q + e]: row wm TM + mb 32 + 8q + 4 lh + e, column l32 of
        // block nb.  The sums are staged in LDS as [group][plane][trajectory][row];
        // then every thread adds the groups' sums of its (trajectory, 4 rows)
        // groups and updates them: consecutive lanes on consecutive spins.
        float *st = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
            __syncthreads();
            if (NPASS == 1 || wn == p) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int c = nb * 32 + l32, plane = CPLX ? c / TRW : 0;
                    const int tr = (NPASS == 1 ? wn * TRW : 0) + (CPLX ? c % TRW : c);
                    float *o = st + ((grp * PL + plane) * TRP + tr) * TP;
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<f32x4 *>(o + wm * TM + mb * 32 + 8 * q + 4 * lh) =
                                f32x4{acc[mb][nb][4 * q], acc[mb][nb][4 * q + 1], acc[mb][nb][4 * q + 2],
                                      acc[mb][nb][4 * q + 3]};
                }
            }
            __syncthreads();
            // UB groups at a time, their state loads in flight together (indices
            // clamped to the planes; groups outside the problem are not written)
            constexpr int UB = EARLY ? NU : (NU < 4 ? NU : 4);
#pragma unroll
            for (int u0 = 0; u0 < NU; u0 += UB) {
                EpiIn in[UB];
                if constexpr (!EARLY && MODE != MODE_ENERGY) {
#pragma unroll
                    for (int v = 0; v < UB; ++v) {
                        const int g = tid + (u0 + v) * NT;
                        epi_load<MODE, CPLX>(a, min(m0 + (g % RG) * 4, a.Np - 4), min(r0 + p * TRP + g / RG, a.R - 1), in[v]);
                    }
                }
#pragma unroll
                for (int v = 0; v < UB && u0 + v < NU; ++v) {
                    const int g = tid + (u0 + v) * NT;
                    if (NGRP % NT != 0 && g >= NGRP) break;
                    const int tr = g / RG, row = (g % RG) * 4;
                    const int r = r0 + p * TRP + tr, i0 = m0 + row;
                    f32x4 cr = *reinterpret_cast<const f32x4 *>(st + tr * TP + row);
                    f32x4 ci = CPLX ? *reinterpret_cast<const f32x4 *>(st + (TRP + tr) * TP + row) : cr;
#pragma unroll
                    for (int q = 1; q < KS; ++q) {
                        cr += *reinterpret_cast<const f32x4 *>(st + (q * PL * TRP + tr) * TP + row);
                        if (CPLX) ci += *reinterpret_cast<const f32x4 *>(st + ((q * PL + 1) * TRP + tr) * TP + row);
                    }
                    if (F32 && !SIGN && a.sum_exp - amp_exp != 0) {
                        cr = ldexp4(cr, a.sum_exp - amp_exp);
                        if (CPLX) ci = ldexp4(ci, a.sum_exp - amp_exp);
                    }
                    const bool inside = i0 < a.Np && r < a.R;
                    if constexpr (MODE == MODE_ENERGY) {
                        // rows past the tile's end add nothing; the row groups of
                        // one trajectory are consecutive lanes
                        double e = inside ? energy_terms4<CPLX, SIGN>(a, i0, r, cr, ci) : 0.0;
#pragma unroll
                        for (int m = RG / 2; m >= 1; m >>= 1) e += __shfl_xor(e, m);
                        if (row == 0 && r < a.R) a.partial[(long long)mt * a.Rp + r] = e;
                    } else if (inside) {
                        if (epi_apply<MODE, CPLX, OPT, true>(a, i0, r, true, EARLY ? pre[u0 + v] : in[v], cr, ci))
                            a.flags[r] = 1;
                    }
                }
            }
        }
    };

    // Every group runs nit iterations, a multiple of JD; chunks past the last
    // load the last one and multiply nothing.  The last JD iterations issue no
    // loads, so the number of operations in flight is known at every wait.
    const int nk = a.Np / BK;
    const int nit = ((nk + KS - 1) / KS + JD - 1) / JD * JD;
    auto chunk_of = [&](int it) { return min(it * KS + grp, nk - 1); };
#pragma unroll
    for (int p = 0; p < JD; ++p) copy_chunk(chunk_of(p) * BK, p);
    __asm__ __volatile__("" ::: "memory");
#pragma unroll
    for (int p = 0; p < JD; ++p)
#pragma unroll
        for (int sl = J8 ? 1 : 0; sl < NSL; sl += J8 ? 2 : 1) load_j(chunk_of(p), p, sl);
    if constexpr (F32 && MODE != MODE_ENERGY) {
        // small amplitudes: the same products in the same order of 2^kAmpExp
        // times the amplitudes, straight from memory (looked at here, where the
        // flag's own load has had the time of the first chunks')
        if (tiny != 0) {
            for (int kc = grp; kc < nk; kc += KS)
#pragma unroll
                for (int sl = 0; sl < NSL; ++sl) {
                    const int k = kc * BK + (J8 ? (sl >> 1) * 32 + 16 * lh + 8 * (sl & 1) : 16 * sl + 8 * lh);
                    u32x4 x0[NB], x1[NB], x2[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        const int c = nb * 32 + l32, plane = CPLX ? c / TRW : 0;
                        const int tr = min(wn * TRW + c % TRW, a.Rp - 1 - r0);
                        const f32x4 *x = reinterpret_cast<const f32x4 *>(
                            static_cast<const float *>(a.B) + plane * a.plane_stride + (r0 + tr) * Np + k);
                        split8(x[0] * kAmpScale, x[1] * kAmpScale, x0[nb], x1[nb], x2[nb]);
                    }
                    products(sl, x0, x1, x2,
                             [&](int mb, int q) { return (jsrc[mb] + (long long)(kc * JPC + q) * 64)[lane]; });
                }
            __builtin_amdgcn_s_waitcnt(0);   // (the copies above, before others use their LDS)
            finish(kAmpExp);
            return;
        }
    }
    int buf = 0;
    // iteration `it` with the couplings of set JS; LAST: one of the last JD
    auto iteration = [&](int it, auto js, auto last) {
        constexpr int JS = decltype(js)::value;
        constexpr bool LAST = decltype(last)::value;
        // the amplitudes of chunk `it` have landed; issued since: the copies
        // of the chunks after it and the couplings from its own on
        constexpr int AHEAD = LAST ? JD - JS : JD;
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((AHEAD - 1) * NCW + AHEAD * NJ));
        __asm__ __volatile__("" ::: "memory");
        if constexpr (NWG > 1) {
            __builtin_amdgcn_s_barrier();
            __asm__ __volatile__("" ::: "memory");
        }
        // refill the buffer read in the previous iteration
        if constexpr (!LAST) copy_chunk(chunk_of(it + JD) * BK, buf == 0 ? JD : buf - 1);
        __asm__ __volatile__("" ::: "memory");
        if (!LAST || it * KS + grp < nk) {
            const unsigned char *Bt = gl + buf * TILEB;
            // raw amplitudes of one slice: this lane's eight are k = 32 m + 16 h
            // + 8 s on (FP8 couplings, slice s of block m) or 16 s + 8 h on
            constexpr int NQ = F32 ? 2 : 1;            // 16-byte words
            u32x4 xr[2][NB][NQ];
            auto lread = [&](int sl, int set) {
                const int slot = NQ * (J8 ? (sl >> 1) * 4 + 2 * lh + (sl & 1) : 2 * sl + lh);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int t = 0; t < NQ; ++t) {
                        const int row = wn * TN + nb * 32 + l32;
                        xr[set][nb][t] =
                            *reinterpret_cast<const u32x4 *>(Bt + row * RB + (((slot + t) ^ row_swz<RB>(row)) * 16));
                    }
            };
            lread(0, 0);
#pragma unroll
            for (int sl = 0; sl < NSL; ++sl) {
                const int set = sl & 1;
                if (sl + 1 < NSL) lread(sl + 1, set ^ 1);
                u32x4 x0[NB], x1[NB], x2[NB];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const f32x4 lo = __builtin_bit_cast(f32x4, xr[set][nb][0]);
                    const f32x4 hi = __builtin_bit_cast(f32x4, xr[set][nb][NQ - 1]);
                    if constexpr (!F32) x0[nb] = xr[set][nb][0];
                    else if constexpr (SIGN) x0[nb] = sign8(lo, hi);
                    else split8(lo, hi, x0[nb], x1[nb], x2[nb]);
                }
                products(sl, x0, x1, x2, [&](int mb, int q) { return jw[JS][mb][q]; });
                // the couplings just used make room for those JD chunks ahead
                if constexpr (!LAST)
                    if (!J8 || set == 1) load_j(chunk_of(it + JD), JS, sl);
            }
        }
        buf = buf == JD ? 0 : buf + 1;
    };
    int it = 0;
    for (; it + JD < nit; it += JD)
        seq_apply([&](auto p) { iteration(it + decltype(p)::value, p, std::false_type{}); },
                  std::make_integer_sequence<int, JD>{});
    seq_apply([&](auto p) { iteration(it + decltype(p)::value, p, std::true_type{}); },
              std::make_integer_sequence<int, JD>{});
    finish(0);
#endif
}

template <int BM, int BN, int BK, int WM, int WN, int KS, int JD, bool CPLX, int JK, int OPT = OP_F32>
hipError_t launch_modes(int mode, const DenseStepArgs &a, hipStream_t st) {
    constexpr int TRAJ = CPLX ? BN / 2 : BN;
    if (a.Np % BK || a.Np % 4 || a.R < 1 || a.R > a.Rp) return hipErrorInvalidValue;
    const dim3 grid(((a.Np + BM - 1) / BM) * ((a.R + TRAJ - 1) / TRAJ)), block(64 * WM * WN * KS);
#define GD_LAUNCH(M) dense_step_split<BM, BN, BK, WM, WN, KS, JD, CPLX, M, JK, OPT><<<grid, block, 0, st>>>(a)
    switch (mode) {
    case MODE_EULER: GD_LAUNCH(MODE_EULER); break;
    case MODE_RK1: GD_LAUNCH(MODE_RK1); break;
    case MODE_RK2: GD_LAUNCH(MODE_RK2); break;
    case MODE_RK3: GD_LAUNCH(MODE_RK3); break;
    case MODE_RK4: GD_LAUNCH(MODE_RK4); break;
    case MODE_ENERGY:
        // (energies of one plane on FP8 couplings come from the sign kernel, but
        // for the tiles that compete with the matrix-vector kernels)
        if constexpr (JK == J_FP8 && !CPLX && OPT == OP_F32 && !(BM == 32 && BN == 32)) return hipErrorInvalidValue;
        else GD_LAUNCH(MODE_ENERGY);
        break;
    default: return hipErrorInvalidValue;
    }
#undef GD_LAUNCH
    return hipGetLastError();
}

template <int BM, int BN, int BK, int WM, int WN, int KS, int JD, bool CPLX, int JK>
hipError_t launch_energy(const DenseStepArgs &a, hipStream_t st) {
    constexpr int TRAJ = CPLX ? BN / 2 : BN;
    if (a.Np % BK || a.Np % 4 || a.R < 1 || a.R > a.Rp) return hipErrorInvalidValue;
    const dim3 grid(((a.Np + BM - 1) / BM) * ((a.R + TRAJ - 1) / TRAJ));
    dense_step_split<BM, BN, BK, WM, WN, KS, JD, CPLX, MODE_ENERGY, JK><<<grid, 64 * WM * WN * KS, 0, st>>>(a);
    return hipGetLastError();
}

// Variants {BM, BN (GEMM columns), BK, WM, WN, KS (K groups), JD (chunks
// ahead)} with FP8 couplings and with split couplings; the runtime times them.
// 32-column tiles with K groups of one wave put enough workgroups on the chip
// for a few hundred trajectories; 64-row waves halve the splitting per product
// where the columns fill the chip; the 256-row tiles are for N = R = 4096.
#define GD_SPLIT_J8_VARIANTS(X)       \
    X(0, 32, 32, 32, 1, 1, 8, 4)      \
    X(1, 32, 32, 32, 1, 1, 4, 4)      \
    X(2, 64, 32, 32, 1, 1, 4, 4)      \
    X(3, 64, 64, 32, 1, 1, 4, 2)      \
    X(4, 64, 64, 32, 1, 1, 8, 1)      \
    X(5, 128, 64, 32, 2, 1, 4, 2)     \
    X(6, 128, 64, 32, 2, 2, 2, 2)     \
    X(7, 32, 32, 32, 1, 1, 4, 2)      \
    X(8, 128, 128, 32, 2, 2, 2, 2)    \
    X(9, 256, 256, 64, 2, 4, 1, 1)    \
    X(10, 256, 256, 32, 2, 4, 1, 2)   \
    X(11, 256, 256, 32, 2, 4, 1, 4)   \
    X(12, 256, 128, 64, 2, 4, 1, 1)   \
    X(13, 64, 32, 32, 1, 1, 8, 2)     \
    X(14, 128, 32, 32, 2, 1, 4, 2)    \
    X(15, 64, 64, 32, 1, 2, 4, 2)
#define GD_SPLIT_J3_VARIANTS(X)       \
    X(0, 32, 32, 32, 1, 1, 8, 2)      \
    X(1, 32, 32, 32, 1, 1, 4, 2)      \
    X(2, 64, 32, 32, 1, 1, 4, 2)      \
    X(3, 64, 64, 32, 1, 1, 4, 1)      \
    X(4, 64, 64, 32, 1, 1, 8, 1)      \
    X(5, 128, 64, 32, 2, 1, 4, 1)     \
    X(6, 128, 64, 32, 2, 2, 2, 2)     \
    X(7, 128, 128, 32, 2, 2, 1, 1)    \
    X(8, 128, 128, 32, 2, 2, 2, 1)    \
    X(9, 256, 128, 32, 4, 2, 1, 1)    \
    X(10, 32, 32, 32, 1, 1, 8, 1)     \
    X(11, 32, 32, 32, 1, 1, 4, 4)     \
    X(12, 128, 32, 32, 2, 1, 4, 2)    \
    X(13, 64, 128, 32, 1, 2, 4, 1)    \
    X(14, 64, 32, 32, 1, 1, 8, 1)     \
    X(15, 64, 64, 32, 1, 2, 4, 1)

// Tiles {BM, BN, BK, WM, WN, KS, JD} of the sign energies.  One product leaves
// a third of the matrix work of a step: N = R = 4096 is bound by the conversion
// and the LDS reads around it.
#define GD_SPLIT_SIGN_VARIANTS(X)     \
    X(0, 32, 32, 32, 1, 1, 4, 4)      \
    X(1, 64, 64, 32, 1, 1, 4, 2)      \
    X(2, 128, 128, 32, 2, 2, 2, 2)    \
    X(3, 256, 256, 32, 2, 4, 1, 2)

// Variants {BM, BN, BK, WM, WN, KS, JD} of the 16-bit operands: one product,
// no splitting, so larger waves; KS = 1 keeps the order of the sums that the
// direct-to-LDS kernels of gd_dense_lp.h have (the same bits), so small problems take small
// tiles instead.  Per step, BF16 (gd_dense_lp.h's best in brackets): N = 1000,
// R = 128 6.9 us (14.2), N = R = 1024 10.3 (15.0), N = 1500, R = 600 12.6
// (20.8), N = R = 2048 30.5 (36.7), N = R = 4096 126 (137).
#define GD_SPLIT_LP_VARIANTS(X)       \
    X(0, 256, 128, 64, 2, 2, 1, 2)    \
    X(1, 128, 128, 64, 2, 2, 1, 2)    \
    X(2, 128, 64, 64, 2, 2, 1, 2)     \
    X(3, 64, 64, 64, 1, 2, 1, 4)      \
    X(4, 32, 32, 64, 1, 1, 1, 4)

}  // namespace split

// launchers of the FP8-coupling and split-coupling instantiations, real and
// complex (one translation unit each)
hipError_t launch_split_j8_re(int idx, int mode, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_j8_cx(int idx, int mode, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_j3_re(int idx, int mode, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_sign(int idx, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_j3_cx(int idx, int mode, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_lp_re(int idx, int mode, int op, const DenseStepArgs &a, hipStream_t st);
hipError_t launch_split_lp_cx(int idx, int mode, int op, const DenseStepArgs &a, hipStream_t st);

}  // namespace gd

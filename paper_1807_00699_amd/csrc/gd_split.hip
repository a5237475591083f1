// Split-FP32 coupling kernels (gd_split.h): the host-side variant table.
#include "gd_split.h"

namespace gd {

namespace {
constexpr int kSplitCfg[2][16][7] = {
#define GD_ROW(id, bm, bn, bk, wm, wn, ks, jd) {bm, bn, bk, wm, wn, ks, jd},
    {GD_SPLIT_J3_VARIANTS(GD_ROW)},
    {GD_SPLIT_J8_VARIANTS(GD_ROW)},
#undef GD_ROW
};
constexpr int kSplitLpCfg[][7] = {
#define GD_ROW(id, bm, bn, bk, wm, wn, ks, jd) {bm, bn, bk, wm, wn, ks, jd},
    GD_SPLIT_LP_VARIANTS(GD_ROW)
#undef GD_ROW
};

DenseConfig config_of(const int *k, bool complex_mode, int id) {
    DenseConfig c{};
    c.id = id;
    c.bm = k[0];
    c.bn = k[1];
    c.bk = k[2];
    c.wn = k[4];
    c.traj_tile = complex_mode ? c.bn / 2 : c.bn;
    c.threads = 64 * k[3] * k[4] * k[5];
    return c;
}

// J in the lane order of the matrix instruction (gd_split.h): one thread per
// lane and 16-byte word
__global__ void tile_j8_k(const unsigned char *__restrict__ J, uint4 *__restrict__ out, int Np) {
    const long long words = (long long)Np * Np / 16;
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < words;
         t += (long long)gridDim.x * blockDim.x) {
        const int lane = int(t & 63);
        const long long blk = t >> 6;
        const long long row = blk / (Np / 32) * 32 + (lane & 31), k = blk % (Np / 32) * 32 + 16 * (lane >> 5);
        out[t] = *reinterpret_cast<const uint4 *>(J + row * Np + k);
    }
}

__global__ void tile_j3_k(const float *__restrict__ J, uint4 *__restrict__ out, int Np, int j_exp) {
    const long long words = (long long)Np * Np / 8;   // lanes; three words each
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < words;
         t += (long long)gridDim.x * blockDim.x) {
        const int lane = int(t & 63);
        const long long blk = t >> 6;
        const long long row = blk / (Np / 16) * 32 + (lane & 31), k = blk % (Np / 16) * 16 + 8 * (lane >> 5);
        const f32x4 *p = reinterpret_cast<const f32x4 *>(J + row * Np + k);
        split::u32x4 w[3];
        split::split8(split::ldexp4(p[0], -j_exp), split::ldexp4(p[1], -j_exp), w[0], w[1], w[2]);
        for (int q = 0; q < 3; ++q) out[(blk * 3 + q) * 64 + lane] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
    }
}

}  // namespace

hipError_t launch_tile_couplings(const float *J, const void *J8, void *out, int Np, int j_exp, hipStream_t st) {
    if (Np % 64) return hipErrorInvalidValue;
    const long long words = (long long)Np * Np / (J8 ? 16 : 8);
    const int grid = int(words / 256 < 65536 ? words / 256 : 65536);
    if (J8) tile_j8_k<<<grid, 256, 0, st>>>(static_cast<const unsigned char *>(J8), static_cast<uint4 *>(out), Np);
    else tile_j3_k<<<grid, 256, 0, st>>>(J, static_cast<uint4 *>(out), Np, j_exp);
    return hipGetLastError();
}

int split_config_count() { return int(sizeof(kSplitCfg[0]) / sizeof(kSplitCfg[0][0])); }

DenseConfig split_config(bool complex_mode, bool j_fp8, int idx) {
    return config_of(kSplitCfg[j_fp8][idx], complex_mode, idx);
}

hipError_t launch_split_step(const DenseConfig &cfg, bool complex_mode, int mode, bool j_fp8, const DenseStepArgs &a,
                             hipStream_t st) {
    const int idx = cfg.id >= kFewBase ? cfg.id - kFewBase : cfg.id;
    if (!a.J || idx < 0 || idx >= split_config_count()) return hipErrorInvalidValue;
    if (j_fp8) return complex_mode ? launch_split_j8_cx(idx, mode, a, st) : launch_split_j8_re(idx, mode, a, st);
    return complex_mode ? launch_split_j3_cx(idx, mode, a, st) : launch_split_j3_re(idx, mode, a, st);
}

int split_lp_config_count() { return int(sizeof(kSplitLpCfg) / sizeof(kSplitLpCfg[0])); }

DenseConfig split_lp_config(bool complex_mode, int idx) {
    return config_of(kSplitLpCfg[idx], complex_mode, kLpSplitBase + idx);
}

hipError_t launch_split_lp(int idx, bool complex_mode, int mode, int op, const DenseStepArgs &a, hipStream_t st) {
    if (!a.J || (op != OP_BF16 && op != OP_F16)) return hipErrorInvalidValue;
    return complex_mode ? launch_split_lp_cx(idx, mode, op, a, st) : launch_split_lp_re(idx, mode, op, a, st);
}

int sign_energy_row_tile(int Np, int R) {
    // the largest tile with a workgroup for every CU
    constexpr int kTile[3] = {256, 128, 64};
    for (const int t : kTile)
        if ((long long)((Np + t - 1) / t) * ((R + t - 1) / t) >= 256) return t;
    return 32;
}

hipError_t launch_sign_energy(const DenseStepArgs &a, hipStream_t st) {
    if (!a.J) return hipErrorInvalidValue;
    const int t = sign_energy_row_tile(a.Np, a.R);
    return launch_split_sign(t == 256 ? 3 : t == 128 ? 2 : t == 64 ? 1 : 0, a, st);
}

}  // namespace gd

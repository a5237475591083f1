// Internal interfaces between the host runtime and the gfx950 kernels of
// libgd.so.  Not part of the public ABI (include/gd.h).
#pragma once
#include <vector>
#include <hip/hip_runtime.h>
#include <cstdint>

namespace gd {

// Records `msg` as the calling thread's last error and returns `code`.
int gd_fail(int code, const char *msg);

// Epilogue of the dense coupling kernel.
enum StepMode : int {
    MODE_EULER = 0,   // psi_out = psi + dt f, gamma += dt phi
    MODE_RK1 = 1,     // k1; acc = k1; stage = y + dt/2 k1
    MODE_RK2 = 2,     // k2; acc += 2 k2; stage = y + dt/2 k2
    MODE_RK3 = 3,     // k3; acc += 2 k3; stage = y + dt k3
    MODE_RK4 = 4,     // k4; y += dt/6 (acc + k4)
    MODE_ENERGY = 5,  // per-trajectory partial sums of Eq. (h) over a row tile
};

// Operand precision of the coupling product.
enum OperandKind : int { OP_F32 = 0, OP_BF16 = 1, OP_F16 = 2 };

// Row tile of every dense kernel and the padding unit of n.
constexpr int kRowTile = 64;

// All pointers are device pointers.  Per-trajectory arrays are "planes" of
// [Rp][Np] floats (trajectory-major, spin contiguous, zero padded); complex
// amplitudes use two consecutive planes (re, im) of plane_stride floats.
struct DenseStepArgs {
    const void *J;         // couplings in the form the launched kernel reads
    const void *B;         // GEMM operand planes (FP32, or BF16/FP16 shadow)
    const float *psi_in;   // stage-input amplitudes at (r, i) (FP32 planes)
    float *psi_out;        // output amplitudes (next stage / next step)
    void *shadow_out;      // reduced-precision copy of psi_out for the next GEMM (or null)
    const float *gam_in;   // stage-input gains
    float *gam_out;        // output gains (may alias gam_in)
    const float *y_psi;    // RK4: amplitudes at the start of the step
    const float *y_gam;    // RK4: gains at the start of the step
    float *acc_psi;        // RK4: k1 + 2 k2 + 2 k3 accumulators
    float *acc_gam;
    const float *eps;      // [Np] per-spin gain rates
    const float *h1;       // [Np] q = 1 resonant term h_1i (zero padded)
    const float *g;        // [Np] external field g_i (energy mode)
    int *flags;            // [Rp] nonzero when trajectory r became non-finite
    double *partial;       // energy mode: [n_row_tiles][Rp]
    long long plane_stride;
    int Np, Rp, n, R;
    float inv_s, dt, gamma_c, rho_th;
    // resonant term h_q conj(Psi)^(q-1) of the complex models (q = 0: none)
    int q;
    float hq;
    // noise of the step's final stage: noise_amp = D sqrt(dt) (0: none),
    // noise_key = SplitMix64 key of this step
    float noise_amp;
    unsigned long long noise_key;
    // split kernels and persistent steps: J is split as J / 2^j_exp; 2^sum_exp
    // times the sums of the products of its pieces are those of J Psi, or (0,
    // modes that step; always for persistent steps) inv_s carries that factor
    int j_exp, sum_exp;
    int *tiny;             // FP32: set when an amplitude other than zero below 2^-100 is written
    // energy mode: weight of the second plane's product (3/4 for the q = 3, 6
    // clock states, whose second plane holds sin(theta) / (sqrt(3)/2))
    float im_weight;
};

// Kernel variants of the dense path.  traj_tile = trajectories per workgroup.
struct DenseConfig {
    int id;
    int bm;        // rows per workgroup (the energy partials use row tiles of bm)
    int bn;        // GEMM columns per workgroup
    int bk;        // K chunk per pipeline stage
    int wn;        // waves along the column dimension
    int traj_tile; // trajectories per workgroup
    int threads;
    int min_np = 0; // smallest padded size the variant runs
};

// FP32 steps on the BF16 matrix cores (gd_split.h): J in FP8 E4M3 (j_fp8) when
// every coupling is exact there, else in three BF16 pieces.  Every variant
// runs every size (row tiles past Np and trajectories past R are not written).
int split_config_count();
DenseConfig split_config(bool complex_mode, bool j_fp8, int idx);
// out: J in the order those kernels read it (Np^2 bytes from the row-major
// FP8 copy J8, or, J8 null, 6 Np^2 bytes from the FP32 J / 2^j_exp)
constexpr int kAmpExp = 24;   // small amplitudes are split as 2^kAmpExp Psi
hipError_t launch_tile_couplings(const float *J, const void *J8, void *out, int Np, int j_exp, hipStream_t st);
hipError_t launch_split_step(const DenseConfig &cfg, bool complex_mode, int mode, bool j_fp8,
                             const DenseStepArgs &a, hipStream_t st);

// Energies of the signs of the amplitudes psi_in = B (one plane), J in FP8 from
// launch_tile_couplings: partial[row tile][r], row tiles of
// sign_energy_row_tile.  The sums are exact when the couplings are integers
// and every row of |J| sums to less than 2^24.
int sign_energy_row_tile(int Np, int R);
hipError_t launch_sign_energy(const DenseStepArgs &a, hipStream_t st);

// Reduced-precision variants (gd_dense_lp.hip): BF16/FP16 operands, FP32
// accumulation; J either in the operand type or FP8 E4M3 (j_fp8).
int dense_lp_config_count();
DenseConfig dense_lp_config(bool complex_mode, int idx);
bool dense_lp_config_fits(const DenseConfig &c, int Np, int Rp);
hipError_t launch_dense_step_lp(const DenseConfig &cfg, bool complex_mode, int mode, int op,
                                bool j_fp8, const DenseStepArgs &a, hipStream_t st);

// What the host reads at the end of a run (out: pinned host memory)
struct RunResult {
    double best_e;   // running best of the checks and its trajectory
    int best_i;
    int diverged;    // trajectories r < R with flags[r] != 0
    long long stalled;   // *stalled, 0 without one
};
// The end of an energy check or of a run (gd_check.h)
struct CheckEnd {
    double *E = nullptr;        // energies of the check, or null
    int R = 0;
    int *best = nullptr;        // argmin and its energy
    double *best_e = nullptr;
    double *run_e = nullptr;    // running best of a run's checks; its first check takes (e0, i0) as the best so far
    int *run_i = nullptr;
    double e0 = 0.0;
    int i0 = 0;
    bool first = false;
    double *trace = nullptr;    // the check's entry of the energy trace
    const int *flags = nullptr;
    const long long *stalled = nullptr;   // PersistArgs::stalled: set, the check's energies are of no state and not taken
    RunResult *out = nullptr;   // end of a run: pinned host memory
    unsigned *count = nullptr;  // workgroups that have arrived, 0 between launches
};

// Persistent steps (gd_persist.hip): FP32, Np > 128; ids reported from
// kPersistBase on
constexpr int kPersistBase = 200;
struct PersistArgs {
    unsigned *x;              // exchange buffers (persist_words), empty before the first launch
    long long *stalled;       // 0; `tag` from the first launch on in which a workgroup waited longer than
                              // `patience`: it and later ones write no state that a later step reads
    long long tag;            // of this launch, not 0
    long long base;           // amplitudes published by earlier launches
    long long t0;             // index of the first step (noise)
    unsigned long long seed;  // noise seed
    long long patience;       // wall-clock ticks (100 MHz); < 0: every workgroup gives up at once
    int steps;
    int groups, pause;        // set by launch_persist
};
long long persist_words(int id, bool cplx, int Np, int R);
bool persist_ends_run(int id);
int persist_variant(bool cplx, bool rk4, bool j8, int Np, int R);
hipError_t launch_persist(int id, bool cplx, bool rk4, bool j8, const DenseStepArgs &a, const PersistArgs &p,
                          const CheckEnd &c, hipStream_t st);

// ---- small-R coupling product (gd_gemv.hip): a J-streaming matrix-vector
// kernel for at most kGemvMaxCols GEMM columns (R real or 2R complex), with
// the same modes and epilogue as the dense kernels.  Its variants carry ids
// kGemvBase + index next to the dense ones; bm = rows per workgroup (16 or
// 32, the row tile of its energy partials).
constexpr int kGemvBase = 100;
constexpr int kGemvMaxCols = 16;
// reduced-precision variants of gd_split.h (FP8-stored couplings): ids kLpSplitBase + index
constexpr int kLpSplitBase = 14;
int split_lp_config_count();
DenseConfig split_lp_config(bool complex_mode, int idx);
hipError_t launch_split_lp(int idx, bool complex_mode, int mode, int op, const DenseStepArgs &a, hipStream_t st);
// FP32 variants of gd_split.h with 32-column tiles competing there: ids kFewBase + index
constexpr int kFewBase = 110;
int gemv_config_count();
DenseConfig gemv_config(int idx);
// variant idx runs C = R (real) or 2R (complex) columns at Np spins with
// operand kind op and FP8-stored J
bool gemv_fits(int idx, int Np, int R, bool complex_mode, int op, bool j_fp8);
hipError_t launch_gemv_step(const DenseConfig &cfg, bool complex_mode, int mode, int op, bool j_fp8,
                            const DenseStepArgs &a, hipStream_t st);

// ---- GD-mod (gd_mod.hip): one Euler step with per-trajectory couplings K
// [R][Np][Np] (updated in place); c_hat = dt * eps_hat.  Needs Np % 16 == 0
// and gdmod_lds_bytes <= 64 KiB.
size_t gdmod_lds_bytes(bool complex_mode, int Np);
// packed K (one triangle, gdmod_packed_floats per trajectory) and the partial
// sums of its step
long long gdmod_packed_floats(int Np);
long long gdmod_part_floats(bool cplx, int Np, int R);
hipError_t launch_gdmod_pack(const float *J, float *K, int Np, int R, hipStream_t st);
hipError_t launch_gdmod_unpack(const float *K, float *out, int Np, int n, hipStream_t st);
hipError_t launch_gdmod_sym(bool complex_mode, const DenseStepArgs &a, const float *J, float *K, float *part, float c_hat,
                            hipStream_t st);
hipError_t launch_gdmod(bool complex_mode, const DenseStepArgs &a, const float *J, float *K, float c_hat,
                        hipStream_t st);

// ---- batched sparse solver (gd_batch.hip)
struct BatchArgs {
    const int *inst_n;            // [K] spins per instance
    const long long *inst_spin;   // [K] offset of the instance's spins in per-spin arrays
    const long long *inst_state;  // [K] offset of the instance's [R][n] state block
    const float *inst_inv_s;      // [K] 1 / coupling scale
    const int *ell_idx;           // [sum n][dmax] local neighbour indices (padding: 0)
    const float *ell_w;           // [sum n][dmax] couplings (padding: 0)
    // packed form (dmax <= 3, one coupling magnitude per instance, n_max < 2^16 - 1):
    // [sum n][2] words, word 0 = idx0 | idx1 << 16, word 1 = idx2 | neg2 << 29 |
    // neg1 << 30 | neg0 << 31 (neg: coupling -mag, else +mag); a missing
    // coupling has index n_k (the instance's size), an amplitude row that holds zeros
    const unsigned int *ell_pack;
    const float *inst_wmag;       // [K] the magnitude of instance k's couplings
    const int *inst_tlog;         // [K] per-instance-width variants: log2 of instance k's item width
    // per-instance-width variants: spins relabeled per instance for the LDS
    // gathers (label = LDS row and slot of a spin): label of spin i, spin of
    // label p (both [sum n], instance-local values), and the packed
    // neighbours in label order with labels as indices ([sum n][2] words)
    const int *tw_label, *tw_spin;
    const unsigned int *tw_pack;
    const float *eps, *h1, *g;    // [sum n]
    float *x, *gam;               // state [sum_k R n_k]
    double *E;                    // [K][R] energies after the launch
    int *flags;                   // [K][R] non-finite flags
    const int *wg_off;            // [nwg + 1] item ranges per workgroup
    const int *items;             // item = k * nslices + slice (per-instance widths: k * R + first trajectory)
    int nslices, R, dmax, nmax, steps;
    float dt, gamma_c, rho_th;
    float eps0;                   // the rate of every spin, for variants that need uniform eps and no field
};

struct BatchConfig {
    int id;
    int traj;     // trajectories per work item (0: chosen per instance, at most 64)
    int threads;  // workgroup size
    int slots;    // spins per thread (n_max <= slots * threads / traj)
    bool packed;  // neighbours in registers from the packed form (LDS: amplitudes only)
    bool uniform; // one eps for every spin and no field (eps0, h_1 = 0): no per-slot constants
    bool dbuf;    // amplitudes double-buffered in LDS (packed form): one barrier per step
};

int batch_config_count();
BatchConfig batch_config(int idx);
size_t batch_lds_bytes(const BatchConfig &c, int nmax, int dmax);
int batch_item_capacity(const BatchConfig &c);   // spin-trajectories of one item (slots x threads)
// resident workgroups per CU of a variant (registers, LDS and threads)
int batch_occupancy(const BatchConfig &c, int nmax, int dmax);

// ---- persistent tuner cache (gd_tune_cache.hip; GD_AUTOTUNE_CACHE=<file>)
// the variant id stored for (kind, key) by this or an earlier process on the
// same device and library build, or -1
int tune_cache_lookup(const char *kind, const std::vector<long long> &key);
void tune_cache_store(const char *kind, const std::vector<long long> &key, int id);
hipError_t prepare_batch(const BatchConfig &c, int nmax, int dmax);   // once per variant, outside capture
hipError_t launch_batch(const BatchConfig &c, int nwg, const BatchArgs &a, hipStream_t st);
// Per instance k < K: (best_E[k], best_r[k]) takes the lowest E[k * R + r]
// (ties -> lowest r) when it is strictly lower
hipError_t launch_batch_best(const double *E, int K, int R, double *best_E, int *best_r, hipStream_t st);

// ---- auxiliary kernels (gd_aux.hip)
// user [R][n] (or [R][n][2]) -> zero-padded planes [P][Rp][Np]; tiny (or null):
// as DenseStepArgs::tiny
hipError_t launch_pack_planes(const float *user, float *planes, int n, int R, int Np, int Rp,
                              int nplanes, int *tiny, hipStream_t st);
// psi (nplanes) and gains at once
hipError_t launch_unpack_state(const float *psi, float *upsi, const float *gam, float *ugam, int n, int R, int Np, int Rp,
                               int nplanes, hipStream_t st);
hipError_t launch_unpack_planes(const float *planes, float *user, int n, int R, int Np, int Rp,
                                int nplanes, hipStream_t st);
// Readout of the amplitudes onto the spin domain of Eq. (h).
enum Readout {
    RO_SIGN = 0,     // real Ising: d = sign(x), sign(+-0) = +1
    RO_PHASOR = 1,   // XY: d = Psi / |Psi| (Psi = 0 -> 1)
    RO_SIGN_RE = 2,  // complex Ising: d = sign(Re Psi)
    RO_CLOCK = 3     // q-state clock: k = floor(q arg(Psi) / 2pi + 1/2) mod q,
                     // d = (cos 2pi k/q, sin 2pi k/q), second plane scaled as
                     // clock_im_weight describes
};
// 3/4 for q = 3 and 6 (the second plane then holds sin / (sqrt(3)/2) in
// {0, +-1}, exact), 1 otherwise
float clock_im_weight(int q);
// Discretised state planes D (null to skip) and their operand copy, zero outside n x R.
// Optional outputs (null to skip): spins8 [R][n] int8, angle [R][n] float in
// [0, 2pi) of the discretised state, states [R][n] int32 (RO_CLOCK).
// flags[r] set on NaN.
hipError_t launch_discretise(const float *psi, float *D, void *shadowD, int op, int readout, int q,
                             int8_t *spins8, float *angle, int32_t *states, int *flags, int n, int R,
                             int Np, int Rp, int nplanes, long long plane_stride, hipStream_t st);
// c.E[r] = sum_t partial[t][r] (fixed order), then the end of the check
hipError_t launch_energy_reduce(const double *partial, int ntiles, int Rp, const CheckEnd &c, hipStream_t st);
// The end of a check or run alone
hipError_t launch_check_end(const CheckEnd &c, hipStream_t st);
// FP64 re-score from the FP32 amplitudes (unit phasors / signs formed in FP64):
// partial[t][r] = sum_{i in tile t} [-Re(conj(d_i) (J d)_i) + g_i Re(d_i)]
// D64: scratch for the FP64 readout planes, nplanes * Rp * Np doubles
hipError_t launch_energy_fp64(const float *J, const float *psi, const float *g, double *D64,
                              double *partial, int Np, int Rp, int n, int R, int nplanes,
                              long long plane_stride, int readout, int q, hipStream_t st);
// shadow copy of FP32 planes in BF16 / FP16
hipError_t launch_make_shadow(const float *src, void *dst, long long count, int op, hipStream_t st);
// J in the order the small-problem kernel reads it (Np 64 or 128; Np^2 floats)
hipError_t launch_small_couplings(const float *J, float *out, int Np, hipStream_t st);
// `steps` Euler or RK4 steps of a small problem (Np 64 or 128; FP32; a.J from
// launch_small_couplings) in one launch: psi_in/gam_in -> psi_out/gam_out (gam_out
// may alias gam_in), flags[r] set if trajectory r ends non-finite.  Noise
// (a.noise_amp != 0): step t0 + k uses the key SplitMix64(seed ^
// SplitMix64(t0 + k)), as the step-by-step path does.  With c.E: the Eq. (h)
// energies of the final state's readout (readout, q), and the end of the check.
hipError_t launch_small_steps(bool complex_mode, bool rk4, const DenseStepArgs &a, int steps,
                              unsigned long long seed, long long t0, int readout, int q, const CheckEnd &c,
                              hipStream_t st);

}  // namespace gd

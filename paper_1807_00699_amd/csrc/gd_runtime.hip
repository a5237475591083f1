// Host runtime and C ABI of libgd.so (declarations and contracts: include/gd.h).
//
// Ingest (once per instance): validate J (finite, exactly symmetric), zero
// the diagonal, compute the coupling scale s, map the external field g of
// Eq. (h) onto the q = 1 term h_1 = -g sqrt(rho_th)/s of Eq. (main), pad to
// the row tile and upload.  Run: one dense coupling launch per Euler step or
// per RK4 stage, with the amplitude/gain update fused in (gd_split.h, gd_gemv.h), or
// all steps in one launch (gd_small.hip, gd_persist.hip).
#include "gd_batch_rt.h"
#include "gd_internal.h"
#include "../../include/gd.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

using namespace gd;

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string &msg) {
    g_last_error = msg;
    // the runtime keeps an error for the next launch check, also of other solvers
    if (code == GD_E_OOM || code == GD_E_DEVICE) (void)hipGetLastError();
    return code;
}

#define GD_HIP(expr)                                                                        \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess) {                                                             \
            return fail(e_ == hipErrorOutOfMemory ? GD_E_OOM : GD_E_DEVICE,                 \
                        std::string(#expr) + ": " + hipGetErrorString(e_));                 \
        }                                                                                   \
    } while (0)

inline long long round_up(long long x, long long m) { return (x + m - 1) / m * m; }

constexpr int kTrajAlign = 128;  // Rp granularity: every dense variant tiles it
constexpr int kProfileEvery = 8;  // GD_F_PROFILE samples the launches of every 8th step
// Wall-clock ticks (2 s) that a workgroup of a persistent launch waits for the
// others: the exchange takes microseconds, but workgroups start when the
// kernels of other streams leave their CUs.  A run that waits longer goes on
// with one launch per step.
constexpr long long kPersistPatience = 200000000;
constexpr int kPersistCheckEvals = 4;   // coupling evaluations between two checks from which steps are persistent
constexpr int kTraceChecks = 1 << 16;  // device checks kept in the energy trace (512 KiB)

// SplitMix64 (Steele, Lea, Flood 2014) -> uniform double in [0, 1).
inline uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
inline double uniform01(uint64_t seed, uint64_t ctr) {
    return double(splitmix64(seed ^ splitmix64(ctr)) >> 11) * (1.0 / 9007199254740992.0);
}

// OCP FP8 E4M3 (4 exponent bits, bias 7, 3 mantissa bits; S.1111.111 is NaN,
// no infinities).  decode: value of a code; encode_exact: code whose value is
// exactly v (normal numbers and zero only), if any.
inline float e4m3_decode(uint8_t c) {
    const int s = c >> 7, e = (c >> 3) & 15, m = c & 7;
    float v;
    if (e == 15 && m == 7) return std::nanf("");
    if (e == 0) v = std::ldexp(float(m), -9);
    else v = std::ldexp(1.0f + float(m) / 8.0f, e - 7);
    return s ? -v : v;
}
inline bool e4m3_encode_exact(float v, uint8_t *out) {
    if (v == 0.0f) { *out = std::signbit(v) ? 0x80 : 0x00; return true; }
    if (!std::isfinite(v)) return false;
    // normal numbers only: |v| = (1 + m/8) 2^(e-7), 1 <= e <= 15, 0 <= m <= 7
    // (e = 15, m = 7 is NaN); frexp gives |v| = f 2^x with f in [0.5, 1)
    int x = 0;
    const double f = std::frexp(std::fabs(double(v)), &x);
    const int e = x + 6;
    const double m8 = (2.0 * f - 1.0) * 8.0;
    if (e < 1 || e > 15 || m8 != std::floor(m8)) return false;
    const int m = int(m8);
    if (e == 15 && m == 7) return false;
    const uint8_t c = uint8_t((std::signbit(v) ? 0x80 : 0x00) | (e << 3) | m);
    if (e4m3_decode(c) != v) return false;
    *out = c;
    return true;
}
inline bool bf16_exact(float v, uint16_t *out) {
    uint32_t b;
    std::memcpy(&b, &v, 4);
    if (b & 0xFFFFu) return false;
    *out = uint16_t(b >> 16);
    return true;
}
inline bool f16_exact(float v, uint16_t *out) {
    const _Float16 h = (_Float16)v;
    if (float(h) != v) return false;
    std::memcpy(out, &h, 2);
    return true;
}

// Staging memory of gd_spins_noalloc: one fixed array per device for callers
// that cannot allocate.  In host code `scratch` names a host-side stand-in,
// not device memory: the device address comes from hipGetSymbolAddress, once
// per device with that device current, and only that address is used.
constexpr long long kModPacked = 25000000;   // GD-mod: R Np^2 from which one triangle of each K is kept (gd_mod.hip)
constexpr size_t kScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mu;
std::map<int, void *> g_scratch_addr;   // device -> address of its scratch

// Device address of `scratch` on device `dev` (looked up on first use).
int scratch_address(int dev, void **out) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch_addr.find(dev);
    if (it != g_scratch_addr.end()) {
        *out = it->second;
        return GD_OK;
    }
    int cur = 0;
    GD_HIP(hipGetDevice(&cur));
    if (cur != dev) GD_HIP(hipSetDevice(dev));
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) GD_HIP(hipSetDevice(cur));
    if (e != hipSuccess || !ptr)
        return fail(GD_E_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_addr[dev] = ptr;
    *out = ptr;
    return GD_OK;
}

std::mutex g_tune_mu;
// (complex + 2 precision + 8 FP8-stored J + 32 FP8 copy of FP32 J, Np, Rp,
// integrator, R if the matrix-vector kernels compete else 0) -> kernel variant
// id; with GD_AUTOTUNE_CACHE also kept in that file across processes
std::map<std::tuple<int, int, int, int, int>, int> g_tune_cache;

}  // namespace

int gd::gd_fail(int code, const char *msg) { return fail(code, msg ? msg : ""); }

namespace gd {
BatchSolver *solver_batch(gd_solver *s);
}

struct gd_solver {
    gd::BatchSolver *batch = nullptr;   // non-null: a batch of instances (gd_create_batch)
    bool track_target = false;          // gd_set_targets was called: record time-to-target
    int n = 0, Np = 0, model = 0, P = 1;
    int ro = RO_SIGN;          // readout of the model
    int q_res = 0;             // order of the resonant term (0: none)
    double hq = 0.0;           // its strength h_q
    gd_params prm{};
    double s = 1.0;
    bool j_integer = false, g_integer = true;
    int j_exp = 0;             // largest |J_ij| in [2^(j_exp - 1), 2^j_exp)
    bool j_sums24 = false;     // if J is integer and exact in FP8: every row of |J| sums to less than 2^24
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int device = 0;
    std::vector<float> hJ;     // padded host copy (for re-validation and tests)
    std::vector<float> hEps;   // per-spin eps actually in use (length n)
    // device constants
    float *dJ = nullptr, *dEps = nullptr, *dH1 = nullptr, *dG = nullptr;
    int op = OP_F32;           // operand precision of the coupling GEMM
    bool jfp8 = false;         // J stored as FP8 E4M3 (reduced-precision modes)
    void *dJlp = nullptr;      // J in FP8 or in the operand type
    // FP32 solvers whose couplings are all exact in FP8 E4M3 (e.g. {-1, 0, +1}): a
    // one-byte copy of J, widened exactly where it is read; GD_J8_COPY=0 keeps
    // FP32 J only
    void *dJ8 = nullptr;
    void *dJt = nullptr;       // J (FP8, or three BF16 pieces) as the split kernels read it
    float *dJs = nullptr;      // FP32 solvers with Np <= 128: J as the fused small-problem kernel reads it
    void *shadow[3] = {nullptr, nullptr, nullptr};   // operand copies of psi[k]
    // persistent steps: variant (-1: one launch per step), exchange buffers
    // and how many amplitude sets went through them; launches left before one
    // launch per step (< 0: no limit), and the wait that ends a launch
    int persist = -1;
    unsigned *xchg = nullptr;
    long long *stalled = nullptr;
    int64_t persist_left = -1, patience = 0;
    unsigned *arrivals = nullptr;   // of the last-workgroup ends of checks and runs
    long long xbase = 0;
    void *shadowD = nullptr;   // operand copy of the discretised state
    // state
    int R = 0, Rp = 0;
    bool have_state = false;
    DenseConfig cfg{};
    float *psi[3] = {nullptr, nullptr, nullptr};
    float *gam = nullptr, *gam_s = nullptr, *acc_psi = nullptr, *acc_gam = nullptr;
    float *D = nullptr;
    float *K = nullptr;        // GD-mod couplings [R][Np][Np], or one triangle of each (K_packed)
    bool K_packed = false;
    float *Kpart = nullptr;    // K_packed: partial coupling sums of a step
    double *D64 = nullptr;     // FP64 readout planes of the re-score (allocated on first use)
    double *partial = nullptr, *dE = nullptr;
    int *flags = nullptr, *dBest = nullptr;
    int *tiny = nullptr;       // DenseStepArgs::tiny of the current state
    // minimum energy of each device check since gd_set_init / gd_set_state
    // (the first kTraceChecks checks) and the step of each
    double *dTrace = nullptr;
    std::vector<int64_t> trace_steps;
    int cur = 0;
    // stats
    int64_t steps_done = 0, spin_updates = 0, launches_timed = 0;
    double run_seconds = 0.0, kernel_ms = 0.0;
    int diverged = 0, target_reached = 0, best_index = -1;
    double ttt_seconds = 0.0, best_energy = HUGE_VAL;
    int64_t ttt_steps = 0;
    std::vector<hipEvent_t> events;
    // time-to-target recording without a stop: each check's (E[best], best)
    // lands in pinned host slots behind an event, read one check later
    struct CheckSlot {
        double e;
        int i;
    };
    CheckSlot *hchk = nullptr;            // 2 slots (hipHostMalloc)
    gd::RunResult *hres = nullptr;        // results of a run (hipHostMalloc at the first)
    hipEvent_t ev_chk[2] = {nullptr, nullptr};
    hipEvent_t ev_run0 = nullptr;         // start of the current gd_run
    hipEvent_t ev_end = nullptr;          // end of the current gd_run
    // device time of the gd_run calls since gd_set_init / gd_set_state
    // (start to end event of each), the clock of the time to target
    double clock_s = 0.0;
    int64_t ev_used = 0;       // event pairs recorded by the current gd_run call
    int64_t ev_launches = 0;   // coupling launches bracketed by those pairs
    // small problems: kGraphSteps steps captured once in a hipGraph (launch
    // overhead dominates there); valid for the buffers of the current state
    // and the amplitude buffer index it was captured from
    hipGraphExec_t step_graph = nullptr;
    int step_graph_cur = -1;

    long long plane() const { return (long long)Rp * Np; }
    bool mod() const { return prm.variant == GD_VARIANT_MOD; }
    bool complex_mode() const { return P == 2; }
    int integrator() const { return prm.integrator; }
};

namespace {

void free_state(gd_solver *s) {
    if (s->step_graph) (void)hipGraphExecDestroy(s->step_graph);
    s->step_graph = nullptr;
    s->step_graph_cur = -1;
    if (s->psi[1] == s->psi[0]) s->psi[1] = nullptr;
    for (float *&p : s->psi) { if (p) (void)hipFree(p); p = nullptr; }
    float **fl[] = {&s->gam, &s->gam_s, &s->acc_psi, &s->acc_gam, &s->D, &s->K, &s->Kpart};
    for (float **p : fl) { if (*p) (void)hipFree(*p); *p = nullptr; }
    for (void *&p : s->shadow) { if (p) (void)hipFree(p); p = nullptr; }
    if (s->shadowD) (void)hipFree(s->shadowD);
    s->shadowD = nullptr;
    if (s->D64) (void)hipFree(s->D64);
    s->D64 = nullptr;
    if (s->xchg) (void)hipFree(s->xchg);
    if (s->stalled) (void)hipFree(s->stalled);
    if (s->arrivals) (void)hipFree(s->arrivals);
    s->arrivals = nullptr;
    s->xchg = nullptr;
    s->stalled = nullptr;
    s->persist = -1;
    if (s->partial) (void)hipFree(s->partial);
    if (s->dE) (void)hipFree(s->dE);
    if (s->flags) (void)hipFree(s->flags);
    if (s->tiny) (void)hipFree(s->tiny);
    s->tiny = nullptr;
    if (s->dBest) (void)hipFree(s->dBest);
    if (s->dTrace) (void)hipFree(s->dTrace);
    s->dTrace = nullptr;
    s->partial = s->dE = nullptr;
    s->flags = s->dBest = nullptr;
    s->have_state = false;
    s->R = s->Rp = 0;
}

void reset_stats(gd_solver *s) {
    s->steps_done = s->spin_updates = s->launches_timed = 0;
    s->run_seconds = s->kernel_ms = 0.0;
    s->diverged = s->target_reached = 0;
    s->best_index = -1;
    s->ttt_seconds = 0.0;
    s->ttt_steps = 0;
    s->best_energy = HUGE_VAL;
    s->clock_s = 0.0;
    s->trace_steps.clear();
}

template <class T>
int dalloc(T **p, size_t count) {
    *p = nullptr;
    if (count == 0) count = 1;
    hipError_t e = hipMalloc(reinterpret_cast<void **>(p), count * sizeof(T));
    if (e != hipSuccess) {
        *p = nullptr;
        return fail(e == hipErrorOutOfMemory ? GD_E_OOM : GD_E_DEVICE,
                    std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    return GD_OK;
}

int alloc_state(gd_solver *s, int R) {
    free_state(s);
    s->R = R;
    s->Rp = (int)round_up(R, kTrajAlign);
    const size_t pl = (size_t)s->plane();
    const size_t P = (size_t)s->P;
    int rc = GD_OK;
    const int npsi = s->integrator() == GD_RK4 ? 3 : 2;
    // Euler steps at reduced precision multiply the operand copy, so they
    // update the FP32 amplitudes in place (psi[1] is psi[0]); the copies
    // alternate.  At N = R = 4096 that leaves 218 MB touched per step, within
    // the 256 MiB of the last-level cache: 126 us per step (two planes: 17 us more
    // with the kernel of that time)
    const bool in_place = s->op != OP_F32 && s->integrator() == GD_EULER;
    for (int k = 0; k < npsi && rc == GD_OK; ++k) {
        if (in_place && k == 1) s->psi[1] = s->psi[0];
        else rc = dalloc(&s->psi[k], pl * P);
    }
    if (rc == GD_OK) rc = dalloc(&s->gam, pl);
    if (rc == GD_OK && s->integrator() == GD_RK4) {
        rc = dalloc(&s->gam_s, pl);
        if (rc == GD_OK) rc = dalloc(&s->acc_psi, pl * P);
        if (rc == GD_OK) rc = dalloc(&s->acc_gam, pl);
    }
    if (rc == GD_OK && s->mod()) {
        rc = dalloc(&s->gam_s, pl);   // gains ping-pong: every row block reads all gains
        s->K_packed = (long long)R * s->Np * s->Np >= kModPacked;
        if (rc == GD_OK) rc = dalloc(&s->K, (size_t)R * (s->K_packed ? gdmod_packed_floats(s->Np) : (long long)s->Np * s->Np));
        if (rc == GD_OK && s->K_packed) rc = dalloc(&s->Kpart, (size_t)gdmod_part_floats(s->complex_mode(), s->Np, R));
    }
    if (rc == GD_OK) rc = dalloc(&s->D, pl * P);
    if (s->op != OP_F32) {
        for (int k = 0; k < npsi && rc == GD_OK; ++k)
            rc = dalloc(reinterpret_cast<uint16_t **>(&s->shadow[k]), pl * P);
        if (rc == GD_OK) rc = dalloc(reinterpret_cast<uint16_t **>(&s->shadowD), pl * P);
    }
    if (rc == GD_OK) rc = dalloc(&s->partial, (size_t)(s->Np / 16) * s->Rp);  // smallest row tile
    // + E[best] of the last check, + running best of a run's checks
    if (rc == GD_OK) rc = dalloc(&s->dE, (size_t)s->Rp + 2);
    if (rc == GD_OK) rc = dalloc(&s->flags, (size_t)s->Rp);
    if (rc == GD_OK) rc = dalloc(&s->tiny, 1);
    if (rc == GD_OK) rc = dalloc(&s->arrivals, 1);
    if (rc == GD_OK) rc = dalloc(&s->dBest, 2);   // best of the last check, running best
    if (rc == GD_OK) rc = dalloc(&s->dTrace, (size_t)kTraceChecks);
    if (rc != GD_OK) {
        free_state(s);
        return rc;
    }
    for (int k = 0; k < 3; ++k) {
        if (s->psi[k]) GD_HIP(hipMemsetAsync(s->psi[k], 0, pl * P * sizeof(float), s->stream));
        if (s->shadow[k]) GD_HIP(hipMemsetAsync(s->shadow[k], 0, pl * P * sizeof(uint16_t), s->stream));
    }
    GD_HIP(hipMemsetAsync(s->flags, 0, (size_t)s->Rp * sizeof(int), s->stream));
    GD_HIP(hipMemsetAsync(s->tiny, 0, sizeof(int), s->stream));
    GD_HIP(hipMemsetAsync(s->arrivals, 0, sizeof(unsigned), s->stream));
    if (s->gam_s) GD_HIP(hipMemsetAsync(s->gam_s, 0, pl * sizeof(float), s->stream));
    s->cur = 0;
    s->have_state = true;
    return GD_OK;
}

// GD-mod: K_ij(0) = J_ij for every trajectory
int reset_mod_couplings(gd_solver *s) {
    if (!s->mod() || !s->K) return GD_OK;
    if (s->K_packed) {
        GD_HIP(launch_gdmod_pack(s->dJ, s->K, s->Np, s->R, s->stream));
        return GD_OK;
    }
    const size_t m = (size_t)s->Np * s->Np;
    for (int r = 0; r < s->R; ++r)
        GD_HIP(hipMemcpyAsync(s->K + (size_t)r * m, s->dJ, m * sizeof(float), hipMemcpyDeviceToDevice,
                              s->stream));
    return GD_OK;
}

DenseStepArgs base_args(gd_solver *s) {
    DenseStepArgs a{};
    a.J = s->dJ;
    a.eps = s->dEps;
    a.h1 = s->dH1;
    a.g = s->dG;
    a.flags = s->flags;
    a.partial = s->partial;
    a.plane_stride = s->plane();
    a.Np = s->Np;
    a.Rp = s->Rp;
    a.n = s->n;
    a.R = s->R;
    a.inv_s = float(1.0 / s->s);
    a.dt = float(s->prm.dt);
    a.gamma_c = float(s->prm.gamma_c);
    a.rho_th = float(s->prm.rho_th);
    a.q = s->q_res;
    a.hq = float(s->hq);
    a.noise_amp = 0.0f;
    a.noise_key = 0;
    a.tiny = s->tiny;
    a.im_weight = s->ro == RO_CLOCK ? clock_im_weight(s->prm.q) : 1.0f;
    return a;
}

// The powers of two of the split operands (gd_split.h): folded into 1/s for the
// modes that step, unless it leaves the normal numbers (couplings and a scale s
// of the caller's in very different units)
// (`amp_exp`: amplitudes are split as 2^amp_exp Psi)
void set_scales(const gd_solver *s, int mode, int amp_exp, DenseStepArgs &a) {
    a.j_exp = s->dJ8 ? 0 : s->j_exp;
    a.sum_exp = a.j_exp - amp_exp;
    const float both = float(std::ldexp(1.0 / s->s, a.sum_exp));
    if (mode == MODE_ENERGY || !std::isnormal(both) || !std::isnormal(a.inv_s)) return;
    a.inv_s = both;
    a.sum_exp = 0;
}

hipError_t launch_coupling(gd_solver *s, const DenseConfig &cfg, int mode, const DenseStepArgs &a) {
    DenseStepArgs b = a;
    if (s->op != OP_F32) b.J = s->dJlp;
    if (cfg.id >= kGemvBase && cfg.id < kFewBase) {
        if (s->op == OP_F32 && s->dJ8) b.J = s->dJ8;
        return launch_gemv_step(cfg, s->complex_mode(), mode, s->op, s->jfp8 || s->dJ8 != nullptr, b, s->stream);
    }
    if (s->op == OP_F32) {
        b.J = s->dJt;
        set_scales(s, mode, 0, b);
        return launch_split_step(cfg, s->complex_mode(), mode, s->dJ8 != nullptr, b, s->stream);
    }
    if (cfg.id >= kLpSplitBase) {
        b.J = s->dJt;
        return launch_split_lp(cfg.id - kLpSplitBase, s->complex_mode(), mode, s->op, b, s->stream);
    }
    return launch_dense_step_lp(cfg, s->complex_mode(), mode, s->op, s->jfp8, b, s->stream);
}

// refresh the operand copy of psi[k] after the FP32 state was written by the host
hipError_t refresh_shadow(gd_solver *s, int k) {
    if (s->op == OP_F32) return hipSuccess;
    return launch_make_shadow(s->psi[k], s->shadow[k], s->plane() * s->P, s->op, s->stream);
}

// HIP event pair around work on the solver's stream (GD_F_PROFILE)
int ev_begin(gd_solver *s) {
    const size_t k = (size_t)s->ev_used * 2;
    while (s->events.size() < k + 2) {
        hipEvent_t e;
        GD_HIP(hipEventCreate(&e));
        s->events.push_back(e);
    }
    GD_HIP(hipEventRecord(s->events[k], s->stream));
    return GD_OK;
}

int ev_end(gd_solver *s, int launches) {
    GD_HIP(hipEventRecord(s->events[(size_t)s->ev_used * 2 + 1], s->stream));
    s->ev_used++;
    s->ev_launches += launches;
    return GD_OK;
}

// Enqueue integration step number t.  `dt_override` >= 0 replaces dt (used
// with 0 by the tuner: the state is then left bit-for-bit unchanged, noise
// included, since its amplitude is D sqrt(dt)).
int enqueue_step(gd_solver *s, const DenseConfig &cfg, float dt_override, bool timed, int64_t t) {
    int rc;
    DenseStepArgs a = base_args(s);
    if (dt_override >= 0.0f) a.dt = dt_override;
    if (s->prm.noise_D != 0.0) {
        a.noise_amp = float(s->prm.noise_D * std::sqrt(double(a.dt)));
        a.noise_key = splitmix64(s->prm.noise_seed ^ splitmix64((uint64_t)t));
    }
    if (s->mod()) {
        // GD-mod: HBM-bound batched product with per-trajectory couplings
        a.psi_in = s->psi[s->cur];
        a.psi_out = s->psi[s->cur ^ 1];
        a.gam_in = s->gam;
        a.gam_out = s->gam_s;
        if (timed && (rc = ev_begin(s)) != GD_OK) return rc;
        const float c_hat = float(double(a.dt) * s->prm.eps_hat);
        if (s->K_packed) GD_HIP(launch_gdmod_sym(s->complex_mode(), a, s->dJ, s->K, s->Kpart, c_hat, s->stream));
        else GD_HIP(launch_gdmod(s->complex_mode(), a, s->dJ, s->K, c_hat, s->stream));
        if (timed && (rc = ev_end(s, 1)) != GD_OK) return rc;
        std::swap(s->gam, s->gam_s);
        s->cur ^= 1;
        return GD_OK;
    }
    auto launch = [&](int mode, const DenseStepArgs &x) -> int {
        GD_HIP(launch_coupling(s, cfg, mode, x));
        return GD_OK;
    };
    const bool lp = s->op != OP_F32;
    // GD_F_PROFILE: one event pair around all coupling launches of the step
    if (timed && (rc = ev_begin(s)) != GD_OK) return rc;
    if (s->integrator() == GD_EULER) {
        a.B = lp ? s->shadow[s->cur] : (const void *)s->psi[s->cur];
        a.shadow_out = s->shadow[s->cur ^ 1];
        a.psi_in = s->psi[s->cur];
        a.psi_out = s->psi[s->cur ^ 1];
        a.gam_in = s->gam;
        a.gam_out = s->gam;
        if ((rc = launch(MODE_EULER, a)) != GD_OK) return rc;
        if (timed && (rc = ev_end(s, 1)) != GD_OK) return rc;
        s->cur ^= 1;
        return GD_OK;
    }
    const int iY = s->cur, iA = s->cur ^ 1, iB = 2;
    float *Y = s->psi[iY], *Sa = s->psi[iA], *Sb = s->psi[iB];
    auto op_of = [&](int k) -> const void * { return lp ? s->shadow[k] : (const void *)s->psi[k]; };
    a.y_psi = Y;
    a.y_gam = s->gam;
    a.acc_psi = s->acc_psi;
    a.acc_gam = s->acc_gam;
    // stage 1: input y
    a.B = op_of(iY); a.psi_in = Y; a.gam_in = s->gam; a.psi_out = Sa; a.gam_out = s->gam_s;
    a.shadow_out = s->shadow[iA];
    if ((rc = launch(MODE_RK1, a)) != GD_OK) return rc;
    a.B = op_of(iA); a.psi_in = Sa; a.gam_in = s->gam_s; a.psi_out = Sb; a.gam_out = s->gam_s;
    a.shadow_out = s->shadow[iB];
    if ((rc = launch(MODE_RK2, a)) != GD_OK) return rc;
    a.B = op_of(iB); a.psi_in = Sb; a.gam_in = s->gam_s; a.psi_out = Sa; a.gam_out = s->gam_s;
    a.shadow_out = s->shadow[iA];
    if ((rc = launch(MODE_RK3, a)) != GD_OK) return rc;
    a.B = op_of(iA); a.psi_in = Sa; a.gam_in = s->gam_s; a.psi_out = Y; a.gam_out = s->gam;
    a.shadow_out = s->shadow[iY];
    if ((rc = launch(MODE_RK4, a)) != GD_OK) return rc;
    if (timed && (rc = ev_end(s, 4)) != GD_OK) return rc;
    return GD_OK;
}

// J in FP8, row-major, if this solver stores it so
const void *couplings_fp8(const gd_solver *s) { return s->op == OP_F32 ? s->dJ8 : (s->jfp8 ? s->dJlp : nullptr); }

// J in the order the split kernels read it, laid out once per solver (at
// reduced precision FP8-stored couplings only)
int tile_couplings(gd_solver *s) {
    const void *j8 = couplings_fp8(s);
    if (s->dJt || (s->op != OP_F32 && !j8)) return GD_OK;
    const size_t m = (size_t)s->Np * s->Np;
    void *t = nullptr;
    const int rc = dalloc(reinterpret_cast<uint8_t **>(&t), j8 ? m : 6 * m);
    if (rc != GD_OK) return rc;
    const hipError_t e = launch_tile_couplings(s->dJ, j8, t, s->Np, s->j_exp, s->stream);
    if (e != hipSuccess) (void)hipFree(t);
    GD_HIP(e);
    s->dJt = t;
    return GD_OK;
}

// Whether the solver's steps read that form
bool steps_read_tiles(const gd_solver *s) {
    if (s->mod() || s->persist >= 0) return false;
    if (s->op != OP_F32) return s->cfg.id >= kLpSplitBase && s->cfg.id < kGemvBase;
    return (s->Np > 128 || std::getenv("GD_DENSE_CONFIG")) && (s->cfg.id < kGemvBase || s->cfg.id >= kFewBase);
}

// Ising readouts with FP8-stored couplings: energies from the signs of the
// amplitudes in one kernel, without readout planes
bool sign_readout(const gd_solver *s) {
    return (s->ro == RO_SIGN || s->ro == RO_SIGN_RE) && couplings_fp8(s) != nullptr;
}

// Partial energies of the current state into s->partial, `ntiles` row tiles:
// the device check path
int device_energies(gd_solver *s, int *ntiles) {
    // (the matrix-vector kernels read J row-major)
    const int rc = s->cfg.id < kGemvBase || s->cfg.id >= kFewBase ? tile_couplings(s) : GD_OK;
    if (rc != GD_OK) return rc;
    DenseStepArgs a = base_args(s);
    if (s->op == OP_F32 && s->cfg.id < kGemvBase && sign_readout(s)) {
        a.J = s->dJt;
        a.B = a.psi_in = s->psi[s->cur];
        GD_HIP(launch_sign_energy(a, s->stream));
        const int bm = sign_energy_row_tile(s->Np, s->R);
        *ntiles = (s->Np + bm - 1) / bm;
        return GD_OK;
    }
    GD_HIP(launch_discretise(s->psi[s->cur], s->D, s->shadowD, s->op, s->ro, s->prm.q, nullptr, nullptr, nullptr,
                             s->flags, s->n, s->R, s->Np, s->Rp, s->P, s->plane(), s->stream));
    a.B = s->op == OP_F32 ? (const void *)s->D : s->shadowD;
    a.psi_in = s->D;
    GD_HIP(launch_coupling(s, s->cfg, MODE_ENERGY, a));
    *ntiles = (s->Np + s->cfg.bm - 1) / s->cfg.bm;
    return GD_OK;
}

// Whether runs of this solver are persistent steps, and their buffers
int choose_persist(gd_solver *s) {
    const bool cx = s->complex_mode();
    s->persist = -1;
    // (asynchronous runs return before anyone looks whether the launch stalled)
    if (s->op != OP_F32 || s->mod() || s->Np <= 128 || (s->prm.flags & GD_F_ASYNC) || std::getenv("GD_DENSE_CONFIG"))
        return GD_OK;
    const char *launches = std::getenv("GD_PERSIST"), *wait = std::getenv("GD_PERSIST_WAIT");
    s->persist_left = launches ? std::atoll(launches) : -1;
    s->patience = wait ? 100 * std::atoll(wait) - 1 : kPersistPatience;
    if (s->persist_left == 0) return GD_OK;
    // A cooperative launch between two checks costs about 20 us more than a
    // step's launch.  us per check interval of 1, 2, 5, 10 steps, one launch per
    // step and persistent: N = 1000, R = 1 17, 23, 35, 59 and 35, 37, 43, 52; N
    // = 300, R = 64 15, 21, 37, 65 and 34, 36, 42, 51; N = 800, R = 100 17, 25,
    // 45, 77 and 39, 42, 52, 68; XY RK4 N = 1000, R = 128, 1 and 2 steps, 52, 83
    // and 66, 83.  The lines are at 1 to 2 RK4 and 6 to 8 Euler steps; below 4
    // evaluations persistent steps lose by half.
    if (s->persist_left < 0 && s->prm.check_interval > 0 &&
        (long long)s->prm.check_interval * (s->integrator() == GD_RK4 ? 4 : 1) < kPersistCheckEvals)
        return GD_OK;
    DenseStepArgs a = base_args(s);
    set_scales(s, MODE_EULER, kAmpExp, a);
    if (a.sum_exp != 0) return GD_OK;
    const int id = persist_variant(cx, s->integrator() == GD_RK4, s->dJ8 != nullptr, s->Np, s->R);
    if (id < 0) return GD_OK;
    if (!s->xchg) {
        const long long words = persist_words(id, cx, s->Np, s->R);
        int rc = dalloc(&s->xchg, (size_t)words);
        if (rc == GD_OK) rc = dalloc(&s->stalled, 1);
        // (a launch keeps the state it starts from: gains in two buffers)
        if (rc == GD_OK && !s->gam_s) {
            rc = dalloc(&s->gam_s, (size_t)s->plane());
            if (rc == GD_OK) GD_HIP(hipMemsetAsync(s->gam_s, 0, (size_t)s->plane() * sizeof(float), s->stream));
        }
        if (rc != GD_OK) return rc;
        GD_HIP(hipMemsetAsync(s->xchg, 0xFF, (size_t)words * 4, s->stream));
        GD_HIP(hipMemsetAsync(s->stalled, 0, sizeof(long long), s->stream));
        s->xbase = 0;
    }
    s->persist = id;
    return GD_OK;
}

// Pick the coupling kernel variant: GD_DENSE_CONFIG forces one; otherwise each
// variant that fits (the GEMM tiles, and for at most kGemvMaxCols GEMM columns
// also the J-streaming matrix-vector kernels, ids kGemvBase + k) is timed on
// the live buffers with dt = 0 (state unchanged) and the fastest is cached per
// (model, precision, J storage, Np, Rp, integrator, R when the matrix-vector
// kernels compete).
int choose_config(gd_solver *s) {
    const bool cx = s->complex_mode();
    const bool lp = s->op != OP_F32;
    const int nc = lp ? kLpSplitBase + (s->jfp8 ? split_lp_config_count() : 0) : split_config_count();
    auto gemv_ok = [&](int k) {
        return !s->mod() && gemv_fits(k, s->Np, s->R, cx, s->op, s->jfp8 || s->dJ8 != nullptr);
    };
    const bool gv = gemv_ok(0);
    const int ng = gv ? gemv_config_count() : 0;
    auto cfg_of = [&](int id) {
        if (id >= kFewBase) {
            DenseConfig c = split_config(cx, s->dJ8 != nullptr, id - kFewBase);
            c.id = id;
            return c;
        }
        if (id >= kGemvBase) return gemv_config(id - kGemvBase);
        if (lp && id >= kLpSplitBase) return split_lp_config(cx, id - kLpSplitBase);
        return lp ? dense_lp_config(cx, id) : split_config(cx, s->dJ8 != nullptr, id);
    };
    // a launch holds fewer than 2^32 threads (32 x 32 tiles of 512: n R < 8.6e9)
    auto grid_fits = [&](const DenseConfig &c) {
        const long long nwg = (long long)((s->Np + c.bm - 1) / c.bm) * ((s->R + c.traj_tile - 1) / c.traj_tile);
        return nwg * c.threads < 1ll << 32;
    };
    auto fits = [&](int id) {
        if (id >= kFewBase) {
            // 32 x 32 tiles; with split couplings the eight-group ones only,
            // whose sums are as close to 64 bits as the matrix-vector ones
            // (N = 4096: 1.15e-7 against 1.33e-7 of the sum; four groups 1.39e-7)
            if (!gv || lp || id >= kFewBase + nc) return false;
            const DenseConfig c = cfg_of(id);
            return c.bm == 32 && c.bn == 32 && (s->dJ8 || c.threads == 512);
        }
        if (id >= kGemvBase) return gemv_ok(id - kGemvBase);
        if (id < 0 || id >= nc) return false;
        return lp && id < kLpSplitBase ? dense_lp_config_fits(cfg_of(id), s->Np, s->Rp) : grid_fits(cfg_of(id));
    };
    // the fused kernel needs its own form of J; the coupling kernels' form is
    // laid out when they first run (here, when they are timed)
    const bool fused = !lp && !s->mod() && s->Np <= 128;
    if (fused && !s->dJs) {
        float *t = nullptr;
        const int rc = dalloc(&t, (size_t)s->Np * s->Np);
        if (rc != GD_OK) return rc;
        const hipError_t e = launch_small_couplings(s->dJ, t, s->Np, s->stream);
        if (e != hipSuccess) (void)hipFree(t);
        GD_HIP(e);
        s->dJs = t;
    }
    if (const char *env = std::getenv("GD_DENSE_CONFIG")) {
        int id = std::atoi(env);
        if (!fits(id))
            return fail(GD_E_INVALID_ARG, "GD_DENSE_CONFIG out of range or does not tile the problem");
        s->cfg = cfg_of(id);
        return GD_OK;
    }
    // Few columns: the matrix-vector kernels against (FP32) the 32 x 32 tiles
    // of the coupling kernels.  Per step at N = 4096, FP8-stored couplings:
    // R = 4 9.8 us against 13.4, R = 5 15.0 against 13.4, R = 16 25.7 against
    // 13.9; split couplings: R = 4 17.2 against 20.5, R = 16 28.2 against 20.6.
    // At reduced precision, against every tile.
    std::vector<int> ids;
    for (int id = 0; id < nc; ++id)
        if (fits(gv && !lp ? kFewBase + id : id)) ids.push_back(gv && !lp ? kFewBase + id : id);
    for (int k = 0; k < ng; ++k)
        if (gemv_ok(k)) ids.push_back(kGemvBase + k);
    auto key = std::make_tuple(int(cx) + 2 * s->op + 8 * int(s->jfp8) + 32 * int(s->dJ8 != nullptr), s->Np,
                               s->Rp, s->integrator(), gv ? s->R : 0);
    const std::vector<long long> fkey{std::get<0>(key), std::get<1>(key), std::get<2>(key), std::get<3>(key),
                                      std::get<4>(key)};
    {
        // the cache file first (GD_AUTOTUNE_CACHE), then this process's table
        const int fid = tune_cache_lookup("dense", fkey);
        if (fid >= 0 && fits(fid)) {
            std::lock_guard<std::mutex> lk(g_tune_mu);
            g_tune_cache[key] = fid;
            s->cfg = cfg_of(fid);
            return GD_OK;
        }
    }
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end() && fits(it->second)) {
            s->cfg = cfg_of(it->second);
            return GD_OK;
        }
    }
    // tiny problems: no point timing.
    // GD-mod steps do not use the variants (only its energy checks do).
    const long long work = (long long)s->Np * s->Np * s->Rp * s->P;
    int best = -1;
    if (work >= (1ll << 26) && !s->mod()) {
        const int rt = tile_couplings(s);
        if (rt != GD_OK) return rt;
        hipEvent_t e0, e1;
        GD_HIP(hipEventCreate(&e0));
        GD_HIP(hipEventCreate(&e1));
        float best_ms = 1e30f;
        std::vector<float> ms_of(ids.size(), 1e30f);
        for (size_t v = 0; v < ids.size(); ++v) {
            DenseConfig c = cfg_of(ids[v]);
            int rc = enqueue_step(s, c, 0.0f, false, 0);  // warm-up
            if (rc != GD_OK) return rc;
            // one step, then at least three and 0.1 ms of them (short kernels
            // hide behind their launches otherwise) unless that one is far
            // from the best
            int reps = 1;
            for (int pass = 0; pass < 2; ++pass) {
                GD_HIP(hipEventRecord(e0, s->stream));
                for (int k = 0; k < reps; ++k)
                    if ((rc = enqueue_step(s, c, 0.0f, false, 0)) != GD_OK) return rc;
                GD_HIP(hipEventRecord(e1, s->stream));
                GD_HIP(hipEventSynchronize(e1));
                float ms = 0.0f;
                GD_HIP(hipEventElapsedTime(&ms, e0, e1));
                ms_of[v] = ms / reps;
                if (ms_of[v] > 1.5f * best_ms) break;
                reps = std::max(3, std::min(16, int(0.1f / ms_of[v])));
            }
            best_ms = std::min(best_ms, ms_of[v]);
        }
        // near-ties (within 1%, below the timing noise) go to the first
        // candidate, so repeated tunings of one problem settle on the same variant
        for (size_t v = 0; v < ids.size() && best < 0; ++v)
            if (ms_of[v] <= 1.01f * best_ms) best = ids[v];
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        GD_HIP(hipMemsetAsync(s->flags, 0, (size_t)s->Rp * sizeof(int), s->stream));
    } else if (gv) {
        // small problems with few trajectories: the matrix-vector kernel reads
        // J once instead of multiplying Rp padded columns
        best = kGemvBase;
    } else if (!lp) {
        // small tiles and four K groups: the most workgroups without idle
        // groups (Ising N = 300, R = 64: 5.8 us per step; eight groups 6.4,
        // 64 x 64 tiles 7.4-7.7)
        best = 1;
    } else {
        long long most = -1;
        for (int id : ids) {
            DenseConfig c = cfg_of(id);
            const long long nblk = (long long)(s->Np / c.bm) * (s->Rp / c.traj_tile) * (c.threads / 64);
            if (nblk > most) { most = nblk; best = id; }
        }
    }
    if (best < 0) return fail(GD_E_UNSUPPORTED, "no dense kernel variant tiles this problem");
    s->cfg = cfg_of(best);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache[key] = best;
    tune_cache_store("dense", fkey, best);
    return GD_OK;
}

// What the steps of a state just set up need: the kernel variant, persistent
// steps' buffers, J as the kernels read it (gd_run allocates nothing for its
// steps, so that asynchronous runs can be captured from the first on).  Without
// it there is no state.
int prepare_steps(gd_solver *s) {
    int rc = choose_config(s);
    if (rc == GD_OK) rc = choose_persist(s);
    if (rc == GD_OK && steps_read_tiles(s)) rc = tile_couplings(s);
    // the three pieces of J (6 N^2 bytes) were laid out to time the variants only
    if (rc == GD_OK && s->dJt && !couplings_fp8(s) && !s->mod() && s->cfg.id >= kGemvBase && s->cfg.id < kFewBase) {
        const hipError_t e = hipFree(s->dJt);   // (waits for the device)
        s->dJt = nullptr;
        if (e != hipSuccess) rc = fail(GD_E_DEVICE, std::string("hipFree: ") + hipGetErrorString(e));
    }
    if (rc != GD_OK) free_state(s);
    return rc;
}

int check_params(const gd_params *p) {
    if (p->struct_size != sizeof(gd_params)) return fail(GD_E_INVALID_ARG, "gd_params.struct_size mismatch");
    if (p->integrator != GD_EULER && p->integrator != GD_RK4) return fail(GD_E_INVALID_ARG, "unknown integrator");
    if (p->precision < GD_PREC_FP32 || p->precision > GD_PREC_FP16) return fail(GD_E_INVALID_ARG, "unknown precision");
    if (!(std::isfinite(p->dt) && p->dt > 0)) return fail(GD_E_INVALID_ARG, "dt must be finite and > 0");
    if (!std::isfinite(p->eps) || !std::isfinite(p->rho_th) || !std::isfinite(p->gamma_c) ||
        !std::isfinite(p->gamma0) || !std::isfinite(p->init_amp))
        return fail(GD_E_INVALID_ARG, "non-finite parameter");
    if (!(std::isfinite(p->j_scale) && p->j_scale >= 0)) return fail(GD_E_INVALID_ARG, "j_scale must be >= 0");
    if (p->check_interval < 0) return fail(GD_E_INVALID_ARG, "check_interval must be >= 0");
    if (!(std::isfinite(p->noise_D) && p->noise_D >= 0)) return fail(GD_E_INVALID_ARG, "noise_D must be >= 0");
    if (!(std::isfinite(p->h_q) && p->h_q >= 0)) return fail(GD_E_INVALID_ARG, "h_q must be >= 0");
    if (p->variant != GD_VARIANT_GD && p->variant != GD_VARIANT_MOD)
        return fail(GD_E_INVALID_ARG, "unknown variant");
    if (!(std::isfinite(p->eps_hat) && p->eps_hat >= 0)) return fail(GD_E_INVALID_ARG, "eps_hat must be >= 0");
    return GD_OK;
}

int copy_in(const gd_solver *s, const float *src, size_t count, std::vector<float> &dst) {
    dst.resize(count);
    if (count == 0) return GD_OK;
    if (s->prm.flags & GD_F_DEVICE_PTRS) {
        GD_HIP(hipMemcpy(dst.data(), src, count * sizeof(float), hipMemcpyDeviceToHost));
    } else {
        std::memcpy(dst.data(), src, count * sizeof(float));
    }
    return GD_OK;
}

bool all_finite(const std::vector<float> &v) {
    for (float x : v)
        if (!std::isfinite(x)) return false;
    return true;
}

// user [R][n](x P) host/device -> device planes
int upload_planes(gd_solver *s, const float *user, float *planes, int R) {
    const size_t cnt = (size_t)R * s->n * s->P;
    float *tmp = nullptr;
    int rc = dalloc(&tmp, cnt);
    if (rc != GD_OK) return rc;
    hipError_t e;
    if (s->prm.flags & GD_F_DEVICE_PTRS)
        e = hipMemcpyAsync(tmp, user, cnt * sizeof(float), hipMemcpyDeviceToDevice, s->stream);
    else
        e = hipMemcpyAsync(tmp, user, cnt * sizeof(float), hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess)
        e = launch_pack_planes(tmp, planes, s->n, R, s->Np, s->Rp, s->P, planes == s->psi[0] ? s->tiny : nullptr, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    (void)hipFree(tmp);
    if (e != hipSuccess) return fail(GD_E_DEVICE, std::string("upload: ") + hipGetErrorString(e));
    return GD_OK;
}

// Whether a kernel may write `bytes` at a caller's device pointer itself: on
// this solver's device and inside its allocation (anything else goes through a
// staging buffer and hipMemcpy, which refuses what is not valid).
bool device_span(const gd_solver *s, const void *p, size_t bytes) {
    hipPointerAttribute_t at{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&at, p) != hipSuccess || at.type != hipMemoryTypeDevice || at.device != s->device ||
        hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const uintptr_t b = reinterpret_cast<uintptr_t>(base), q = reinterpret_cast<uintptr_t>(p);
    return q >= b && q - b <= size && bytes <= size - (q - b);
}

// Planes into the caller's [R][n] (or [R][n][2]) array, on the solver's stream:
// straight into device memory, else through D (the readout planes' scratch,
// rewritten before every use).
int download_planes(gd_solver *s, const float *planes, float *user, int P) {
    const size_t bytes = (size_t)s->R * s->n * P * sizeof(float);
    const bool dev = (s->prm.flags & GD_F_DEVICE_PTRS) != 0;
    if (dev && reinterpret_cast<uintptr_t>(user) % 4 == 0 && device_span(s, user, bytes)) {
        GD_HIP(launch_unpack_planes(planes, user, s->n, s->R, s->Np, s->Rp, P, s->stream));
        return GD_OK;
    }
    GD_HIP(launch_unpack_planes(planes, s->D, s->n, s->R, s->Np, s->Rp, P, s->stream));
    GD_HIP(hipMemcpyAsync(user, s->D, bytes, dev ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, s->stream));
    return GD_OK;
}

int set_eps(gd_solver *s, const float *eps) {
    std::vector<float> pad((size_t)s->Np, 0.0f);
    if (eps) {
        std::vector<float> e;
        int rc = copy_in(s, eps, (size_t)s->n, e);
        if (rc != GD_OK) return rc;
        if (!all_finite(e)) return fail(GD_E_NONFINITE, "eps has non-finite entries");
        s->hEps = e;
    } else {
        s->hEps.assign((size_t)s->n, float(s->prm.eps));
    }
    std::copy(s->hEps.begin(), s->hEps.end(), pad.begin());
    GD_HIP(hipMemcpy(s->dEps, pad.data(), pad.size() * sizeof(float), hipMemcpyHostToDevice));
    return GD_OK;
}

int default_init(gd_solver *s, int R, const float *gamma0) {
    const int n = s->n, P = s->P;
    std::vector<float> h((size_t)R * n * P);
    const double amp = s->prm.init_amp;
    for (int r = 0; r < R; ++r)
        for (int i = 0; i < n; ++i) {
            const uint64_t ctr = (uint64_t)r * (uint64_t)n + (uint64_t)i;
            const double u = uniform01(s->prm.seed, ctr);
            if (P == 1) {
                h[(size_t)r * n + i] = float(amp * (2.0 * u - 1.0));
            } else {
                const double phi = 2.0 * M_PI * u;
                h[((size_t)r * n + i) * 2] = float(amp * std::cos(phi));
                h[((size_t)r * n + i) * 2 + 1] = float(amp * std::sin(phi));
            }
        }
    const uint32_t saved = s->prm.flags;
    s->prm.flags &= ~GD_F_DEVICE_PTRS;  // h is host memory
    int rc = upload_planes(s, h.data(), s->psi[0], R);
    const int savedP = s->P;
    s->P = 1;
    if (rc == GD_OK && !gamma0) {
        std::vector<float> g((size_t)R * n, float(s->prm.gamma0));
        rc = upload_planes(s, g.data(), s->gam, R);
    }
    s->prm.flags = saved;
    if (rc == GD_OK && gamma0) rc = upload_planes(s, gamma0, s->gam, R);
    s->P = savedP;
    return rc;
}

// The state of gd_set_init
int fill_state(gd_solver *s, int32_t batch, const float *psi0, const float *gamma0) {
    int rc;
    if (psi0) {
        if ((rc = upload_planes(s, psi0, s->psi[0], batch)) != GD_OK) return rc;
        const int savedP = s->P;
        s->P = 1;
        if (gamma0) {
            rc = upload_planes(s, gamma0, s->gam, batch);
        } else {
            std::vector<float> g((size_t)batch * s->n, float(s->prm.gamma0));
            const uint32_t saved = s->prm.flags;
            s->prm.flags &= ~GD_F_DEVICE_PTRS;
            rc = upload_planes(s, g.data(), s->gam, batch);
            s->prm.flags = saved;
        }
        s->P = savedP;
        if (rc != GD_OK) return rc;
    } else {
        if ((rc = default_init(s, batch, gamma0)) != GD_OK) return rc;
    }
    GD_HIP(refresh_shadow(s, 0));
    if ((rc = reset_mod_couplings(s)) != GD_OK) return rc;
    return GD_OK;
}

}  // namespace

gd::BatchSolver *gd::solver_batch(gd_solver *s) { return s ? s->batch : nullptr; }

extern "C" {

void gd_default_params(gd_params *p) {
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->struct_size = sizeof(gd_params);
    p->integrator = GD_EULER;
    p->precision = GD_PREC_FP32;
    p->flags = 0;
    p->dt = 0.05;
    p->eps = 0.1;
    p->rho_th = 1.0;
    p->gamma_c = 0.0;
    p->gamma0 = 0.0;
    p->j_scale = 0.0;
    p->init_amp = 0.1;
    p->seed = 0;
    p->check_interval = 0;
    p->has_target = 0;
    p->target_energy = 0.0;
    p->stream = nullptr;
    p->noise_D = 0.0;
    p->noise_seed = 0;
    p->q = 2;
    p->variant = GD_VARIANT_GD;
    p->h_q = 0.0;
    p->eps_hat = 0.1;
}

const char *gd_error_string(int code) {
    switch (code) {
    case GD_OK: return "ok";
    case GD_E_INVALID_ARG: return "invalid argument";
    case GD_E_NOT_SYMMETRIC: return "J is not symmetric";
    case GD_E_NONFINITE: return "non-finite input";
    case GD_E_OOM: return "out of device memory";
    case GD_E_DEVICE: return "device (HIP) error";
    case GD_E_STATE: return "call out of order";
    case GD_E_DIVERGED: return "a trajectory diverged";
    case GD_E_UNSUPPORTED: return "unsupported";
    default: return "unknown error";
    }
}

const char *gd_last_error(void) { return g_last_error.c_str(); }

int gd_create(gd_solver **out, int32_t n, const float *J, const float *g, int32_t model,
              const gd_params *p) {
    if (!out) return fail(GD_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > 65536) return fail(GD_E_INVALID_ARG, "n out of range [1, 65536]");
    if (!J) return fail(GD_E_INVALID_ARG, "J is NULL");
    if (model < GD_ISING || model > GD_POTTS) return fail(GD_E_INVALID_ARG, "unknown model");
    gd_params prm;
    if (p) prm = *p;
    else gd_default_params(&prm);
    int rc = check_params(&prm);
    if (rc != GD_OK) return rc;
    if (model == GD_POTTS && (prm.q < 2 || prm.q > 8))
        return fail(GD_E_INVALID_ARG, "GD_POTTS needs 2 <= q <= 8");
    if (model == GD_POTTS && prm.q > 2 && !(prm.h_q > 0))
        return fail(GD_E_INVALID_ARG, "GD_POTTS with q > 2 needs h_q > 0");
    if (prm.variant == GD_VARIANT_MOD &&
        (prm.integrator != GD_EULER || prm.precision != GD_PREC_FP32 || n > 4096))
        return fail(GD_E_UNSUPPORTED, "GD-mod runs Euler steps in FP32 with n <= 4096");

    gd_solver *s = new (std::nothrow) gd_solver();
    if (!s) return fail(GD_E_OOM, "host allocation failed");
    s->n = n;
    s->model = model;
    s->P = model == GD_ISING ? 1 : 2;
    s->ro = model == GD_ISING ? RO_SIGN : model == GD_XY ? RO_PHASOR
          : model == GD_ISING_COMPLEX ? RO_SIGN_RE : RO_CLOCK;
    s->q_res = model == GD_ISING_COMPLEX ? 2 : model == GD_POTTS ? prm.q : 0;
    if (model == GD_ISING_COMPLEX) prm.q = 2;
    s->prm = prm;
    s->Np = (int)round_up(n, kRowTile);
    auto bail = [&](int code) {
        gd_destroy(s);
        return code;
    };

    std::vector<float> hj, hg;
    if ((rc = copy_in(s, J, (size_t)n * n, hj)) != GD_OK) return bail(rc);
    if (!all_finite(hj)) return bail(fail(GD_E_NONFINITE, "J has non-finite entries"));
    if (g) {
        if ((rc = copy_in(s, g, (size_t)n, hg)) != GD_OK) return bail(rc);
        if (!all_finite(hg)) return bail(fail(GD_E_NONFINITE, "g has non-finite entries"));
    }
    double ss = 0.0;
    float jmax = 0.0f;
    bool integer = true;
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) {
            if (i == j) continue;
            const float v = hj[(size_t)i * n + j];
            if (v != hj[(size_t)j * n + i]) {
                char buf[96];
                std::snprintf(buf, sizeof buf, "J[%d][%d] != J[%d][%d]", i, j, j, i);
                return bail(fail(GD_E_NOT_SYMMETRIC, buf));
            }
            ss += double(v) * double(v);
            jmax = std::max(jmax, std::fabs(v));
            integer = integer && (v == std::nearbyint(v));
        }
    s->j_integer = integer;
    if (jmax > 0.0f) (void)std::frexp(jmax, &s->j_exp);
    // (FP8 couplings are at most 448 in magnitude)
    s->j_sums24 = integer;
    for (int i = 0; i < n && s->j_sums24 && n > 16777216 / 448; ++i) {
        double row = 0.0;
        for (int j = 0; j < n; ++j)
            if (j != i) row += std::fabs(double(hj[(size_t)i * n + j]));
        s->j_sums24 = row < 16777216.0;
    }
    for (float v : hg) s->g_integer = s->g_integer && (v == std::nearbyint(v));
    s->s = prm.j_scale > 0 ? prm.j_scale : std::sqrt(ss / n);
    if (!(s->s > 0)) s->s = 1.0;
    if (s->q_res) {
        // default h_2: 10% above max_i sum_{j != i} |J_ij| / s
        double rowmax = 0.0;
        for (int i = 0; i < n; ++i) {
            double a = 0.0;
            for (int j = 0; j < n; ++j)
                if (j != i) a += std::fabs(double(hj[(size_t)i * n + j]));
            rowmax = std::max(rowmax, a);
        }
        s->hq = prm.h_q > 0 ? prm.h_q : 1.1 * rowmax / s->s;
    }

    if (hipGetDevice(&s->device) != hipSuccess) return bail(fail(GD_E_DEVICE, "no HIP device"));
    const int Np = s->Np;
    s->hJ.assign((size_t)Np * Np, 0.0f);
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j)
            if (i != j) s->hJ[(size_t)i * Np + j] = hj[(size_t)i * n + j];
    std::vector<float> h1((size_t)Np, 0.0f), gp((size_t)Np, 0.0f);
    const double k1 = -std::sqrt(prm.rho_th) / s->s;
    for (int i = 0; i < (int)hg.size(); ++i) {
        h1[i] = float(k1 * hg[i]);
        gp[i] = hg[i];
    }

    if (prm.stream) {
        s->stream = static_cast<hipStream_t>(prm.stream);
    } else {
        if (hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking) != hipSuccess)
            return bail(fail(GD_E_DEVICE, "hipStreamCreate failed"));
        s->own_stream = true;
    }
    // reduced precision: J must be exact in FP8 E4M3 (stored as one byte) or
    // in the operand type itself
    std::vector<uint8_t> j8;
    std::vector<uint16_t> j16;
    if (prm.precision != GD_PREC_FP32) {
        s->op = prm.precision == GD_PREC_BF16 ? OP_BF16 : OP_F16;
        bool fp8 = true;
        j8.assign((size_t)Np * Np, 0);
        for (int i = 0; i < n && fp8; ++i)
            for (int j = 0; j < n && fp8; ++j)
                if (i != j) fp8 = e4m3_encode_exact(hj[(size_t)i * n + j], &j8[(size_t)i * Np + j]);
        s->jfp8 = fp8;
        if (!fp8) {
            j8.clear();
            j16.assign((size_t)Np * Np, 0);
            bool ok = true;
            for (int i = 0; i < n && ok; ++i)
                for (int j = 0; j < n && ok; ++j)
                    if (i != j) {
                        const float v = hj[(size_t)i * n + j];
                        uint16_t *o = &j16[(size_t)i * Np + j];
                        ok = s->op == OP_BF16 ? bf16_exact(v, o) : f16_exact(v, o);
                    }
            if (!ok)
                return bail(fail(GD_E_UNSUPPORTED, "J is not exactly representable in the requested "
                                                   "operand precision (nor in FP8)"));
        }
    }
    const char *j8env = std::getenv("GD_J8_COPY");
    if (prm.precision == GD_PREC_FP32 && prm.variant != GD_VARIANT_MOD && !(j8env && std::atoi(j8env) == 0)) {
        bool fp8 = true;
        j8.assign((size_t)Np * Np, 0);
        for (int i = 0; i < n && fp8; ++i)
            for (int j = 0; j < n && fp8; ++j)
                if (i != j) fp8 = e4m3_encode_exact(hj[(size_t)i * n + j], &j8[(size_t)i * Np + j]);
        if (fp8) {
            if ((rc = dalloc(reinterpret_cast<uint8_t **>(&s->dJ8), j8.size())) != GD_OK) return bail(rc);
            if (hipMemcpy(s->dJ8, j8.data(), j8.size(), hipMemcpyHostToDevice) != hipSuccess)
                return bail(fail(GD_E_DEVICE, "upload of FP8 J failed"));
        }
        j8.clear();
    }
    if ((rc = dalloc(&s->dJ, (size_t)Np * Np)) != GD_OK) return bail(rc);
    if (s->jfp8) {
        if ((rc = dalloc(reinterpret_cast<uint8_t **>(&s->dJlp), j8.size())) != GD_OK) return bail(rc);
        if (hipMemcpy(s->dJlp, j8.data(), j8.size(), hipMemcpyHostToDevice) != hipSuccess)
            return bail(fail(GD_E_DEVICE, "upload of FP8 J failed"));
    } else if (!j16.empty()) {
        if ((rc = dalloc(reinterpret_cast<uint16_t **>(&s->dJlp), j16.size())) != GD_OK) return bail(rc);
        if (hipMemcpy(s->dJlp, j16.data(), j16.size() * 2, hipMemcpyHostToDevice) != hipSuccess)
            return bail(fail(GD_E_DEVICE, "upload of 16-bit J failed"));
    }
    if ((rc = dalloc(&s->dEps, (size_t)Np)) != GD_OK) return bail(rc);
    if ((rc = dalloc(&s->dH1, (size_t)Np)) != GD_OK) return bail(rc);
    if ((rc = dalloc(&s->dG, (size_t)Np)) != GD_OK) return bail(rc);
    if (hipMemcpy(s->dJ, s->hJ.data(), s->hJ.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->dH1, h1.data(), h1.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->dG, gp.data(), gp.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        return bail(fail(GD_E_DEVICE, "upload of J failed"));
    if ((rc = set_eps(s, nullptr)) != GD_OK) return bail(rc);
    *out = s;
    return GD_OK;
}

void gd_destroy(gd_solver *s) {
    if (!s) return;
    if (s->batch) {
        batch_destroy(s->batch);
        delete s;
        return;
    }
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    free_state(s);
    if (s->dJ) (void)hipFree(s->dJ);
    if (s->dEps) (void)hipFree(s->dEps);
    if (s->dH1) (void)hipFree(s->dH1);
    if (s->dG) (void)hipFree(s->dG);
    if (s->dJlp) (void)hipFree(s->dJlp);
    if (s->dJ8) (void)hipFree(s->dJ8);
    if (s->dJt) (void)hipFree(s->dJt);
    if (s->dJs) (void)hipFree(s->dJs);
    for (hipEvent_t e : s->events) (void)hipEventDestroy(e);
    for (hipEvent_t e : {s->ev_chk[0], s->ev_chk[1], s->ev_run0, s->ev_end})
        if (e) (void)hipEventDestroy(e);
    if (s->hchk) (void)hipHostFree(s->hchk);
    if (s->hres) (void)hipHostFree(s->hres);
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
}

int gd_set_init(gd_solver *s, int32_t batch, const float *psi0, const float *gamma0,
                const float *eps) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_set_init(s->batch, batch, psi0, gamma0, eps);
    if (batch < 1 || batch > (1 << 22)) return fail(GD_E_INVALID_ARG, "batch out of range");
    int rc;
    if ((rc = set_eps(s, eps)) != GD_OK) return rc;
    if (psi0 || gamma0) {
        std::vector<float> chk;
        if (psi0) {
            if ((rc = copy_in(s, psi0, (size_t)batch * s->n * s->P, chk)) != GD_OK) return rc;
            if (!all_finite(chk)) return fail(GD_E_NONFINITE, "psi0 has non-finite entries");
        }
        if (gamma0) {
            if ((rc = copy_in(s, gamma0, (size_t)batch * s->n, chk)) != GD_OK) return rc;
            if (!all_finite(chk)) return fail(GD_E_NONFINITE, "gamma0 has non-finite entries");
        }
    }
    if ((rc = alloc_state(s, batch)) != GD_OK) return rc;
    reset_stats(s);
    rc = fill_state(s, batch, psi0, gamma0);
    if (rc != GD_OK) {
        free_state(s);
        return rc;
    }
    return prepare_steps(s);
}

// Replay the captured kGraphSteps steps (capturing them first if the
// amplitude buffer index differs from the capture's).  kGraphSteps is even,
// so the Euler buffer ping-pong ends where it started.
constexpr int kGraphSteps = 32;
constexpr int kSmallStepsPerLaunch = 4096;
constexpr int kPersistSteps = 4096;
constexpr long long kGraphWork = 1ll << 28;   // Np^2 Rp P below which steps are replayed
static_assert(kGraphSteps % 2 == 0, "Euler ping-pong parity");

static int launch_step_graph(gd_solver *s) {
    if (!s->step_graph || s->step_graph_cur != s->cur) {
        if (s->step_graph) (void)hipGraphExecDestroy(s->step_graph);
        s->step_graph = nullptr;
        const int cur0 = s->cur;
        hipGraph_t g = nullptr;
        GD_HIP(hipStreamBeginCapture(s->stream, hipStreamCaptureModeThreadLocal));
        int rc = GD_OK;
        for (int q = 0; q < kGraphSteps && rc == GD_OK; ++q) rc = enqueue_step(s, s->cfg, -1.0f, false, 0);
        const hipError_t ce = hipStreamEndCapture(s->stream, &g);
        if (rc != GD_OK || ce != hipSuccess) {
            if (g) (void)hipGraphDestroy(g);
            s->cur = cur0;
            return rc != GD_OK ? rc : fail(GD_E_DEVICE, std::string("step graph capture: ") + hipGetErrorString(ce));
        }
        const hipError_t ie = hipGraphInstantiate(&s->step_graph, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (ie != hipSuccess) {
            s->step_graph = nullptr;
            return fail(GD_E_DEVICE, std::string("step graph: ") + hipGetErrorString(ie));
        }
        s->step_graph_cur = cur0;
        // capture only recorded the steps; s->cur has come back to cur0
    }
    GD_HIP(hipGraphLaunch(s->step_graph, s->stream));
    return GD_OK;
}

int gd_run(gd_solver *s, int32_t batch, int64_t steps) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_run(s->batch, batch, steps);
    if (steps < 0) return fail(GD_E_INVALID_ARG, "steps must be >= 0");
    int rc;
    if (!s->have_state) {
        if ((rc = gd_set_init(s, batch, nullptr, nullptr, nullptr)) != GD_OK) return rc;
    } else if (batch != s->R) {
        return fail(GD_E_INVALID_ARG, "batch differs from the current number of trajectories");
    }
    const bool timed = (s->prm.flags & GD_F_PROFILE) != 0;
    s->ev_used = 0;
    s->ev_launches = 0;
    const auto t0 = std::chrono::steady_clock::now();
    const int ci = s->prm.check_interval;
    // Np <= 128, FP32 (no pinned variant): the fused multi-step kernel, one
    // event pair per launch when profiled, counting its coupling evaluations
    // (those of its steps, and J d of an energy check that closes it) as
    // launches.  Otherwise small problems replay captured
    // graphs, except with profiling events, noise (its key changes every
    // step) or GD-mod.  Problems whose J fits the registers of the chip run
    // persistent steps, a bounded number per launch, whatever the chunk: a
    // trajectory does not depend on how a run is cut (but for launches that the
    // runtime refuses or that give up: the steps from there on are the coupling
    // kernels', which add in another order).
    const bool rk4 = s->integrator() == GD_RK4;
    const bool small_ok = !s->mod() && s->op == OP_F32 && s->Np <= 128 &&
                          std::getenv("GD_DENSE_CONFIG") == nullptr;
    if (steps_read_tiles(s) && (rc = tile_couplings(s)) != GD_OK) return rc;   // (at set-up, unless GD_DENSE_CONFIG changed)
    // The matrix-vector kernels of few trajectories run for microseconds, so
    // they are always replayed from graphs (with GD_F_PROFILE one event pair
    // brackets each replay and its launches, in-graph dispatch gaps included).
    const bool gemv_path = s->cfg.id >= kGemvBase;
    const bool graph_ok = !small_ok && s->prm.noise_D == 0.0 && !s->mod() &&
                          (gemv_path || (!timed && (long long)s->Np * s->Np * s->Rp * s->P < kGraphWork));
    // Without a target (nothing to stop on or to time) the best energy of
    // the checks is kept on the device and read back with the run's end.
    const bool deferred = ci > 0 && !s->prm.has_target && !s->track_target &&
                          !(s->prm.flags & GD_F_ASYNC);
    // What the host reads of the run at its end is written to pinned memory by
    // the kernel that ends its last check or steps.
    const bool async = (s->prm.flags & GD_F_ASYNC) != 0;
    if (!async && !s->hres) GD_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->hres), sizeof(RunResult)));
    bool first_check = true, ended = false;
    auto end_of = [&](bool check, bool run_end) {
        CheckEnd c;
        c.R = s->R;
        c.count = s->arrivals;
        if (deferred) {
            c.run_e = s->dE + s->Rp + 1;
            c.run_i = s->dBest + 1;
            c.first = first_check;
            c.e0 = s->best_energy;
            c.i0 = s->best_index;
        }
        if (check) {
            c.E = s->dE;
            c.best = s->dBest;
            c.best_e = s->dE + s->Rp;
            first_check = false;
        }
        if (s->persist >= 0) c.stalled = s->stalled;
        if (run_end) {
            c.flags = s->flags;
            c.out = s->hres;
            ended = true;
        }
        return c;
    };
    auto trace_slot = [&](int64_t step) -> double * {
        if (s->trace_steps.size() >= (size_t)kTraceChecks) return nullptr;
        s->trace_steps.push_back(step);
        return s->dTrace + s->trace_steps.size() - 1;
    };
    // Recording the time to target without stopping: each check is read back
    // one check later (the next chunk is queued meanwhile) and timed by
    // events from the start of the run.
    const bool lookahead = ci > 0 && s->track_target && !s->prm.has_target &&
                           !(s->prm.flags & GD_F_ASYNC);
    int pend = -1;              // slot of the check not yet read, or -1
    int64_t pend_step = 0;
    // a time to target (recorded, or a stop) is device time: events at the
    // start of each call and after each check
    const bool clocked = ci > 0 && (s->prm.has_target || s->track_target);
    if (lookahead && !s->hchk)
        GD_HIP(hipHostMalloc(reinterpret_cast<void **>(&s->hchk), 2 * sizeof(gd_solver::CheckSlot)));
    if (clocked) {
        for (hipEvent_t *e : {&s->ev_chk[0], &s->ev_chk[1], &s->ev_run0, &s->ev_end})
            if (!*e) GD_HIP(hipEventCreate(e));
        GD_HIP(hipEventRecord(s->ev_run0, s->stream));
    }
    const double clock0 = s->clock_s;
    // host rule of a check read back: best energy, first check at the
    // target (returns true at that check)
    auto take_check = [&](double emin, int bi, int64_t step, double seconds) -> bool {
        if (emin < s->best_energy) {
            s->best_energy = emin;
            s->best_index = bi;
        }
        if ((s->prm.has_target || s->track_target) && !s->target_reached && emin <= s->prm.target_energy) {
            s->target_reached = 1;
            s->ttt_steps = step;
            s->ttt_seconds = seconds;
            return true;
        }
        return false;
    };
    auto read_pending = [&]() -> int {
        if (pend < 0) return GD_OK;
        GD_HIP(hipEventSynchronize(s->ev_chk[pend]));
        float ms = 0.0f;
        GD_HIP(hipEventElapsedTime(&ms, s->ev_run0, s->ev_chk[pend]));
        take_check(s->hchk[pend].e, s->hchk[pend].i, pend_step, clock0 + ms * 1e-3);
        pend = -1;
        return GD_OK;
    };
    int64_t done = 0;
    // A persistent launch gave up (`tag`: the steps of this call done before it
    // and the amplitude buffer it read): back to the state it started from, and
    // one launch per step from there on.
    auto step_by_launch = [&](long long tag) {
        const int64_t back = done - ((tag - 1) >> 1);
        const int cur = int((tag - 1) & 1);
        if (s->cur != cur) std::swap(s->gam, s->gam_s);   // (a persistent launch swaps both)
        s->cur = cur;
        done -= back;
        s->steps_done -= back;
        s->spin_updates -= (int64_t)s->n * s->R * back;
        while (!s->trace_steps.empty() && s->trace_steps.back() > s->steps_done) s->trace_steps.pop_back();
        s->persist = -1;
        ended = false;
    };
take_steps:
    while (done < steps) {
        int64_t chunk = steps - done;
        if (ci > 0) {
            const int64_t to_check = ci - (s->steps_done % ci);
            chunk = std::min<int64_t>(chunk, to_check);
        }
        int64_t k = 0;
        const bool check_due = ci > 0 && (s->steps_done + chunk) % ci == 0, last = !async && done + chunk == steps;
        if (small_ok) {
            // all steps of the chunk in LDS, a bounded number per launch
            while (k < chunk) {
                const int m = int(std::min<int64_t>(chunk - k, kSmallStepsPerLaunch));
                DenseStepArgs a = base_args(s);
                a.J = s->dJs;
                a.psi_in = s->psi[s->cur];
                a.psi_out = s->psi[s->cur ^ 1];
                a.gam_in = s->gam;
                a.gam_out = s->gam;
                if (timed && (rc = ev_begin(s)) != GD_OK) return rc;
                if (s->prm.noise_D != 0.0) a.noise_amp = float(s->prm.noise_D * std::sqrt(double(a.dt)));
                // the launch that ends at a check also forms its energies
                CheckEnd c;
                const bool tail = k + m == chunk;
                if (tail && (check_due || last)) c = end_of(check_due, last);
                if (tail && check_due) c.trace = trace_slot(s->steps_done + chunk);
                GD_HIP(launch_small_steps(s->complex_mode(), rk4, a, m, s->prm.noise_seed, s->steps_done + k,
                                          s->ro, s->prm.q, c, s->stream));
                if (timed && (rc = ev_end(s, m * (rk4 ? 4 : 1) + (c.E ? 1 : 0))) != GD_OK) return rc;
                s->cur ^= 1;
                k += m;
            }
        }
        bool behind = false;
        while (s->persist >= 0 && k < chunk) {
            const int m = int(std::min<int64_t>(chunk - k, kPersistSteps));
            DenseStepArgs a = base_args(s);
            a.J = s->dJ8 ? s->dJ8 : (const void *)s->dJ;
            set_scales(s, rk4 ? MODE_RK1 : MODE_EULER, kAmpExp, a);
            a.psi_in = s->psi[s->cur];
            a.psi_out = s->psi[s->cur ^ 1];
            a.gam_in = s->gam;
            a.gam_out = s->gam_s;
            if (s->prm.noise_D != 0.0) a.noise_amp = float(s->prm.noise_D * std::sqrt(double(a.dt)));
            PersistArgs p{};
            p.x = s->xchg;
            p.stalled = s->stalled;
            p.tag = 2 * (done + k) + s->cur + 1;
            p.base = s->xbase;
            p.t0 = s->steps_done + k;
            p.seed = s->prm.noise_seed;
            p.patience = s->patience;
            p.steps = m;
            if (timed && (rc = ev_begin(s)) != GD_OK) return rc;
            CheckEnd c;
            if (last && !check_due && k + m == chunk && persist_ends_run(s->persist)) c = end_of(false, true);
            const hipError_t pe = s->persist_left == 0 ? hipErrorCooperativeLaunchTooLarge
                                                       : launch_persist(s->persist, s->complex_mode(), rk4,
                                                                        s->dJ8 != nullptr, a, p, c, s->stream);
            if (pe != hipSuccess) {
                (void)hipGetLastError();
                // refused (hipErrorIllegalState: cooperative launches of another
                // process on the device): one launch per step from here on, or
                // from an earlier launch of this call that gave up
                if (pe != hipErrorIllegalState && pe != hipErrorCooperativeLaunchTooLarge &&
                    pe != hipErrorLaunchOutOfResources)
                    return fail(GD_E_DEVICE, std::string("persistent steps: ") + hipGetErrorString(pe));
                ended = false;
                long long tag = 0;
                GD_HIP(hipMemcpyAsync(&tag, s->stalled, sizeof tag, hipMemcpyDeviceToHost, s->stream));
                GD_HIP(hipStreamSynchronize(s->stream));
                if ((behind = tag != 0)) step_by_launch(tag);
                s->persist = -1;
                if (steps_read_tiles(s) && (rc = tile_couplings(s)) != GD_OK) return rc;
                break;
            }
            if (s->persist_left > 0) --s->persist_left;
            if (timed && (rc = ev_end(s, m * (rk4 ? 4 : 1))) != GD_OK) return rc;
            s->xbase += m * (rk4 ? 4 : 1);
            s->cur ^= 1;
            std::swap(s->gam, s->gam_s);
            k += m;
        }
        if (behind) continue;
        if (graph_ok) {
            for (; chunk - k >= kGraphSteps; k += kGraphSteps) {
                if (timed && (rc = ev_begin(s)) != GD_OK) return rc;
                if ((rc = launch_step_graph(s)) != GD_OK) return rc;
                if (timed && (rc = ev_end(s, kGraphSteps * (rk4 ? 4 : 1))) != GD_OK) return rc;
            }
        }
        for (; k < chunk; ++k) {
            // GD_F_PROFILE: HIP events around the coupling launches of every
            // kProfileEvery-th step only, so the events barely perturb the run
            const bool sample = timed && ((s->steps_done + k) % kProfileEvery == 0);
            if ((rc = enqueue_step(s, s->cfg, -1.0f, sample, s->steps_done + k)) != GD_OK) return rc;
        }
        done += chunk;
        s->steps_done += chunk;
        s->spin_updates += (int64_t)s->n * s->R * chunk;
        if (ci > 0 && s->steps_done % ci == 0) {
            // device check: energy GEMM of the readout, deterministic reduction
            // (small problems: done by the last step launch)
            if (!small_ok) {
                int ntiles = 0;
                if ((rc = device_energies(s, &ntiles)) != GD_OK) return rc;
                CheckEnd c = end_of(true, last);
                c.trace = trace_slot(s->steps_done);
                GD_HIP(launch_energy_reduce(s->partial, ntiles, s->Rp, c, s->stream));
            }
            if (deferred) continue;
            if (lookahead) {
                const int slot = pend == 0 ? 1 : 0;
                GD_HIP(hipMemcpyAsync(&s->hchk[slot].e, s->dE + s->Rp, sizeof(double), hipMemcpyDeviceToHost,
                                      s->stream));
                GD_HIP(hipMemcpyAsync(&s->hchk[slot].i, s->dBest, sizeof(int), hipMemcpyDeviceToHost, s->stream));
                GD_HIP(hipEventRecord(s->ev_chk[slot], s->stream));
                if ((rc = read_pending()) != GD_OK) return rc;
                pend = slot;
                pend_step = s->steps_done;
                continue;
            }
            double emin = 0.0;
            int bi = 0;
            GD_HIP(hipMemcpyAsync(&bi, s->dBest, sizeof(int), hipMemcpyDeviceToHost, s->stream));
            GD_HIP(hipMemcpyAsync(&emin, s->dE + s->Rp, sizeof(double), hipMemcpyDeviceToHost, s->stream));
            if (clocked) GD_HIP(hipEventRecord(s->ev_chk[0], s->stream));
            GD_HIP(hipStreamSynchronize(s->stream));
            float ms = 0.0f;
            if (clocked) GD_HIP(hipEventElapsedTime(&ms, s->ev_run0, s->ev_chk[0]));
            const bool hit = take_check(emin, bi, s->steps_done, clock0 + ms * 1e-3);
            if (hit && s->prm.has_target) break;
        }
    }
    if (s->prm.flags & GD_F_ASYNC) return GD_OK;
    if ((rc = read_pending()) != GD_OK) return rc;
    if (clocked) GD_HIP(hipEventRecord(s->ev_end, s->stream));
    // one wait for the steps and for what the host reads of them
    if (!ended) GD_HIP(launch_check_end(end_of(false, true), s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    if (const long long tag = s->hres->stalled) {
        step_by_launch(tag);
        if (steps_read_tiles(s) && (rc = tile_couplings(s)) != GD_OK) return rc;
        goto take_steps;
    }
    s->run_seconds += std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (clocked) {
        float ms = 0.0f;
        GD_HIP(hipEventElapsedTime(&ms, s->ev_run0, s->ev_end));
        s->clock_s += ms * 1e-3;
    }
    if (timed) {
        for (int64_t k = 0; k < s->ev_used; ++k) {
            float ms = 0.0f;
            GD_HIP(hipEventElapsedTime(&ms, s->events[(size_t)k * 2], s->events[(size_t)k * 2 + 1]));
            s->kernel_ms += ms;
        }
        s->launches_timed += s->ev_launches;
        s->ev_used = 0;
        s->ev_launches = 0;
    }
    const int cnt = s->hres->diverged;
    s->diverged = cnt;
    if (deferred) {
        s->best_energy = s->hres->best_e;
        s->best_index = s->hres->best_i;
    }
    if (cnt) {
        char buf[64];
        std::snprintf(buf, sizeof buf, "%d trajectories became non-finite", cnt);
        return fail(GD_E_DIVERGED, buf);
    }
    return GD_OK;
}

static int energies(gd_solver *s, double *E, int32_t *best, bool fp64) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_energy(s->batch, E, best);
    if (!s->have_state) return fail(GD_E_STATE, "no state: call gd_set_init or gd_run first");
    if (!E) return fail(GD_E_INVALID_ARG, "E is NULL");
    int ntiles = s->Np / 64, rc;
    // Integer couplings and fields: the sums of the signs are exact in FP32
    // and the terms in FP64, in any order, so the FP8 path gives the FP64
    // re-score's numbers (N = R = 4096: 0.16 ms against 2.4 ms)
    const bool exact = fp64 && sign_readout(s) && s->j_integer && s->j_sums24 && s->g_integer;
    if (exact) {
        if ((rc = tile_couplings(s)) != GD_OK) return rc;
        DenseStepArgs a = base_args(s);
        a.J = s->dJt;
        a.B = a.psi_in = s->psi[s->cur];
        GD_HIP(launch_sign_energy(a, s->stream));
        const int bm = sign_energy_row_tile(s->Np, s->R);
        ntiles = (s->Np + bm - 1) / bm;
    } else if (fp64) {
        if (!s->D64 && (rc = dalloc(&s->D64, (size_t)s->plane() * s->P)) != GD_OK) return rc;
        GD_HIP(launch_energy_fp64(s->dJ, s->psi[s->cur], s->dG, s->D64, s->partial, s->Np, s->Rp, s->n, s->R, s->P,
                                  s->plane(), s->ro, s->prm.q, s->stream));
    } else if ((rc = device_energies(s, &ntiles)) != GD_OK) {
        return rc;
    }
    CheckEnd c;
    c.E = s->dE;
    c.R = s->R;
    c.best = s->dBest;
    c.best_e = s->dE + s->Rp;
    c.count = s->arrivals;
    GD_HIP(launch_energy_reduce(s->partial, ntiles, s->Rp, c, s->stream));
    int bi = 0;
    if (s->prm.flags & GD_F_DEVICE_PTRS) {
        GD_HIP(hipMemcpyAsync(E, s->dE, sizeof(double) * s->R, hipMemcpyDeviceToDevice, s->stream));
        if (best) GD_HIP(hipMemcpyAsync(best, s->dBest, sizeof(int), hipMemcpyDeviceToDevice, s->stream));
    } else {
        GD_HIP(hipMemcpyAsync(E, s->dE, sizeof(double) * s->R, hipMemcpyDeviceToHost, s->stream));
        GD_HIP(hipMemcpyAsync(&bi, s->dBest, sizeof(int), hipMemcpyDeviceToHost, s->stream));
    }
    GD_HIP(hipStreamSynchronize(s->stream));
    if (best && !(s->prm.flags & GD_F_DEVICE_PTRS)) *best = bi;
    return GD_OK;
}

int gd_energy(gd_solver *s, double *E, int32_t *best) { return energies(s, E, best, true); }

int gd_energy_device(gd_solver *s, double *E, int32_t *best) { return energies(s, E, best, false); }

int gd_spins(gd_solver *s, void *out, int32_t fmt) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) {
        if (!out) return fail(GD_E_INVALID_ARG, "out is NULL");
        return batch_spins(s->batch, out, fmt);
    }
    if (!s->have_state) return fail(GD_E_STATE, "no state");
    if (!out) return fail(GD_E_INVALID_ARG, "out is NULL");
    if (fmt != GD_SPINS_I8 && fmt != GD_SPINS_ANGLE_F32 && fmt != GD_SPINS_STATE_I32)
        return fail(GD_E_INVALID_ARG, "unknown format");
    if (fmt == GD_SPINS_I8 && s->ro != RO_SIGN && s->ro != RO_SIGN_RE)
        return fail(GD_E_INVALID_ARG, "int8 spins need an Ising model");
    if (fmt == GD_SPINS_STATE_I32 && s->ro != RO_CLOCK)
        return fail(GD_E_INVALID_ARG, "int32 states need the Potts model");
    const size_t cnt = (size_t)s->R * s->n;
    const size_t bytes = cnt * (fmt == GD_SPINS_I8 ? 1 : 4);
    // straight into the caller's device memory, else through a buffer
    const bool direct = (s->prm.flags & GD_F_DEVICE_PTRS) &&
                        (fmt == GD_SPINS_I8 || reinterpret_cast<uintptr_t>(out) % 4 == 0) && device_span(s, out, bytes);
    void *tmp = out;
    if (!direct) GD_HIP(hipMalloc(&tmp, bytes));
    hipError_t e = launch_discretise(s->psi[s->cur], nullptr, nullptr, OP_F32, s->ro, s->prm.q,
                                     fmt == GD_SPINS_I8 ? static_cast<int8_t *>(tmp) : nullptr,
                                     fmt == GD_SPINS_ANGLE_F32 ? static_cast<float *>(tmp) : nullptr,
                                     fmt == GD_SPINS_STATE_I32 ? static_cast<int32_t *>(tmp) : nullptr,
                                     s->flags, s->n, s->R, s->Np, s->Rp, s->P, s->plane(), s->stream);
    if (e == hipSuccess && !direct)
        e = hipMemcpyAsync(out, tmp, bytes,
                           (s->prm.flags & GD_F_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                           s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (!direct) (void)hipFree(tmp);
    if (e != hipSuccess) return fail(GD_E_DEVICE, std::string("gd_spins: ") + hipGetErrorString(e));
    return GD_OK;
}

int gd_spins_noalloc(gd_solver *s, void *out, int32_t fmt) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return fail(GD_E_UNSUPPORTED, "gd_spins_noalloc serves single-instance solvers");
    if (!s->have_state) return fail(GD_E_STATE, "no state");
    if (!out) return fail(GD_E_INVALID_ARG, "out is NULL");
    if (fmt != GD_SPINS_I8 && fmt != GD_SPINS_ANGLE_F32 && fmt != GD_SPINS_STATE_I32)
        return fail(GD_E_INVALID_ARG, "unknown format");
    if (fmt == GD_SPINS_I8 && s->ro != RO_SIGN && s->ro != RO_SIGN_RE)
        return fail(GD_E_INVALID_ARG, "int8 spins need an Ising model");
    if (fmt == GD_SPINS_STATE_I32 && s->ro != RO_CLOCK)
        return fail(GD_E_INVALID_ARG, "int32 states need the Potts model");
    const size_t bytes = (size_t)s->R * s->n * (fmt == GD_SPINS_I8 ? 1 : 4);
    if (bytes > kScratchBytes) {
        char buf[160];
        std::snprintf(buf, sizeof buf, "gd_spins_noalloc: %zu bytes of spins exceed its %zu-byte staging array",
                      bytes, kScratchBytes);
        return fail(GD_E_INVALID_ARG, buf);
    }
    void *stage = nullptr;
    int rc = scratch_address(s->device, &stage);
    if (rc != GD_OK) return rc;
    // the readout kernel writes every one of the R x n entries, so nothing
    // left over from an earlier call is read back
    GD_HIP(launch_discretise(s->psi[s->cur], nullptr, nullptr, OP_F32, s->ro, s->prm.q,
                             fmt == GD_SPINS_I8 ? static_cast<int8_t *>(stage) : nullptr,
                             fmt == GD_SPINS_ANGLE_F32 ? static_cast<float *>(stage) : nullptr,
                             fmt == GD_SPINS_STATE_I32 ? static_cast<int32_t *>(stage) : nullptr,
                             s->flags, s->n, s->R, s->Np, s->Rp, s->P, s->plane(), s->stream));
    GD_HIP(hipMemcpyAsync(out, stage, bytes,
                          (s->prm.flags & GD_F_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                          s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    return GD_OK;
}

int gd_get_state(gd_solver *s, float *psi, float *gamma, int64_t *step) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_get_state(s->batch, psi, gamma, step);
    if (!s->have_state) return fail(GD_E_STATE, "no state");
    int rc;
    const bool both = psi && gamma && (s->prm.flags & GD_F_DEVICE_PTRS) != 0 &&
                      (reinterpret_cast<uintptr_t>(psi) | reinterpret_cast<uintptr_t>(gamma)) % 4 == 0 &&
                      device_span(s, psi, (size_t)s->R * s->n * s->P * sizeof(float)) &&
                      device_span(s, gamma, (size_t)s->R * s->n * sizeof(float));
    if (both) {
        GD_HIP(launch_unpack_state(s->psi[s->cur], psi, s->gam, gamma, s->n, s->R, s->Np, s->Rp, s->P, s->stream));
    } else {
        if (psi && (rc = download_planes(s, s->psi[s->cur], psi, s->P)) != GD_OK) return rc;
        if (gamma && (rc = download_planes(s, s->gam, gamma, 1)) != GD_OK) return rc;
    }
    if (psi || gamma) GD_HIP(hipStreamSynchronize(s->stream));
    if (step) *step = s->steps_done;
    return GD_OK;
}

int gd_set_state(gd_solver *s, int32_t batch, const float *psi, const float *gamma, int64_t step) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_set_state(s->batch, batch, psi, gamma, step);
    if (!psi || !gamma) return fail(GD_E_INVALID_ARG, "psi and gamma are required");
    if (batch < 1 || batch > (1 << 22) || step < 0) return fail(GD_E_INVALID_ARG, "bad batch or step");
    std::vector<float> chk;
    int rc;
    if ((rc = copy_in(s, psi, (size_t)batch * s->n * s->P, chk)) != GD_OK) return rc;
    if (!all_finite(chk)) return fail(GD_E_NONFINITE, "psi has non-finite entries");
    if ((rc = copy_in(s, gamma, (size_t)batch * s->n, chk)) != GD_OK) return rc;
    if (!all_finite(chk)) return fail(GD_E_NONFINITE, "gamma has non-finite entries");
    if (!s->have_state || batch != s->R) {
        if ((rc = alloc_state(s, batch)) != GD_OK) return rc;
        if ((rc = prepare_steps(s)) != GD_OK) return rc;
    }
    reset_stats(s);
    s->cur = 0;
    GD_HIP(hipMemsetAsync(s->tiny, 0, sizeof(int), s->stream));
    if ((rc = upload_planes(s, psi, s->psi[0], batch)) != GD_OK) return rc;
    const int savedP = s->P;
    s->P = 1;
    rc = upload_planes(s, gamma, s->gam, batch);
    s->P = savedP;
    if (rc != GD_OK) return rc;
    GD_HIP(refresh_shadow(s, 0));
    if ((rc = reset_mod_couplings(s)) != GD_OK) return rc;
    GD_HIP(hipMemsetAsync(s->flags, 0, (size_t)s->Rp * sizeof(int), s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    s->steps_done = step;
    return GD_OK;
}

int gd_mod_couplings(gd_solver *s, int32_t traj, float *K) {
    if (!s || !K) return fail(GD_E_INVALID_ARG, "NULL argument");
    if (s->batch || !s->mod()) return fail(GD_E_INVALID_ARG, "not a GD-mod solver");
    if (!s->have_state || !s->K) return fail(GD_E_STATE, "no state");
    if (traj < 0 || traj >= s->R) return fail(GD_E_INVALID_ARG, "trajectory out of range");
    const hipMemcpyKind kind =
        (s->prm.flags & GD_F_DEVICE_PTRS) ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    if (s->K_packed) {
        const float *src = s->K + (size_t)traj * gdmod_packed_floats(s->Np);
        // straight into the caller's device memory, else through a buffer
        const size_t m = (size_t)s->n * s->n;
        const bool direct = (s->prm.flags & GD_F_DEVICE_PTRS) && reinterpret_cast<uintptr_t>(K) % 4 == 0 &&
                            device_span(s, K, m * sizeof(float));
        float *full = K;
        if (!direct) {
            const int rc = dalloc(&full, m);
            if (rc != GD_OK) return rc;
        }
        hipError_t e = launch_gdmod_unpack(src, full, s->Np, s->n, s->stream);
        const size_t row = (size_t)s->n * sizeof(float);
        if (e == hipSuccess && !direct) e = hipMemcpy2DAsync(K, row, full, row, row, (size_t)s->n, kind, s->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
        if (!direct) (void)hipFree(full);
        GD_HIP(e);
        return GD_OK;
    }
    const float *src = s->K + (size_t)traj * s->Np * s->Np;
    GD_HIP(hipMemcpy2DAsync(K, (size_t)s->n * sizeof(float), src, (size_t)s->Np * sizeof(float),
                            (size_t)s->n * sizeof(float), (size_t)s->n, kind, s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    return GD_OK;
}

int gd_stats(gd_solver *s, gd_run_stats *out) {
    if (!s || !out) return fail(GD_E_INVALID_ARG, "NULL argument");
    if (out->struct_size != sizeof(gd_run_stats)) return fail(GD_E_INVALID_ARG, "gd_run_stats.struct_size mismatch");
    if (s->batch) return batch_stats(s->batch, out);
    out->batch = s->R;
    out->steps_done = s->steps_done;
    out->spin_updates = s->spin_updates;
    out->run_seconds = s->run_seconds;
    out->kernel_ms = s->kernel_ms;
    out->kernel_launches = s->launches_timed;
    out->diverged = s->diverged;
    out->target_reached = s->target_reached;
    out->ttt_seconds = s->ttt_seconds;
    out->ttt_steps = s->ttt_steps;
    out->best_energy = s->best_energy;
    out->best_index = s->best_index;
    // (until a run: the variant that energy checks use)
    out->kernel_config = s->persist >= 0 && s->xbase > 0 ? kPersistBase + s->persist : s->cfg.id;
    return GD_OK;
}

int gd_trajectory_status(gd_solver *s, int32_t *out, int64_t count) {
    if (!s || !out) return fail(GD_E_INVALID_ARG, "NULL argument");
    if (s->batch) return batch_trajectory_status(s->batch, out, count);
    if (!s->have_state) return fail(GD_E_STATE, "no state: call gd_set_init or gd_run first");
    if (count != s->R) return fail(GD_E_INVALID_ARG, "count must equal the number of trajectories");
    static_assert(sizeof(int) == sizeof(int32_t), "flag words are 32-bit");
    GD_HIP(hipMemcpyAsync(out, s->flags, (size_t)count * sizeof(int), hipMemcpyDeviceToHost, s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    for (int64_t r = 0; r < count; ++r) out[r] = out[r] != 0;
    return GD_OK;
}

int gd_best_trace(gd_solver *s, int64_t *steps, double *best, int32_t cap, int32_t *count) {
    if (!s || !count) return fail(GD_E_INVALID_ARG, "NULL argument");
    if (s->batch) return fail(GD_E_INVALID_ARG, "no energy trace for a batch of instances (see gd_ttt)");
    if (cap < 0) return fail(GD_E_INVALID_ARG, "cap must be >= 0");
    const int32_t n = (int32_t)s->trace_steps.size();
    *count = n;
    const int32_t m = std::min(n, cap);
    if (m == 0) return GD_OK;
    if (!steps || !best) return fail(GD_E_INVALID_ARG, "NULL argument");
    GD_HIP(hipMemcpyAsync(best, s->dTrace, (size_t)m * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    GD_HIP(hipStreamSynchronize(s->stream));
    for (int32_t k = 0; k < m; ++k) {
        steps[k] = s->trace_steps[(size_t)k];
        if (k > 0 && best[k - 1] < best[k]) best[k] = best[k - 1];
    }
    return GD_OK;
}

int gd_coupling_scale(gd_solver *s, double *scale) {
    if (!s || !scale) return fail(GD_E_INVALID_ARG, "NULL argument");
    if (s->batch) {
        *scale = batch_scale(s->batch, 0);
        return GD_OK;
    }
    *scale = s->s;
    return GD_OK;
}

int gd_create_batch(gd_solver **out, int32_t count, const gd_instance *inst, int32_t model,
                    const gd_params *p) {
    if (!out) return fail(GD_E_INVALID_ARG, "out is NULL");
    *out = nullptr;
    gd_params prm;
    if (p) prm = *p;
    else gd_default_params(&prm);
    int rc = check_params(&prm);
    if (rc != GD_OK) return rc;
    gd::BatchSolver *b = nullptr;
    if ((rc = batch_create(&b, count, inst, model, &prm)) != GD_OK) return rc;
    gd_solver *s = new (std::nothrow) gd_solver();
    if (!s) {
        batch_destroy(b);
        return fail(GD_E_OOM, "host allocation failed");
    }
    s->batch = b;
    s->prm = prm;
    s->model = model;
    *out = s;
    return GD_OK;
}

int gd_set_targets(gd_solver *s, const double *targets) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_set_targets(s->batch, targets);
    s->track_target = targets != nullptr;
    if (targets) s->prm.target_energy = targets[0];
    s->target_reached = 0;
    return GD_OK;
}

int gd_ttt(gd_solver *s, double *seconds, int64_t *steps, double *best_energy) {
    if (!s) return fail(GD_E_INVALID_ARG, "solver is NULL");
    if (s->batch) return batch_ttt(s->batch, seconds, steps, best_energy);
    if (seconds) *seconds = s->target_reached ? s->ttt_seconds : -1.0;
    if (steps) *steps = s->target_reached ? s->ttt_steps : -1;
    if (best_energy) *best_energy = s->best_energy;
    return GD_OK;
}

}  // extern "C"

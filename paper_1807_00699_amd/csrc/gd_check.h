// The end of an energy check or of a run, done by the last workgroup to finish
// of the kernel that formed its inputs, instead of a kernel of its own
// (3-5 us each with its launch; Ising N = 64, R = 100, 100 steps and two checks:
// 66 us with four such kernels).  Up to kEndRows trajectories: every arrival is
// an atomic on one word (14 ns each), and one wave reads the trajectories'
// results.  Ising N = 64, 20 steps, a check every two: R = 64 75 us so, 86 with a
// launch for every end; R = 200 88-92 and 77-100 (the host's time to launch);
// R = 400 114-122 and 76-102; R = 4000 628 and 120.
#pragma once
#include "gd_internal.h"

namespace gd {

constexpr int kEndRows = 256;

// stores that the last workgroup reads (any CU, in the same launch)
__device__ inline void store_agent(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_agent(long long *p, long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void store_agent(int *p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in every thread of the last of `total` workgroups to call it; the
// store_agent stores of all of them have arrived then.  *count is zero before
// and after.
__device__ inline bool last_arrival(unsigned *count, unsigned total) {
    __shared__ bool last;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        last = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == total - 1;
        if (last) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return last;
}

// By one workgroup of whole waves (at most 16): with c.E, b = argmin_r E[r]
// (ties: the lowest r) into best, E[b] into best_e and trace, and the running
// best; with c.out, what the host reads at the end of a run.  Energies of steps
// that were not taken (*c.stalled) read as NaN, below no target and no best.  A thread has the
// loads of U trajectories in flight.
template <int U = 1>
__device__ inline void check_end(const CheckEnd &c) {
    const long long stalled = c.stalled ? __hip_atomic_load(c.stalled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    __shared__ double se[16];
    __shared__ int si[16], sc[16];
    double bv = __builtin_inf();
    int bi = 0x7fffffff, bad = 0;
    for (int r0 = threadIdx.x; r0 < c.R; r0 += U * blockDim.x) {
        double s[U];
        int f[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = min(r0 + u * int(blockDim.x), c.R - 1);
            s[u] = c.E ? __hip_atomic_load(c.E + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : bv;
            f[u] = c.out ? __hip_atomic_load(c.flags + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * int(blockDim.x);
            if (r >= c.R) break;
            if (c.E && (s[u] < bv || (s[u] == bv && r < bi))) {
                bv = s[u];
                bi = r;
            }
            bad += f[u] != 0;
        }
    }
    auto merge = [&](double ov, int oi, int ob) {
        if (ov < bv || (ov == bv && oi < bi)) {
            bv = ov;
            bi = oi;
        }
        bad += ob;
    };
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) merge(__shfl_xor(bv, m), __shfl_xor(bi, m), __shfl_xor(bad, m));
    if ((threadIdx.x & 63) == 0) {
        se[threadIdx.x >> 6] = bv;
        si[threadIdx.x >> 6] = bi;
        sc[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (unsigned w = 1; w < blockDim.x / 64; ++w) merge(se[w], si[w], sc[w]);
    double run = c.first ? c.e0 : 0.0;
    int run_i = c.i0;
    if (c.run_e && !c.first) {
        run = *c.run_e;
        run_i = *c.run_i;
    }
    if (c.E) {
        const int b = bi == 0x7fffffff ? 0 : bi;
        const double eb = stalled ? __builtin_nan("") : bi == 0x7fffffff ? __hip_atomic_load(c.E, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : bv;
        if (c.best) *c.best = b;
        if (c.best_e) *c.best_e = eb;
        if (c.trace) *c.trace = eb;
        if (c.run_e) {
            if (eb < run) {
                run = eb;
                run_i = b;
            }
            *c.run_e = run;
            *c.run_i = run_i;
        }
    }
    if (c.out) {
        c.out->diverged = bad;
        c.out->stalled = stalled;
        if (c.run_e) {
            c.out->best_e = run;
            c.out->best_i = run_i;
        }
    }
}

}  // namespace gd

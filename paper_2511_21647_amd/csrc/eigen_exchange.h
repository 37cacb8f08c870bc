// What the two cooperative eigensolvers (eigen.hip, eigen_lds.hip) share: the exchange
// between a plane's work-groups and its barrier.
#pragma once

#include "eigen.h"

#include <float.h>

namespace ulm {

constexpr int kCoopThreads = 256;
constexpr int kCoopWaves = kCoopThreads / 64;
constexpr int kCoopRows = 8;     // rows per lane of a column at most: F <= 512
constexpr int kPoints = 16;      // multisection points per eigenvalue and round
constexpr int kGroups = 64 / kPoints;   // eigenvalues per wave at a time
// Polls before a wait gives up and flags the status word, some seconds: far beyond what a
// work-group can be late for by another kernel on its CU, and far below a hang's limits.
constexpr int kMaxPolls = 1 << 23;

__device__ inline double2 cmul2(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline double bmax(double v, double *red) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = red[0];
    for (int i = 1; i < kCoopWaves; ++i) s = fmax(s, red[i]);
    return s;
}

// Cross-work-group traffic.  A plane's work-groups are dealt to one XCD when
// the kernel runs alone; kernels running at the same time on other streams
// shift the dispatcher's XCD rotation and can split a plane over XCDs, whose
// L2s are not coherent with each other.  Each work-group therefore sets its
// hardware XCC id's bit in a per-plane mask at system scope before the first
// grid barrier (which also runs at system scope), and the plane then runs in
// one of two modes:
//  - local: every work-group on one XCD.  They share its L2: plain stores, complete
//    once they reach it, and agent-scope loads (which miss the CU's L1 and read the
//    L2) exchange the data.  In the reduction the data is its own flag: a slot holds
//    kUnset (a NaN that no arithmetic produces) until its value is published, and a
//    reader loads until neither half of any value it needs is kUnset (8-byte accesses
//    are single).  Slots rotate over three steps.  A wave that has read all of step
//    k - 1 knows that every wave has read all of step k - 2, so during step k each
//    slot of step k - 2, the next to be written at step k + 1, is set back by its next
//    writer, complete before that writer publishes anything of step k; whoever reads
//    step k + 1 has by then read that.  Elsewhere a barrier is a plain flag store and
//    an agent-scope poll.
//  - fenced: the plane spans XCDs.  Stores and loads are agent-scope atomics,
//    and every exchange is a barrier: a release fence (L2 write-back) before a
//    system-scope flag store and an acquire fence (cache invalidation) after
//    a system-scope poll.
// A work-group arrives at a barrier only after its own stores have completed
// (s_waitcnt 0).  Up to 64 frames a plane has one work-group: it exchanges through
// LDS, and a barrier is the work-group's.
__device__ inline void st_c(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline double ld_c(const double *p) {
    return __hip_atomic_load(const_cast<double *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_c2(double2 *p, double2 v) {
    st_c((double *)p, v.x);
    st_c((double *)p + 1, v.y);
}
__device__ inline double2 ld_c2(const double2 *p) {
    return make_double2(ld_c((const double *)p), ld_c((const double *)p + 1));
}
__device__ inline void put(double *p, double v, bool local) {
    if (local) *p = v;
    else st_c(p, v);
}
__device__ inline void put2(double2 *p, double2 v, bool local) {
    if (local) *p = v;
    else st_c2(p, v);
}
// The XCC (XCD) this wave runs on.
__device__ inline int xcc_id() { return (int)(__builtin_amdgcn_s_getreg((15 << 11) | 20) & 0xf); }
__device__ inline void st_sys2(double2 *p, double2 v) {
    __hip_atomic_store((double *)p, v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store((double *)p + 1, v.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ inline double2 ld_sys2(const double2 *p) {
    return make_double2(
        __hip_atomic_load(const_cast<double *>((const double *)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM),
        __hip_atomic_load(const_cast<double *>((const double *)p + 1), __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_SYSTEM));
}
enum BarMode { kBarSystem, kBarFenced, kBarLocal, kBarSolo };
// Grid barrier among the W work-groups of one plane: work-group w publishes
// the number of barriers it has reached in its own flag, and lanes 0..W-1 of
// the first wave each wait for one work-group's flag, so no single counter is
// contended.  Returns false if the wait timed out (the caller then exits).
__device__ inline int load_flag(const int *p, BarMode mode) {
    int *q = const_cast<int *>(p);
    return mode == kBarLocal ? __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                             : __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ inline bool plane_barrier(int *flags, int w, int W, int step, int *abort_s, int *status,
                                     BarMode mode) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (mode == kBarSolo) return *abort_s == 0;      // the plane's only work-group
    if (threadIdx.x == 0) {
        if (mode == kBarLocal) {
            flags[w] = step;
        } else {
            if (mode == kBarFenced) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __hip_atomic_store(flags + w, step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    if ((int)threadIdx.x < W) {
        int spins = 0;
        while (load_flag(flags + threadIdx.x, mode) < step) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > kMaxPolls) {
                *abort_s = 1;
                atomicOr(status, kStatusBarrier);
                break;
            }
        }
    }
    __syncthreads();
    if (mode == kBarFenced) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return *abort_s == 0;
}

}  // namespace ulm

// FP64 Hermitian eigensolver for the clutter filter (paper Section II-A2: the
// covariance of the Casorati matrix is eigendecomposed and the eigenvectors of
// the largest eigenvalues span the clutter subspace).
//
// eigen_coop_kernel: W work-groups of four waves per plane, launched cooperatively;
// the plane's grid slots are dealt to one XCD (see the exchange modes below).
//   1. Householder reduction to real tridiagonal form T = Q^H C Q (the
//      unblocked Hermitian reduction).  Wave g of the plane's 4 W keeps columns g,
//      g + 4 W, .. of C in registers for the whole reduction (row i in lane i % 64,
//      register i / 64).  Every wave forms the reflector v_k itself from the published
//      column k, applies the rank-2 update of step k-1 to its columns in the same
//      pass as the product p_k = tau_k A v_k of step k, and publishes its part of p_k
//      and, if it owns it, column k+1.  The work-group then reads all of p and that
//      column into LDS, and every wave forms p^H v and applies the step's update to
//      column k+1.  A step is one exchange and one LDS barrier.
//   2. Every eigenvalue of T by multisection on Sturm counts (16 lanes per
//      eigenvalue, 16 points per round), spread over the plane's waves.
//   3. Inverse iteration (partial-pivoting tridiagonal LU in LDS) for the c
//      largest eigenvalues, one eigenvector per wave.
//   4. Work-group 0: Gram-Schmidt over the c vectors in LDS.
//   5. Back-transformation x = H_0 H_1 ... H_{F-2} y, one wave per vector with x in
//      registers.
// The reduction is bound by latency: a step's chain is the norm's and the products'
// sums over the lanes (DPP moves and lane swaps, not LDS permutes), a square root and
// two reciprocals, and one trip through the XCD's L2.  Against columns in LDS, a work-group
// barrier for each of a step's sums and a flag barrier for its exchange (eigen_lds.hip):
// 2 planes of 300 frames 2013 -> 1061 us (the reduction 1233 -> 750), 70 planes 10.8 ->
// 4.65 ms, 2 planes of 20 frames 120 -> 66 us.
// Waits are bounded: a wave that waits too long flags the status word and exits, so
// every wave always finishes.
#include "eigen_exchange.h"

namespace ulm {

// Sum over the wave's lanes, in every lane: neighbours, pairs, quads and halves of a
// row of 16 by DPP, rows and halves of the wave by lane swaps.  (A chain of six LDS
// permutes takes several times as long, and these sums are most of a step's chain.)
template <int CTRL>
__device__ inline double dpp_move(double v) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// Two values at once: the lower half-wave gets a's sum over the two halves and the
// upper b's (lane swap of the halves), or the even rows a's sums over row pairs and
// the odd rows b's.
__device__ inline double merge_swap(unsigned a0, unsigned a1, unsigned b0, unsigned b1) {
    return __builtin_bit_cast(double, (unsigned long long)b0 << 32 | a0) +
           __builtin_bit_cast(double, (unsigned long long)b1 << 32 | a1);
}
__device__ inline double merge_halves(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return merge_swap(l[0], l[1], h[0], h[1]);
}
__device__ inline double merge_rows(double a, double b) {
    const unsigned long long x = __builtin_bit_cast(unsigned long long, a), y = __builtin_bit_cast(unsigned long long, b);
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    return merge_swap(l[0], l[1], h[0], h[1]);
}
__device__ inline double row_sum(double v) {
    v += dpp_move<0xb1>(v);     // quad_perm 1,0,3,2
    v += dpp_move<0x4e>(v);     // quad_perm 2,3,0,1
    v += dpp_move<0x141>(v);    // row_half_mirror
    v += dpp_move<0x140>(v);    // row_mirror
    return v;
}
__device__ inline double wsum(double v) {
    v = merge_halves(v, v);
    return row_sum(merge_rows(v, v));
}
// Lane l's value in every lane (l uniform).
__device__ inline double lane_value(double v, int l) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// Sums of N complex values over the wave, in every lane: re and im share a register
// by halves, two values one by rows, so a value costs about a quarter of a wsum.
template <int N>
__device__ inline void wsum_complex(double2 (&v)[N]) {
    double r[(N + 1) / 2];
#pragma unroll
    for (int i = 0; i < N; i += 2) {
        const double a = merge_halves(v[i].x, v[i].y);
        const double b = i + 1 < N ? merge_halves(v[i + 1 < N ? i + 1 : i].x, v[i + 1 < N ? i + 1 : i].y) : a;
        r[i / 2] = merge_rows(a, b);
    }
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i) r[i] = row_sum(r[i]);
#pragma unroll
    for (int i = 0; i < N; ++i)
        v[i] = make_double2(lane_value(r[i / 2], 16 * (i & 1)), lane_value(r[i / 2], 32 + 16 * (i & 1)));
}
__device__ inline double bsum(double v, double *red) {
    v = wsum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < kCoopWaves; ++i) s += red[i];
    return s;
}
// 1 / sqrt(x) and 1 / x to about an ulp (the hardware's estimate and two Newton steps).
__device__ inline double rsqrt_newton(double x) {
    double r = __builtin_amdgcn_rsq(x);
    r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
    return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}
__device__ inline double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// x - a b and acc + conj(x) v as fused sums.
__device__ inline double2 sub_mul(double2 x, double2 a, double2 b) {
    return make_double2(fma(a.y, b.y, fma(-a.x, b.x, x.x)), fma(-a.y, b.x, fma(-a.x, b.y, x.y)));
}
__device__ inline double2 add_conj_mul(double2 acc, double2 x, double2 v) {
    return make_double2(fma(x.y, v.y, fma(x.x, v.x, acc.x)), fma(-x.y, v.x, fma(x.x, v.y, acc.y)));
}

constexpr unsigned kUnsetHi = 0x7ff8dead;       // upper word of an exchange slot not yet written
__device__ inline double2 unset2() {
    const double u = __builtin_bit_cast(double, (unsigned long long)kUnsetHi << 32);
    return make_double2(u, u);
}

// What a wave carries from step to step of the reduction (NR rows per lane, NC
// columns per wave), every array indexed by row / 64.
template <int NR, int NC>
struct Reduction {
    double2 col[NC][NR];    // own columns
    double2 x[NR];          // column k, every update applied (rows >= k)
    double2 v[NR], p[NR];   // the pending update's vectors (zero above their pivot)
    double a2r;             // 2 Re(alpha) of the pending update
    double nrm_part;        // this lane's share of the next reflector's |x_2..|^2
    double diag;            // d[k]
};

struct ReductionArgs {
    int F, gw, nwv, lane;
    bool local;             // one XCD
    int last_wg;            // the work-group's last column (-1: none)
    int c_off;              // bytes from pbuf to cbuf
    double2 *ex;            // LDS: p and column as read, [2][2 F] by step parity
    double2 *H, *tau;
    double *d, *e;
    double2 *pbuf, *cbuf;   // [3][F] exchange slots by step
    double2 *vl, *pl;       // LDS: this wave's copy of v and p
    int *flags, *abort_s, *status;
    int w, W;
};

// Steps whose pivot row k + 1 lies in row block MB: the blocks above it are done.
template <int NR, int NC, int MB>
__device__ inline bool reduce_steps(Reduction<NR, NC> &s, const ReductionArgs &a, int &nbar)
{
    constexpr bool kSolo = NR == 1;               // one work-group: LDS is the exchange
    const bool local = kSolo || a.local;
    const int F = a.F, lane = a.lane;
    const int kb1 = min(64 * (MB + 1), F);
    // both exchange areas in one descriptor: this plane's columns lie c_off past its p
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
        a.pbuf, 0, a.c_off + 3 * F * (int)sizeof(double2), 0x00027000);
    for (int kb = max(64 * MB, 1); kb < kb1; ++kb) {
        const int k = kb - 1, pl = kb & 63;
        const int now = k % 3 * F, next = (k + 1) % 3 * F;
        // set back the slots that this wave writes at the next step
        if (local && !kSolo) {
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                const int j = a.gw + q * a.nwv;
                if (j > kb && j < F) {
                    if (lane == 0) a.pbuf[next + j] = unset2();
                    if (j == kb + 1) {
#pragma unroll
                        for (int m = MB; m < NR; ++m) {
                            const int i = lane + 64 * m;
                            if (i > kb && i < F) a.cbuf[next + i] = unset2();
                        }
                    }
                }
            }
        }
        // reflector of column k (LAPACK's elementary reflector convention):
        // H^H x = (beta, 0, ...)^T, H = I - tau v v^H, v_{k+1} = 1
        const double nrm = wsum(s.nrm_part);
        const double2 alpha = make_double2(lane_value(s.x[MB].x, pl), lane_value(s.x[MB].y, pl));
        double2 tk = make_double2(0.0, 0.0), scale = make_double2(0.0, 0.0);
        const double s2 = alpha.x * alpha.x + alpha.y * alpha.y + nrm;
        double beta = s2 < kNoReflector ? 0.0 : alpha.x;
        if (s2 >= kNoReflector && (nrm > 0.0 || alpha.y != 0.0)) {
            // with s = |x|: beta = -sign(re alpha) s, tau = (beta - alpha) / beta, and
            // v = x / (alpha - beta)
            const double is = rsqrt_newton(s2), s1 = s2 * is;
            const double sn = fma(fma(-s1, s1, s2), 0.5 * is, s1);
            beta = -copysign(sn, alpha.x);
            const double2 den = make_double2(alpha.x - beta, alpha.y);
            const double ib = -copysign(is, alpha.x), idd = recip(den.x * den.x + den.y * den.y);
            tk = make_double2(-den.x * ib, -alpha.y * ib);
            scale = make_double2(den.x * idd, -den.y * idd);
        }
        double2 vn[NR];
#pragma unroll
        for (int m = MB; m < NR; ++m) {
            const int i = lane + 64 * m;
            vn[m] = cmul2(s.x[m], scale);
            if (m == MB) {
                if (i == kb) vn[m] = make_double2(1.0, 0.0);
                if (i < kb) vn[m] = make_double2(0.0, 0.0);
            }
        }
        // own columns j > k: pending update, then p_j = tau_k sum_i conj(A[i][j]) v_i
        double2 dot[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int j = a.gw + q * a.nwv;
            dot[q] = make_double2(0.0, 0.0);
            if (j > k && j < F) {
                const double2 pj = a.pl[j], vj = a.vl[j];
                // pending rank-2 update A -= v p^H + p v^H + a2r v v^H of column j
                const double2 cvj = make_double2(vj.x, -vj.y);
                const double2 wj = make_double2(fma(s.a2r, cvj.x, pj.x), fma(s.a2r, cvj.y, -pj.y));
#pragma unroll
                for (int m = MB; m < NR; ++m) {
                    const double2 x = sub_mul(sub_mul(s.col[q][m], s.v[m], wj), s.p[m], cvj);
                    s.col[q][m] = x;
                    dot[q] = add_conj_mul(dot[q], x, vn[m]);
                }
            }
        }
        wsum_complex<NC>(dot);
        // every slot set back above is complete before anything of this step is published
        const int n = F - 64 * MB;
        double2 *const ex = a.ex + (k & 1) * 2 * F;
        if constexpr (!kSolo) {
            __builtin_amdgcn_s_waitcnt(0);
            asm volatile("" ::: "memory");
        }
        bool owner = false;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const int j = a.gw + q * a.nwv;
            if (j > k && j < F) {
                if (j == kb) {
                    owner = true;
#pragma unroll
                    for (int m = MB; m < NR; ++m) {
                        const int i = lane + 64 * m;
                        if (i >= kb && i < F) {
                            if constexpr (kSolo) ex[n + i - 64 * MB] = s.col[q][m];
                            else put2(a.cbuf + now + i, s.col[q][m], local);
                        }
                    }
                }
                if (lane == 0) {
                    const double2 pj = cmul2(tk, dot[q]);
                    if constexpr (kSolo) ex[j - 64 * MB] = pj;
                    else put2(a.pbuf + now + j, pj, local);
                }
            }
        }
        // the reflector, by the owner of column k + 1, ahead of the loads below (after them its
        // values would stay in registers across the wait; within 1% either way).  Nothing
        // reads it before the next plane barrier, which waits for it.  (A lambda because the
        // compiler spills three times as much of the five-row form with it written in place.)
        auto store_reflector = [&]() {
            if (!owner) return;
#pragma unroll
            for (int m = MB; m < NR; ++m) {
                const int i = lane + 64 * m;
                if (i >= kb && i < F) put2(a.H + (size_t)k * F + i, vn[m], local);
            }
            if (lane == 0) {
                put(a.d + k, s.diag, local);
                put(a.e + k, beta, local);
                put2(a.tau + k, tk, local);
            }
        };
        store_reflector();
        // a work-group whose columns are done leaves before it reads: every work-group
        // that reads a step publishes in the next one, which is what frees the step's
        // slots (the owner of the last column stays for its diagonal entry)
        if (local && !kSolo && a.last_wg <= kb && kb + 1 < F) {
            return true;
        }
        // all of p and column k + 1, rows from 64 MB on: the work-group's threads load
        // each value once and share it through LDS (every wave loading all of it took
        // more time than the trip through the L2).  Rows that need no value read row
        // F - 1's, which every step publishes.
        if (!local && !plane_barrier(a.flags, a.w, a.W, ++nbar, a.abort_s, a.status, kBarFenced)) return false;
        constexpr int kRounds = (2 * 64 * (NR - MB) + kCoopThreads - 1) / kCoopThreads;
        for (int spins = 0; !kSolo;) {
            bool wait = false;
            asm volatile("" ::: "memory");        // loaded again every time
            double2 got[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int id = threadIdx.x + kCoopThreads * r;
                const int i = 64 * MB + (id < n ? id : id - n);
                const int ii = i >= kb && i < F ? i : F - 1;
                if (local) {
                    constexpr int kAgent = 0x10;       // sc1, agent scope: past the L1
                    const int off = (id < n ? 0 : a.c_off) + ii * (int)sizeof(double2);
                    got[r] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                             rp, off, now * (int)sizeof(double2), kAgent));
                } else {
                    got[r] = ld_c2((id < n ? a.pbuf : a.cbuf) + now + ii);
                }
            }
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                auto is_unset = [](double x) {
                    return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) == kUnsetHi;
                };
                wait |= is_unset(got[r].x) | is_unset(got[r].y);
            }
            if (!local || __ballot(wait) == 0ull) {
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    const int id = threadIdx.x + kCoopThreads * r;
                    if (id < 2 * n) ex[id] = got[r];
                }
                break;
            }
            if (++spins > kMaxPolls) {
                *a.abort_s = 1;
                if (lane == 0) atomicOr(a.status, kStatusBarrier);
                break;
            }
        }
        lds_barrier();
        if (*a.abort_s) return false;
        double2 pv[NR], cv[NR];
#pragma unroll
        for (int m = MB; m < NR; ++m) {
            const int id = min(lane + 64 * (m - MB), n - 1);
            pv[m] = ex[id];
            cv[m] = ex[n + id];
        }
        const double2 pk1 = make_double2(lane_value(pv[MB].x, pl), lane_value(pv[MB].y, pl));
        double2 pvh[1] = {{0.0, 0.0}};
#pragma unroll
        for (int m = MB; m < NR; ++m) {
            const int i = lane + 64 * m;
            s.v[m] = vn[m];
            s.p[m] = i >= kb && i < F ? pv[m] : make_double2(0.0, 0.0);
            pvh[0] = add_conj_mul(pvh[0], s.p[m], vn[m]);
            if (i < F) {
                a.vl[i] = s.v[m];
                a.pl[i] = s.p[m];
            }
        }
        // alpha = -1/2 tau (p^H v); the pending update uses 2 Re(alpha)
        wsum_complex<1>(pvh);
        s.a2r = 2.0 * cmul2(make_double2(-0.5 * tk.x, -0.5 * tk.y), pvh[0]).x;
        const double2 wk = make_double2(pk1.x + s.a2r, -pk1.y);      // v_{k+1} = 1
        s.nrm_part = 0.0;
#pragma unroll
        for (int m = MB; m < NR; ++m) {
            const int i = lane + 64 * m;
            const bool live = i >= kb && i < F;
            const double2 x = sub_mul(make_double2(cv[m].x - s.p[m].x, cv[m].y - s.p[m].y), s.v[m], wk);
            s.x[m] = live ? x : make_double2(0.0, 0.0);
            if (i >= kb + 2) s.nrm_part = fma(s.x[m].x, s.x[m].x, fma(s.x[m].y, s.x[m].y, s.nrm_part));
        }
        s.diag = lane_value(s.x[MB].x, pl);
    }
    if constexpr (MB + 1 < NR) return reduce_steps<NR, NC, MB + 1>(s, a, nbar);
    else return true;
}

template <int NR, int NC>
__global__ __launch_bounds__(kCoopThreads, NR <= 6 ? 2 : 1) void eigen_coop_kernel(EigArgs a)
{
    const int g = blockIdx.x, xcd = g & 7, slot = g >> 3;
    const int W = a.W, F = a.F, c = a.c;
    const int plane = a.plane0 + xcd + 8 * (slot / W), w = slot % W;
    if (plane >= a.planes) return;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    extern __shared__ double2 lds2[];
    __shared__ double red[kCoopWaves];
    __shared__ int abort_s;
    if (t == 0) abort_s = 0;

    const double2 *C = a.C + (size_t)plane * F * F;
    double2 *H = a.H + (size_t)plane * F * F;
    double2 *tau = a.tau + (size_t)plane * F;
    double *d = a.d + (size_t)plane * F, *e = a.e + (size_t)plane * F;
    int *flags = a.bar + (size_t)plane * kBarStride;
    int nbar = 0;

    ReductionArgs ra;
    ra.F = F;
    ra.nwv = W * kCoopWaves;
    ra.gw = w * kCoopWaves + wave;
    ra.lane = lane;
    // the last column of any of the work-group's waves (4 w .. 4 w + 3 modulo 4 W)
    ra.last_wg = -1;
    for (int v = 0; v < kCoopWaves; ++v) {
        const int c0 = w * kCoopWaves + v;
        if (c0 < F) ra.last_wg = max(ra.last_wg, c0 + (F - 1 - c0) / ra.nwv * ra.nwv);
    }
    ra.H = H;
    ra.tau = tau;
    ra.d = d;
    ra.e = e;
    ra.pbuf = a.xbuf + (size_t)plane * 6 * F;
    ra.cbuf = ra.pbuf + 3 * F;
    ra.c_off = 3 * F * (int)sizeof(double2);
    ra.ex = lds2 + (size_t)2 * kCoopWaves * F;
    ra.vl = lds2 + (size_t)2 * wave * F;
    ra.pl = ra.vl + F;
    ra.flags = flags;
    ra.abort_s = &abort_s;
    ra.status = a.status;
    ra.w = w;
    ra.W = W;
    // load own columns and column 0 (A[i][j] = conj(C[j][i]), contiguous in i); check
    // the own ones
    Reduction<NR, NC> s;
    double bad = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        const int j = ra.gw + q * ra.nwv;
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const int i = lane + 64 * m;
            double2 v = make_double2(0.0, 0.0);
            if (j < F && i < F) v = C[(size_t)j * F + i];
            if (!isfinite(v.x) || !isfinite(v.y)) bad = 1.0;
            s.col[q][m] = make_double2(v.x, -v.y);
        }
    }
    s.nrm_part = 0.0;
    s.a2r = 0.0;
#pragma unroll
    for (int m = 0; m < NR; ++m) {
        const int i = lane + 64 * m;
        const double2 v = i < F ? C[i] : make_double2(0.0, 0.0);
        s.x[m] = make_double2(v.x, -v.y);
        s.v[m] = s.p[m] = make_double2(0.0, 0.0);
        if (i >= 2) s.nrm_part += v.x * v.x + v.y * v.y;
        if (i < F) ra.vl[i] = ra.pl[i] = make_double2(0.0, 0.0);
    }
    s.diag = lane_value(s.x[0].x, 0);
    bad = bmax(bad, red);
    if (t == 0) {
        if (bad > 0.0) __hip_atomic_fetch_or(a.flag + plane, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_fetch_or(flags + kPlaceWord, 1 << xcc_id(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // this barrier runs at system scope: the mode is not known yet
    constexpr bool solo = NR == 1;
    if (!plane_barrier(flags, w, W, ++nbar, &abort_s, a.status, solo ? kBarSolo : kBarSystem)) return;
    if (__hip_atomic_load(a.flag + plane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) {
        if (w == 0) {
            double2 *V = a.V + (size_t)plane * F * (c > 0 ? c : 1);
            for (int i = t; i < F * c; i += kCoopThreads) V[i] = make_double2(0.0, 0.0);
            for (int i = t; i < F; i += kCoopThreads) {
                a.lam[(size_t)plane * F + i] = __builtin_nan("");
                if (a.lam_out) a.lam_out[(size_t)plane * F + i] = __builtin_nan("");
            }
            if (t == 0) atomicOr(a.status, kStatusNumeric);
        }
        return;
    }
    const unsigned xccs = (unsigned)__builtin_amdgcn_readfirstlane(
        __hip_atomic_load(flags + kPlaceWord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM));
    const bool local = solo || (!a.agent_scope && __popc(xccs) == 1);
    ra.local = local;
    const BarMode bmode = solo ? kBarSolo : local ? kBarLocal : kBarFenced;
    if (!reduce_steps<NR, NC, 0>(s, ra, nbar)) return;
    // last diagonal entry: column F-1 with the update of step F-2 applied
    if ((F - 1) % ra.nwv == ra.gw && lane == 0) {
        put(d + F - 1, s.diag, local);
        put(e + F - 1, 0.0, local);
        put2(tau + F - 1, make_double2(0.0, 0.0), local);
    }
    if (!plane_barrier(flags, w, W, ++nbar, &abort_s, a.status, bmode)) return;

    // 2. every eigenvalue by multisection on Sturm counts: a group of `pts`
    //    lanes per eigenvalue counts at as many interior points of its bracket, so each
    //    round narrows the bracket (pts + 1)-fold.  The count is the sign
    //    changes of the leading minors' sequence p_i = (d_i - x) p_{i-1} - e_{i-1}^2
    //    p_{i-2}, whose chain is one FMA a row (the quotient form's is a reciprocal
    //    and three); T is scaled by a power of two to a norm near 1 and the sequence
    //    every kScaleRows rows, so that it stays in range.
    double2 *sde = lds2;                          // (d, e^2), scaled
    double *sd = (double *)(sde + F);
    double *se = sd + F;
    double lo_b = 1e300, hi_b = -1e300, emax = 0.0;
    for (int i = t; i < F; i += kCoopThreads) {
        const double di = ld_c(d + i), ei = (i + 1 < F) ? ld_c(e + i) : 0.0;
        const double em = (i > 0) ? ld_c(e + i - 1) : 0.0;
        const double r = fabs(em) + fabs(ei);
        lo_b = fmin(lo_b, di - r);
        hi_b = fmax(hi_b, di + r);
        sd[i] = di;
        se[i] = ei;
        emax = fmax(emax, ei * ei);
    }
    hi_b = bmax(hi_b, red);
    lo_b = -bmax(-lo_b, red);
    emax = bmax(emax, red);
    const double tnorm = fmax(fabs(lo_b), fabs(hi_b));
    const double pivmin = fmax(DBL_MIN, DBL_MIN * emax);
    lo_b -= 2.0 * DBL_EPSILON * tnorm + 2.0 * pivmin;
    hi_b += 2.0 * DBL_EPSILON * tnorm + 2.0 * pivmin;
    const int tex = tnorm > 0.0 ? -ilogb(tnorm) : 0;
    for (int i = t; i < F; i += kCoopThreads) {
        const double es = ldexp(se[i], tex);
        sde[i] = make_double2(ldexp(sd[i], tex), es * es);
    }
    __syncthreads();
    double *lam = a.lam + (size_t)plane * F;
    constexpr int kScaleRows = 8;
    // 16 points, or where four waves would then pass over the eigenvalues twice or more
    // so few that one pass does (20 frames: 17 rounds instead of 2 x 13)
    const int lp = NR > 1 || F <= 16 ? 4 : (F <= 32 ? 3 : 2), pts = 1 << lp, groups = 64 >> lp;
    for (int idx0 = ra.gw * groups; idx0 < F; idx0 += ra.nwv * groups) {
        const int g = lane >> lp, pi = lane & (pts - 1);
        const int idx = idx0 + g;
        const bool mine = idx < F;
        const int target = F - 1 - idx;                   // eigenvalues below this one
        double lo = lo_b, hi = hi_b;
        bool act = mine;
        for (int it = 0; it < 200; ++it) {
            if (act && hi - lo <= 2.0 * DBL_EPSILON * tnorm) act = false;
            if (__ballot(act) == 0ull) break;
            const double x = lo + (hi - lo) * (double)(pi + 1) / (double)(pts + 1);
            const double xs = ldexp(x, tex);
            double p0 = 1.0, p1 = sde[0].x - xs, e2 = sde[0].y;
            int cnt = __double2hiint(p1) < 0;
            auto row = [&](double2 de) {
                const double pn = fma(de.x - xs, p1, -(e2 * p0));
                cnt += (unsigned)(__double2hiint(pn) ^ __double2hiint(p1)) >> 31;
                p0 = p1;
                p1 = pn;
                e2 = de.y;
            };
            int i = 1;
            for (; i + kScaleRows <= F; i += kScaleRows) {
                double2 de[kScaleRows];
#pragma unroll
                for (int r = 0; r < kScaleRows; ++r) de[r] = sde[i + r];
#pragma unroll
                for (int r = 0; r < kScaleRows; ++r) row(de[r]);
                // both zero (x on an eigenvalue of a decoupled block): any sign counts it
                const double big = fmax(fabs(p0), fabs(p1));
                const int ex = -__builtin_amdgcn_frexp_exp(big);
                p0 = __builtin_amdgcn_ldexp(p0, ex);
                p1 = big > 0.0 ? __builtin_amdgcn_ldexp(p1, ex) : copysign(1.0, p1);
            }
            for (; i < F; ++i) row(sde[i]);
            // counts grow with x: the eigenvalue lies between the last point
            // below and the first point above
            const unsigned long long m = __ballot(cnt > target);
            const unsigned bits = (unsigned)((m >> (g * pts)) & ((1ull << pts) - 1ull));
            const int first = bits ? __ffs(bits) - 1 : pts;
            const double nlo = __shfl(x, g * pts + (first > 0 ? first - 1 : 0));
            const double nhi = __shfl(x, g * pts + (first < pts ? first : pts - 1));
            const double lo2 = first > 0 ? nlo : lo, hi2 = first < pts ? nhi : hi;
            if (act && lo2 == lo && hi2 == hi) act = false;
            if (act) {
                lo = lo2;
                hi = hi2;
            }
        }
        if (mine && pi == 0) {
            put(lam + idx, 0.5 * (lo + hi), local);
            if (a.lam_out) a.lam_out[(size_t)plane * F + idx] = 0.5 * (lo + hi);
        }
    }
    if (!plane_barrier(flags, w, W, ++nbar, &abort_s, a.status, bmode)) return;
    if (c <= 0) return;

    // 3. inverse iteration for eigenvector vi of T (the vi-th largest
    //    eigenvalue), one lane of a wave (waves of different work-groups first):
    //    partial-pivoting LU of T - lambda I in LDS, three solves with recurrences carried in registers.
    //    The operands of kRun rows are read together and the next run's ahead of
    //    them, so that a row costs its arithmetic and no LDS latency.
    double *ts = a.tscr + (size_t)plane * c * 6 * F;
    double2 *__restrict__ uu = (double2 *)(se + F) + (size_t)3 * F * wave;   // (u1, u2): above the pivots
    double2 *__restrict__ mi = uu + F;                          // (multiplier, 1 / pivot)
    double *__restrict__ y = (double *)(mi + F);
    int *__restrict__ sw = (int *)(y + F);
    constexpr int kRun = 4;
    for (int vi = wave * W + w; vi < c; vi += ra.nwv) {
        // the start vector, by every lane (the factor and solves below are
        // serial recurrences, run by the first)
        const bool equal = vi > 0 && equal_eigenvalues(ld_c(lam + vi - 1), ld_c(lam + vi), tnorm);
        for (int i = lane; i < F; i += 64) y[i] = start_entry(i, vi, equal);
        __builtin_amdgcn_wave_barrier();
        double inv = 1.0;                // the last solution's scale, applied as it is read
        if (lane == 0) {
            const double lm = iteration_shift(ld_c(lam + vi), tnorm, equal);
            const double tiny = least_pivot(tnorm, pivmin);
            // factor: rows i, i+1 enter step i as (c0, c1 | sub) over (next0, next1);
            // one reciprocal a step, of the pivot
            double c0 = sd[0] - lm, c1 = F > 1 ? se[0] : 0.0;
            double eb[2][kRun + 1], db[2][kRun];
            auto read_t = [&](int b, int i0) {     // rows past the end read the last
#pragma unroll
                for (int u = 0; u <= kRun; ++u) eb[b][u] = se[min(i0 + u, F - 1)];
#pragma unroll
                for (int u = 0; u < kRun; ++u) db[b][u] = sd[min(i0 + u + 1, F - 1)];
            };
            auto factor = [&](int b, int i0, bool whole) {
#pragma unroll
                for (int u = 0; u < kRun; ++u) {
                    const int i = i0 + u;
                    if (whole || i + 1 < F) {
                        const double sub = eb[b][u], n0 = db[b][u] - lm, n1 = eb[b][u + 1];   // e[F-1] = 0
                        const bool swp = !(fabs(c0) >= fabs(sub));
                        if (!swp && c0 == 0.0) c0 = tiny;
                        const double piv = swp ? sub : c0, oth = swp ? c0 : sub;
                        const double r = recip(piv), mul = oth * r;
                        uu[i] = make_double2(swp ? n0 : c1, swp ? n1 : 0.0);
                        mi[i] = make_double2(mul, r);
                        sw[i] = swp;
                        const double d0 = swp ? c1 - mul * n0 : n0 - mul * c1;
                        const double d1 = swp ? -mul * n1 : n1;
                        c0 = d0;
                        c1 = d1;
                    }
                }
            };
            read_t(0, 0);
            int i1 = 0;
            for (; i1 + 2 * kRun < F; i1 += 2 * kRun) {       // whole pairs of runs
                read_t(1, i1 + kRun);
                factor(0, i1, true);
                read_t(0, i1 + 2 * kRun);
                factor(1, i1 + kRun, true);
            }
            read_t(1, i1 + kRun);
            factor(0, i1, false);
            factor(1, i1 + kRun, false);
            if (c0 == 0.0) c0 = tiny;
            const double ilast = recip(c0);
            for (int it = 0; it < 3; ++it) {
                // forward: apply the row swaps and multipliers
                double cur = y[0] * inv;
                double yb[2][kRun], mb[2][kRun];
                int sb[2][kRun];
                auto read_f = [&](int b, int i0) {
#pragma unroll
                    for (int u = 0; u < kRun; ++u) {
                        const int i = min(i0 + u, max(F - 2, 0));
                        yb[b][u] = y[min(i + 1, F - 1)];
                        mb[b][u] = mi[i].x;
                        sb[b][u] = sw[i];
                    }
                };
                auto forward = [&](int b, int i0, bool whole) {
#pragma unroll
                    for (int u = 0; u < kRun; ++u)
                        if (whole || i0 + u + 1 < F) {
                            const double nxt = yb[b][u] * inv;
                            const double top = sb[b][u] ? nxt : cur, bot = sb[b][u] ? cur : nxt;
                            y[i0 + u] = top;
                            cur = fma(-mb[b][u], top, bot);
                        }
                };
                read_f(0, 0);
                for (i1 = 0; i1 + 2 * kRun < F; i1 += 2 * kRun) {
                    read_f(1, i1 + kRun);
                    forward(0, i1, true);
                    read_f(0, i1 + 2 * kRun);
                    forward(1, i1 + kRun, true);
                }
                read_f(1, i1 + kRun);
                forward(0, i1, false);
                forward(1, i1 + kRun, false);
                // back substitution
                double x1 = cur * ilast, x2 = 0.0, n2 = x1 * x1;
                y[F - 1] = x1;
                double2 ub[2][kRun];
                auto read_b = [&](int b, int i0) {          // rows i0, i0 - 1, ..
#pragma unroll
                    for (int u = 0; u < kRun; ++u) {
                        const int i = max(i0 - u, 0);
                        yb[b][u] = y[i];
                        ub[b][u] = uu[i];
                        mb[b][u] = mi[i].y;
                    }
                };
                auto back = [&](int b, int i0, bool whole) {
#pragma unroll
                    for (int u = 0; u < kRun; ++u)
                        if (whole || i0 - u >= 0) {
                            const double xi = fma(-ub[b][u].x, x1, fma(-ub[b][u].y, x2, yb[b][u])) * mb[b][u];
                            y[i0 - u] = xi;
                            n2 = fma(xi, xi, n2);
                            x2 = x1;
                            x1 = xi;
                        }
                };
                read_b(0, F - 2);
                for (i1 = F - 2; i1 >= 2 * kRun; i1 -= 2 * kRun) {
                    read_b(1, i1 - kRun);
                    back(0, i1, true);
                    read_b(0, i1 - 2 * kRun);
                    back(1, i1 - kRun, true);
                }
                read_b(1, i1 - kRun);
                back(0, i1, false);
                back(1, i1 - kRun, false);
                inv = 1.0 / sqrt(n2);
            }
        }
        __builtin_amdgcn_wave_barrier();
        inv = lane_value(inv, 0);
        double *yo = ts + (size_t)vi * 6 * F + 4 * F;
        for (int i = lane; i < F; i += 64) put(yo + i, y[i] * inv, local);
    }
    if (!plane_barrier(flags, w, W, ++nbar, &abort_s, a.status, bmode)) return;

    // 4. work-group 0: classical Gram-Schmidt over the c vectors (staged in LDS),
    //    twice where the first pass cancels, then normalise
    if (w == 0) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        double *Y = se + F;                            // [c][F]
        double *gdot = Y + (size_t)c * F;              // [c]
        for (int i = t; i < c * F; i += kCoopThreads)
            Y[i] = ts[(size_t)(i / F) * 6 * F + 4 * F + (i % F)];
        __syncthreads();
        for (int i = 0; i < c; ++i) {
            double *bi = Y + (size_t)i * F;
            double n2 = 1.0;               // the vectors come in normalised
            for (int pass = 0; pass < 2; ++pass) {
                for (int j = wave; j < i; j += kCoopWaves) {
                    const double *bj = Y + (size_t)j * F;
                    double s = 0.0;
                    for (int q = lane; q < F; q += 64) s += bj[q] * bi[q];
                    s = wsum(s);
                    if (lane == 0) gdot[j] = s;
                }
                __syncthreads();
                n2 = 0.0;
                for (int q = t; q < F; q += kCoopThreads) {
                    double x = bi[q];
                    for (int j = 0; j < i; ++j) x -= gdot[j] * Y[(size_t)j * F + q];
                    bi[q] = x;
                    n2 += x * x;
                }
                n2 = bsum(n2, red);
                // a second pass only where the first took much of the vector away
                if (n2 > 0.5) break;
            }
            const double inv = 1.0 / sqrt(n2);
            for (int q = t; q < F; q += kCoopThreads) bi[q] *= inv;
            __syncthreads();
        }
        for (int i = t; i < c * F; i += kCoopThreads)
            put(ts + (size_t)(i / F) * 6 * F + 4 * F + (i % F), Y[i], local);
    }
    if (!plane_barrier(flags, w, W, ++nbar, &abort_s, a.status, bmode)) return;

    // 5. back-transformation x = H_0 H_1 ... H_{F-2} y: one wave per vector (waves of
    //    different work-groups first), rows as in the reduction.  Two reflectors share
    //    one sum over the lanes: h_b^H (x - tau_a (h_a^H x) h_a) follows from h_a^H x,
    //    h_b^H x and h_b^H h_a.  The rows of the next two pairs are in flight.
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    double2 *V = a.V + (size_t)plane * F * c;
    for (int vi = wave * W + w; vi < c; vi += ra.nwv) {
        const double *y = ts + (size_t)vi * 6 * F + 4 * F;
        double2 x[NR];
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const int q = lane + 64 * m;
            x[m] = make_double2(q < F ? y[q] : 0.0, 0.0);
        }
        constexpr int kPairs = NR <= 6 ? 3 : 2;
        double2 h[kPairs][2][NR], tk[kPairs][2];
        // rows above the pivot, past the last or past step 0 are outside the descriptor
        // and read as zero
        const __amdgpu_buffer_rsrc_t rh =
            __builtin_amdgcn_make_buffer_rsrc(H, 0, F * F * (int)sizeof(double2), 0x00027000);
        auto fetch = [&](int k, double2 (&hr)[NR], double2 &t1) {
            t1 = tau[max(k, 0)];
#pragma unroll
            for (int m = 0; m < NR; ++m) {
                const int q = lane + 64 * m;
                const int off = k >= 0 && q > k && q < F ? q * (int)sizeof(double2) : 0x7ffffff0;
                hr[m] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                        rh, off, max(k, 0) * F * (int)sizeof(double2), 0));
            }
        };
#pragma unroll
        for (int r = 0; r + 1 < kPairs; ++r)
#pragma unroll
            for (int b = 0; b < 2; ++b) fetch(F - 2 - 2 * r - b, h[r][b], tk[r][b]);
        for (int k0 = F - 2; k0 >= 0; k0 -= 2 * kPairs) {
#pragma unroll
            for (int r = 0; r < kPairs; ++r) {
                const int nx = (r + kPairs - 1) % kPairs;
#pragma unroll
                for (int b = 0; b < 2; ++b) fetch(k0 - 2 * (r + kPairs - 1) - b, h[nx][b], tk[nx][b]);
                double2 sum[3] = {{0.0, 0.0}, {0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    sum[0] = add_conj_mul(sum[0], h[r][0][m], x[m]);
                    sum[1] = add_conj_mul(sum[1], h[r][1][m], x[m]);
                    sum[2] = add_conj_mul(sum[2], h[r][1][m], h[r][0][m]);
                }
                wsum_complex<3>(sum);
                const double2 sa = cmul2(tk[r][0], sum[0]), ga = cmul2(sum[2], sa);
                const double2 sb = cmul2(tk[r][1], make_double2(sum[1].x - ga.x, sum[1].y - ga.y));
#pragma unroll
                for (int m = 0; m < NR; ++m) x[m] = sub_mul(sub_mul(x[m], h[r][0][m], sa), h[r][1][m], sb);
            }
        }
#pragma unroll
        for (int m = 0; m < NR; ++m) {
            const int q = lane + 64 * m;
            if (q < F) V[(size_t)q * c + vi] = x[m];
        }
    }
}

size_t eigen_coop_lds(int F, int c) {
    if (F > 64 * kCoopRows) return SIZE_MAX;
    // reduction: v and p of every wave, the values read; tail: d, e, (d, e^2) and either every
    // wave's LU arrays and iterate or the c Gram-Schmidt vectors plus their dots
    const size_t red_b = (size_t)(2 * kCoopWaves + 4) * F * sizeof(double2);
    const size_t tail_b = (4 * (size_t)F + std::max((size_t)6 * kCoopWaves * F, (size_t)c * F + c)) * sizeof(double);
    return std::max(red_b, tail_b) + 64 * sizeof(double);
}

using EigKernel = void (*)(EigArgs);
template <int NR>
static EigKernel eigen_kernel_of(int columns) {
    if constexpr (NR == 1)
        return columns == 5 ? eigen_coop_kernel<1, 5> : (columns == 8 ? eigen_coop_kernel<1, 8> : eigen_coop_kernel<1, 16>);
    else if constexpr (NR > 6) return eigen_coop_kernel<NR, 4>;
    else return columns == 3 ? eigen_coop_kernel<NR, 3>
                             : (columns == 4 ? eigen_coop_kernel<NR, 4> : eigen_coop_kernel<NR, 5>);
}
static EigKernel eigen_kernel(int F, int columns) {
    switch (cdiv(F, 64)) {
        case 1: return eigen_kernel_of<1>(columns);
        case 2: return eigen_kernel_of<2>(columns);
        case 3: return eigen_kernel_of<3>(columns);
        case 4: return eigen_kernel_of<4>(columns);
        case 5: return eigen_kernel_of<5>(columns);
        case 6: return eigen_kernel_of<6>(columns);
        case 7: return eigen_kernel_of<7>(columns);
        case 8: return eigen_kernel_of<8>(columns);
        default: return nullptr;
    }
}

// A cooperative launch needs every work-group resident at once, so the planes
// are solved in groups: as many whole rounds of 8 planes (one per XCD) as fit.
// Columns per wave: all of a small plane's in one work-group; from 385 frames four, which 32
// work-groups hold up to the largest size; else 3 to 5, the fewest of those that need the
// fewest groups at two work-groups a CU, because fewer columns make a step's arithmetic
// shorter and take fewer registers, and more let more planes share an XCD (a third and
// fourth work-group a CU lengthen every step as much as they save: 70 planes of 128 frames
// 1.12 ms with three columns, 1.07 with five).  The filter of 70 planes in ms, by columns 3,
// 4, 5 (* the choice): 300 frames -, 5.90*, 6.35; 321 frames 9.27, 7.08*, 8.31; 352 frames
// 9.97, 10.55, 9.04*; 384 frames (one work-group a CU by LDS) 15.1*, 16.6, 20.3 (with
// registers spilled).  10 planes: 321 frames 1.91*, 2.00, 2.23.
hipError_t launch_eigen_coop(const EigArgs &args, hipStream_t st) {
    const int F = args.F;
    const unsigned lds = (unsigned)eigen_coop_lds(F, args.c);
    if (F > 64 * kCoopRows) return hipErrorInvalidValue;
    if (F <= 64) {      // no work-group waits for another: an ordinary launch
        EigArgs a = args;
        a.W = 1;
        hipLaunchKernelGGL(eigen_kernel(F, F <= 20 ? 5 : (F <= 32 ? 8 : 16)),
                           dim3(8 * cdiv(a.planes - a.plane0, 8)), dim3(kCoopThreads), lds, st, a);
        return hipGetLastError();
    }
    int dev = 0, ncu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    int W = 0, group = 0, launches = 0;
    EigKernel k = nullptr;
    for (int columns = F > 384 ? 4 : 3; columns <= (F > 384 ? 4 : 5); ++columns) {
        const int w = cdiv(F, kCoopWaves * columns);
        const EigKernel kc = eigen_kernel(F, columns);
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kc, kCoopThreads, lds);
        if (e != hipSuccess) return e;
        // whole rounds of 8 planes, of two work-groups a CU for the choice
        const int fit = std::min(per_cu, 2) * ncu / (8 * w) * 8;
        if (fit == 0 || (k && cdiv(args.planes, fit) >= launches)) continue;
        launches = cdiv(args.planes, fit);
        W = w;
        group = per_cu * ncu / (8 * w) * 8;
        k = kc;
        if (launches == 1) break;
    }
    if (!k) return hipErrorCooperativeLaunchTooLarge;
    for (int p0 = 0; p0 < args.planes; p0 += group) {
        EigArgs a = args;
        a.W = W;
        a.plane0 = p0;
        a.planes = std::min(args.planes, p0 + group);        // planes [p0, a.planes)
        const int n = a.planes - p0;
        dim3 grid(8 * cdiv(n, 8) * W), block(kCoopThreads);
        void *params[] = {&a};
        e = hipLaunchCooperativeKernel((const void *)k, grid, block, params, lds, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Exchange slots, barrier flags, per-plane flags and the status word before a solve.
__global__ void eigen_clear_kernel(int *status, int *bar, int *eflag, double2 *xbuf, int planes, int F)
{
    const int i0 = blockIdx.x * blockDim.x + threadIdx.x, n = gridDim.x * blockDim.x;
    if (i0 == 0) *status = 0;
    for (int i = i0; i < planes * kBarStride; i += n) bar[i] = 0;
    for (int i = i0; i < planes; i += n) eflag[i] = 0;
    for (int i = i0; i < planes * 6 * F; i += n) xbuf[i] = unset2();
}

hipError_t launch_eigen_clear(int *status, int *bar, int *eflag, double2 *xbuf, int planes, int F,
                              hipStream_t st) {
    const int wgs = std::min(64, cdiv(planes * 6 * F, 256));
    hipLaunchKernelGGL(eigen_clear_kernel, dim3(wgs), dim3(256), 0, st, status, bar, eflag, xbuf, planes, F);
    return hipGetLastError();
}

}  // namespace ulm

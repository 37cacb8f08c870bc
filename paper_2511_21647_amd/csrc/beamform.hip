// Stage 2 of the two-stage row-column beamforming (paper Section II-A1, and
// the sub-block sum projection of Section II-A4): extrapolation along the
// transmit direction, coherent compounding and slab projection collapse into
// one complex axial FIR per (transmit, slab):
//   P(u, z) = sum_k sum_d H_k[d] S_k(u, z + d).
#include "common.h"

#include <stdint.h>

namespace ulm {

// G slabs per work-group: for each transmit the slice tile covers the union of
// the G slabs' tap ranges and is read from HBM once for all of them.
template <int G>
__global__ __launch_bounds__(256, 4) void stage2_fir_kernel(
    const float2 *__restrict__ S, float2 *__restrict__ P, const float2 *__restrict__ taps,
    const int2 *__restrict__ meta, Geometry g, int max_taps)
{
    // logical work-group order ((o F + f) tiles + tile) NG + slab group: the slab
    // groups of one tile and frame run back to back on one XCD and share its L2
    // copy of the slice tiles
    const int NG = cdiv(g.n_blocks, G);
    const int n_tu = cdiv(g.nu, kFirTileU), tiles = n_tu * cdiv(g.nz, kFirTileZ);
    const int n_wg = 2 * g.n_frames * tiles * NG;
    int lw = xcd_remap(blockIdx.x, n_wg);
    const int b0 = (lw % NG) * G;
    lw /= NG;
    const int ti = lw % tiles;
    lw /= tiles;
    const int f = lw % g.n_frames, o = lw / g.n_frames;
    const int tu = ti % n_tu, tz = ti / n_tu;
    const int c = threadIdx.x % kFirTileU;
    const int rg = threadIdx.x / kFirTileU;          // 8 groups of 8 rows
    const int u = tu * kFirTileU + c;
    const int l0 = tz * kFirTileZ;
    const size_t plane = (size_t)g.nz * g.nu;

    __shared__ float2 tile[kFirTileZ + kFirMaxTaps][kFirTileU];
    float2 acc[G][8];
#pragma unroll
    for (int gb = 0; gb < G; ++gb)
#pragma unroll
        for (int r = 0; r < 8; ++r) acc[gb][r] = make_float2(0.f, 0.f);

    // union of the group's tap offsets for transmit k: [lo, hi)
    auto span_of = [&](int k, int &lo, int &hi) {
        lo = INT32_MAX;
        hi = INT32_MIN;
#pragma unroll
        for (int gb = 0; gb < G; ++gb)
            if (b0 + gb < g.n_blocks) {
                const int2 m = meta[k * g.n_blocks + b0 + gb];
                lo = min(lo, m.x);
                hi = max(hi, m.x + m.y);
            }
    };
    // the slice tile of transmit k (rows l0 + lo .. , one row past the last tap
    // of each window): element e = t + 256 i of the tile goes through pre[i]
    constexpr int kPer = ((kFirTileZ + kFirMaxTaps) * kFirTileU + 255) / 256;
    float2 pre[kPer];
    auto fetch = [&](int k, int lo, int rows) {
        const float2 *src = S + ((size_t)(o * g.n_angles + k) * g.n_frames + f) * plane;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = threadIdx.x + 256 * i;
            const int rr = e / kFirTileU, cc = e % kFirTileU;
            const int zz = l0 + lo + rr, uu = tu * kFirTileU + cc;
            pre[i] = make_float2(0.f, 0.f);
            if (rr < rows && zz >= 0 && zz < g.nz && uu < g.nu) pre[i] = src[(size_t)zz * g.nu + uu];
        }
    };
    auto stash = [&](int rows) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = threadIdx.x + 256 * i;
            if (e < rows * kFirTileU) tile[e / kFirTileU][e % kFirTileU] = pre[i];
        }
    };
    auto filter = [&](int k, int lo_k) {
#pragma unroll
        for (int gb = 0; gb < G; ++gb) {
            if (b0 + gb >= g.n_blocks) continue;
            const int2 m = meta[k * g.n_blocks + b0 + gb];
            // 8 consecutive output rows per thread: a rotating window of 8 input rows
            // in registers, so each tap costs one LDS read instead of eight
            const float2 *h = taps + (size_t)(k * g.n_blocks + b0 + gb) * max_taps;
            const int base = rg * 8 + (m.x - lo_k);
            float2 win[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) win[r] = tile[base + r][c];
            auto step = [&](int tt, int uu) {   // tap tt = 8 q + uu
                const float2 hv = h[tt];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float2 x = win[(r + uu) & 7];
                    acc[gb][r].x = fmaf(hv.x, x.x, fmaf(-hv.y, x.y, acc[gb][r].x));
                    acc[gb][r].y = fmaf(hv.x, x.y, fmaf(hv.y, x.x, acc[gb][r].y));
                }
                win[uu] = tile[base + 8 + tt][c];     // row base + tt is no longer needed
            };
            int tt = 0;
            for (; tt + 8 <= m.y; tt += 8) {
#pragma unroll
                for (int uu = 0; uu < 8; ++uu) step(tt + uu, uu);
            }
#pragma unroll
            for (int uu = 0; uu < 8; ++uu)
                if (tt + uu < m.y) step(tt + uu, uu);
        }
    };
    int lo, hi;
    if constexpr (G == 1) {
        // one slab: the next transmit's tile is loaded while this one is filtered
        span_of(0, lo, hi);
        fetch(0, lo, kFirTileZ + (hi - lo));
        for (int k = 0; k < g.n_angles; ++k) {
            stash(kFirTileZ + (hi - lo));
            __syncthreads();
            const int lo_k = lo;
            if (k + 1 < g.n_angles) {
                span_of(k + 1, lo, hi);
                fetch(k + 1, lo, kFirTileZ + (hi - lo));
            }
            filter(k, lo_k);
            __syncthreads();
        }
    } else {
        // G slabs hold G x 8 accumulators: no registers to spare for a prefetch
        for (int k = 0; k < g.n_angles; ++k) {
            span_of(k, lo, hi);
            const int rows = kFirTileZ + (hi - lo);
            const float2 *src = S + ((size_t)(o * g.n_angles + k) * g.n_frames + f) * plane;
            for (int e = threadIdx.x; e < rows * kFirTileU; e += blockDim.x) {
                const int rr = e / kFirTileU, cc = e % kFirTileU;
                const int zz = l0 + lo + rr, uu = tu * kFirTileU + cc;
                float2 v = make_float2(0.f, 0.f);
                if (zz >= 0 && zz < g.nz && uu < g.nu) v = src[(size_t)zz * g.nu + uu];
                tile[rr][cc] = v;
            }
            __syncthreads();
            filter(k, lo);
            __syncthreads();
        }
    }
    if (u >= g.nu) return;
#pragma unroll
    for (int gb = 0; gb < G; ++gb) {
        if (b0 + gb >= g.n_blocks) continue;
        float2 *dst = P + ((size_t)(o * g.n_blocks + b0 + gb) * g.n_frames + f) * plane;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int l = l0 + rg * 8 + r;
            if (l < g.nz) dst[(size_t)l * g.nu + u] = acc[gb][r];
        }
    }
}

// Many narrow slabs (kSlabGroup per work-group, at most kSlabMaxTaps taps each, the
// paper's slabs of 8 slices): the same sums in the same order, with the tap loops
// unrolled.  A slab of few taps leaves little arithmetic per fixed cost, which bounded
// the form above (one scalar load and one loop step per tap: 12.4 ms for 2 x 35 slabs
// of 250 x 274 x 300).  Here a (transmit, slab) costs two LDS reads for its taps
// (staged once per work-group) and eleven reads of the slice tile for 8 x taps x 4
// FMAs; the next transmit's tile is in flight during it.  The planes, which nothing
// reads soon, are stored past the caches where their rows are whole 64-byte pieces, the
// least that memory takes at once (114 x 136 planes, 4 transmits 95 -> 76 us; 250 x 272, 2
// transmits 237 -> 160), or the stores come slowly, with more than four transmits (250 x 274,
// 9 transmits, 20 frames 520 -> 503 us).  Otherwise smaller parts would reach memory one by
// one, which the L2 joins (250 x 274, one transmit 357 -> 254 us, four 369 -> 350; over 149
// sizes of 1, 2, 3 and 4 transmits 0.70, 0.89, 0.91 and 0.95 of the time, at worst 1.17).
// Lines a work-group fills stored past the caches and the rest through them lose to the
// better of the two by up to 26%.  6.1 ms: 4.6 without the stores
// of 11.5 GB, about 3.5 of FMAs alone.  Groups of 5 to 12 slabs with 4 or 8 rows per thread and 3 to
// 6 waves per SIMD all take 6.1-7.2 ms.
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Taps are added in order, each under a uniform branch, so that the accumulators stay
// where they are (one body per tap count makes the compiler copy them).
template <int R>
__device__ inline void slab_taps(const float2 (*tile)[kFirTileU], const float2 *h, int n, int base,
                                 int c, float2 (&acc)[R])
{
    float2 x[R + kSlabMaxTaps - 1], hv[kSlabMaxTaps];
#pragma unroll
    for (int i = 0; i < kSlabMaxTaps; ++i) hv[i] = h[i];
#pragma unroll
    for (int i = 0; i < R + kSlabMaxTaps - 1; ++i) x[i] = tile[base + i][c];
#pragma unroll
    for (int i = 0; i < kSlabMaxTaps; ++i)
        if (i == 0 || i < n) {       // a slab has a tap
#pragma unroll
            for (int r = 0; r < R; ++r) {
                acc[r].x = fmaf(hv[i].x, x[r + i].x, fmaf(-hv[i].y, x[r + i].y, acc[r].x));
                acc[r].y = fmaf(hv[i].x, x[r + i].y, fmaf(hv[i].y, x[r + i].x, acc[r].y));
            }
#pragma unroll
            for (int r = 0; r < R; ++r) asm volatile("" : "+v"(acc[r].x), "+v"(acc[r].y));
        }
}

// SPAN: halo rows (the union of the group's tap ranges fits); PAST: stores past the caches
template <int SPAN, bool PAST>
__global__ __launch_bounds__(256, 3) void stage2_slab_kernel(
    const float2 *__restrict__ S, float2 *__restrict__ P, const float2 *__restrict__ taps,
    const int2 *__restrict__ meta, Geometry g, int max_taps)
{
    constexpr int G = kSlabGroup, R = kSlabRows;
    constexpr int kTile = 8 * R, kRows = kTile + SPAN;
    // work-group order as stage2_fir_kernel
    const int NG = cdiv(g.n_blocks, G);
    const int n_tu = cdiv(g.nu, kFirTileU), tiles = n_tu * cdiv(g.nz, kTile);
    const int n_wg = 2 * g.n_frames * tiles * NG;
    int lw = xcd_remap(blockIdx.x, n_wg);
    const int b0 = (lw % NG) * G;
    lw /= NG;
    const int ti = lw % tiles;
    lw /= tiles;
    const int f = lw % g.n_frames, o = lw / g.n_frames;
    const int tu = ti % n_tu, tz = ti / n_tu;
    const int t = threadIdx.x, c = t % kFirTileU, rg = t / kFirTileU;
    const int u = tu * kFirTileU + c;
    const int l0 = tz * kTile;
    const size_t plane = (size_t)g.nz * g.nu;

    // the last rows are read but meet no tap
    __shared__ float2 tile[kRows + kSlabMaxTaps - 1][kFirTileU];
    __shared__ __attribute__((aligned(16))) float2 hs[ULM_MAX_ANGLES][G][kSlabMaxTaps];
    for (int e = t; e < g.n_angles * G * kSlabMaxTaps; e += 256) {
        const int q = e % kSlabMaxTaps, gb = (e / kSlabMaxTaps) % G, k = e / (kSlabMaxTaps * G);
        hs[k][gb][q] = q < max_taps && b0 + gb < g.n_blocks
                           ? taps[(size_t)(k * g.n_blocks + b0 + gb) * max_taps + q] : make_float2(0.f, 0.f);
    }
    // per transmit: the first row of the tile, and each slab's first row within it and
    // tap count (none for a slab past the last), in LDS: a chain of scalar loads of
    // them ahead of the tile's loads cost as much as the arithmetic
    __shared__ int lo_s[ULM_MAX_ANGLES], slab_s[ULM_MAX_ANGLES][G];
    if (t < g.n_angles) {
        int lo = INT32_MAX;
        for (int gb = 0; gb < G && b0 + gb < g.n_blocks; ++gb) lo = min(lo, meta[t * g.n_blocks + b0 + gb].x);
        for (int gb = 0; gb < G; ++gb) {
            const int2 m = meta[t * g.n_blocks + min(b0 + gb, g.n_blocks - 1)];
            slab_s[t][gb] = b0 + gb < g.n_blocks ? (m.x - lo) * 8 + m.y : 0;
        }
        lo_s[t] = lo;
    }
    __syncthreads();
    float2 acc[G][R];
#pragma unroll
    for (int gb = 0; gb < G; ++gb)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[gb][r] = make_float2(0.f, 0.f);

    // thread t moves column t % 32 of the tile's rows t / 32 + 8 i
    constexpr int kPer = kRows / 8;
    float2 pre[kPer];
    const int uc = min(u, g.nu - 1);
    auto fetch = [&](int k, int lo) {
        const float2 *src = S + ((size_t)(o * g.n_angles + k) * g.n_frames + f) * plane + uc;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int zz = l0 + lo + rg + 8 * i;
            pre[i] = src[(size_t)min(max(zz, 0), g.nz - 1) * g.nu];
        }
    };
    int lo = __builtin_amdgcn_readfirstlane(lo_s[0]);
    fetch(0, lo);
    for (int k = 0; k < g.n_angles; ++k) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            // rows outside the plane are zeros (set here, so that nothing waits on the
            // loads before the previous transmit is done)
            const bool in = (unsigned)(l0 + lo + rg + 8 * i) < (unsigned)g.nz;
            tile[rg + 8 * i][c] = make_float2(in ? pre[i].x : 0.f, in ? pre[i].y : 0.f);
        }
        __syncthreads();
        const int kn = min(k + 1, g.n_angles - 1);
        lo = __builtin_amdgcn_readfirstlane(lo_s[kn]);
        fetch(kn, lo);
        int slab[G];
#pragma unroll
        for (int gb = 0; gb < G; ++gb) slab[gb] = __builtin_amdgcn_readfirstlane(slab_s[k][gb]);
#pragma unroll
        for (int gb = 0; gb < G; ++gb) {
            const int base = rg * R + (slab[gb] >> 3);
            slab_taps<R>(tile, hs[k][gb], slab[gb] & 7, base, c, acc[gb]);
        }
        __syncthreads();
    }
    if (u >= g.nu) return;
#pragma unroll
    for (int gb = 0; gb < G; ++gb) {
        if (b0 + gb >= g.n_blocks) continue;
        float2 *dst = P + ((size_t)(o * g.n_blocks + b0 + gb) * g.n_frames + f) * plane;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int l = l0 + rg * R + r;
            if (l >= g.nz) continue;
            float2 *at = &dst[(size_t)l * g.nu + u];
            if constexpr (PAST)
                __builtin_nontemporal_store(f32x2{acc[gb][r].x, acc[gb][r].y}, reinterpret_cast<f32x2 *>(at));
            else
                *at = acc[gb][r];
        }
    }
}

hipError_t launch_stage2(const ulm_ctx *ctx, const float2 *slices, float2 *proj, hipStream_t st)
{
    const Geometry &g = ctx->geo;
    const int G = ctx->tab.fir_group;
    const size_t n_wg = (size_t)2 * g.n_frames * cdiv(g.nu, kFirTileU) * cdiv(g.nz, G == kSlabGroup ? 8 * kSlabRows : kFirTileZ) *
                        cdiv(g.n_blocks, G);
    if (n_wg > (size_t)INT32_MAX) return hipErrorInvalidConfiguration;
    if (G == kSlabGroup) {
        const bool narrow = ctx->tab.fir_span <= kSlabSpan, past = g.nu % 8 == 0 || g.n_angles > 4;
        hipLaunchKernelGGL(narrow ? (past ? stage2_slab_kernel<kSlabSpan, true> : stage2_slab_kernel<kSlabSpan, false>)
                                  : (past ? stage2_slab_kernel<kSlabMaxSpan, true>
                                          : stage2_slab_kernel<kSlabMaxSpan, false>),
                           dim3((unsigned)n_wg), dim3(256), 0, st, slices, proj, ctx->tab.taps,
                           ctx->tab.tap_meta, g, ctx->tab.n_taps);
    } else if (G == kFirGroup)
        hipLaunchKernelGGL(stage2_fir_kernel<kFirGroup>, dim3((unsigned)n_wg), dim3(256), 0, st,
                           slices, proj, ctx->tab.taps, ctx->tab.tap_meta, g, ctx->tab.n_taps);
    else
        hipLaunchKernelGGL(stage2_fir_kernel<1>, dim3((unsigned)n_wg), dim3(256), 0, st, slices,
                           proj, ctx->tab.taps, ctx->tab.tap_meta, g, ctx->tab.n_taps);
    return hipGetLastError();
}

}  // namespace ulm

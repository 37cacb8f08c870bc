// NCC microbubble localisation (paper Section II-A4) on filtered planes.
//
//   ncc_stream_kernel  one work-group per band of rows x full width: streams the
//                      band's rows once, eight NCC rows at a time (two separable
//                      passes, Fig. 1g, of three sums: template, box, box of
//                      squares), finds the 3x3 regional maxima at or above the
//                      NCC threshold in raster order, and the band's envelope
//                      maximum
//   ncc_count_kernel   per image: the frame maximum from its bands', and how many
//                      of each band's maxima reach the intensity threshold
//   loc_scan_kernel    exclusive scan of the per-image counts
//   ncc_write_kernel   sub-pixel fit of the records that reach it, at their
//                      offset in the output
//   frame_max_kernel   per-(plane, frame) maximum of the envelope |P| (the learned
//                      localiser's input scale)
//   loc_scatter_kernel copies the learned localiser's rows to their output offset
// Output order is (plane, frame, row, column) without any sort: bands are full
// width and are laid out in that order.
#include "common.h"
#include "roots.h"

#include <float.h>
#include <math.h>

namespace ulm {

struct NccParams {
    int half;             // template half width h
    float kbar;           // mean of the template
    float inv_w;          // 1 / size^2
    float inv_sk;         // 1 / sqrt(sum (K - Kbar)^2)
    float tau, alpha;
    float gz[kNccMaxHalf + 1], gu[kNccMaxHalf + 1];   // first half of the taps, centre last
};

__global__ __launch_bounds__(256) void frame_max_kernel(const float2 *__restrict__ P,
                                                        float *__restrict__ fmax_out, int npix)
{
    const float2 *src = P + (size_t)blockIdx.x * npix;
    float m = 0.f;
    // eight loads in flight per thread (the launch is one work-group per image)
    int i = threadIdx.x;
    for (; i + 7 * 256 < npix; i += 8 * 256) {
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[i + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, sqrtf(v[u].x * v[u].x + v[u].y * v[u].y));
    }
    for (; i < npix; i += 256) {
        const float2 v = src[i];
        m = fmaxf(m, sqrtf(v.x * v.x + v.y * v.y));
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    __shared__ float red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) fmax_out[blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__device__ inline float subpix(float nm, float n0, float np) {
    float d;
    if (nm > 0.f && n0 > 0.f && np > 0.f) {
        const float lm = logf(nm), l0 = logf(n0), lp = logf(np);
        const float den = 2.f * (lm - 2.f * l0 + lp);
        d = den < 0.f ? (lm - lp) / den : 0.f;
    } else {
        const float den = 2.f * (nm - 2.f * n0 + np);
        d = den < 0.f ? (nm - np) / den : 0.f;
    }
    return fminf(fmaxf(d, -0.5f), 0.5f);
}

// |P| with the rounding sequence that every step of the localiser shares (re^2
// fused onto the rounded im^2), so the intensity of a record, the frame maximum
// and the NCC windows see the same value.
__device__ inline float ncc_mag2(float2 v) { return fmaf(v.x, v.x, v.y * v.y); }
__device__ inline float ncc_mag(float2 v) { return sqrtf(ncc_mag2(v)); }

// A regional maximum as ncc_stream_kernel stages it (the size of a record): the
// NCC there and at the four neighbours that the sub-pixel fit reads.
struct NccPeak {
    int iz, iu;
    float up, dn, left, right, n0;
    float intensity;      // written by ncc_count_kernel
};
static_assert(sizeof(NccPeak) == sizeof(ulm_loc_t), "staged in the records' slots");

// One work-group: one band of band_rows rows (8 m - 2) of one image, full width.
// The image is read once, from the band's first input row down; eight NCC rows
// form a batch:
//   V: thread t owns input column t and slides the three vertical sums down it
//      (the window of 8 + 2H envelope values in registers, the next batch's eight
//      rows in flight during this one), into LDS;
//   H: thread (row, group of 8 columns) forms the NCC of eight neighbouring
//      pixels from 8 + 2H sums of each kind, read as 16-byte vectors and used
//      from registers (4 + H bytes of LDS read per kind of sum and pixel instead of
//      4 (2H + 1): 8 instead of 36 for 9 x 9);
//   peaks: thread (row, group) tests its eight pixels of the rows whose lower
//      neighbour is known; offsets in raster order from ballots.
// Bound by VALU issue: the two passes are 6 (2H + 1) sums a pixel, plus the
// correctly rounded root of every value read.  The batch shape keeps both passes
// at one work item per thread for any width (8 rows x ceil((nu + 2) / 8) groups
// need no more threads than the columns do) with three barriers per eight rows;
// a band taller than 16 rows reads and roots fewer halo rows.  The intensity
// threshold needs the whole image's maximum, so it is applied afterwards to the
// few maxima (ncc_count_kernel) and the planes are not read a first time for it.
constexpr int kNccBatch = 8;
constexpr int kNccMaxThreads = 576;      // widest plane accepted: 553 input columns

// LDS of the batch: row strides of the vertical sums and of the NCC rows
__host__ __device__ inline int ncc_groups(int nu) { return (nu + 2 + 7) / 8; }
__host__ __device__ inline int ncc_vstride(int nu, int h) { return 8 * ncc_groups(nu) + (2 * h + 7) / 8 * 8; }
__host__ __device__ inline int ncc_nstride(int nu) { return 8 * ncc_groups(nu) + 4; }

// Five waves a SIMD where the registers nearly allow it: up to 7 x 7 they do, and 9 x 9 is
// worth three spilled ones (600 images of 250 x 274 220 us, with four waves and none spilled
// 272; 21,000 images 8.1 and 9.9 ms with the pairing).  From 11 x 11 four.
template <int H>
__global__ __launch_bounds__(kNccMaxThreads, H <= 4 ? 5 : 4) void ncc_stream_kernel(
    const float2 *__restrict__ P, float *__restrict__ band_max, NccPeak *__restrict__ staged,
    int *__restrict__ band_cnt, NccParams prm, int nz, int nu, int bands, int band_rows,
    int band_cap)
{
    constexpr int S = 2 * H + 1;
    constexpr int NW = kNccBatch + 2 * H;           // envelope rows of a batch
    constexpr int NV = (8 + 2 * H + 3) / 4;         // 16-byte vectors per item and kind of sum
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int G8 = ncc_groups(nu), VS = ncc_vstride(nu, H), NS = ncc_nstride(nu);
    float *V = smem;                                // [3][8][VS]
    float *ncc = smem + 3 * kNccBatch * VS;         // [2 carried rows + 8][NS]
    __shared__ int wave_tot[2][kNccMaxThreads / 64];
    __shared__ float wave_max[kNccMaxThreads / 64];

    // the bands of an image run on one XCD: its L2 serves the halo rows
    const int slot = xcd_remap(blockIdx.x, gridDim.x);
    const int band = slot % bands, img = slot / bands;
    const int r0 = band * band_rows, r1 = min(r0 + band_rows, nz);
    const int n_batch = (r1 - r0 + 2 + kNccBatch - 1) / kNccBatch;
    const float2 *src = P + (size_t)img * nz * nu;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, nw = blockDim.x >> 6;

    // V: this thread's column; its slot in a row of sums swaps neighbouring
    // 16-byte vectors in every other run of eight, so that the items' reads at a
    // stride of two vectors fall on distinct banks
    const int u = t - 1 - H, uc = min(max(u, 0), nu - 1);
    const bool cu = u >= 0 && u < nu;
    const bool vok = t < VS;
    float *const vdst = V + (((t >> 2) ^ ((t >> 5) & 1)) << 2) + (t & 3);
    // H and peaks: this thread's item
    const int ir = t / G8, ig = t - ir * G8;
    const bool item = ir < kNccBatch;
    int voff[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int vec = 2 * ig + q;
        voff[q] = (item ? ir * VS : 0) + ((vec ^ ((vec >> 3) & 1)) << 2);
    }

    const unsigned ubytes = (unsigned)uc * sizeof(float2);
    const unsigned cmask = cu ? ~0u : 0u;
    // rows are loaded through a buffer descriptor on the band's first row: a scalar
    // row offset plus the column's, no address arithmetic per lane
    const int zt = r0 - 1 - H, zf = max(zt, 0);     // first envelope row of the band
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(src + (size_t)zf * nu), 0, (int)((size_t)min(nz - zf, band_rows + 2 * H + 24) * nu * sizeof(float2)),
        0x00027000);
    auto load = [&](int z) {
        const int row = (min(max(z, 0), min(nz, zf + band_rows + 2 * H + 24) - 1) - zf) * nu * (int)sizeof(float2);
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)ubytes, row, 0);
        return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
    };
    // envelopes of N rows from z on, zero outside the image; m: their maximum
    float m = 0.f;
    auto envelope = [&](const auto &raw, int z, float *dst) {
        constexpr int N = sizeof(raw) / sizeof(float2);
        float x[N], r[N];
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = ncc_mag2(raw[i]);
        exact_roots<N>(x, r);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const unsigned zmask = (unsigned)(z + i) < (unsigned)nz ? ~0u : 0u;     // uniform
            dst[i] = __uint_as_float(__float_as_uint(r[i]) & (cmask & zmask));
            m = fmaxf(m, dst[i]);
        }
    };
    float col[NW];
    float2 nx[kNccBatch];
    {
        float2 raw[NW];
#pragma unroll
        for (int i = 0; i < NW; ++i) raw[i] = load(zt + i);
#pragma unroll
        for (int i = 0; i < kNccBatch; ++i) nx[i] = load(zt + NW + i);
        envelope(raw, zt, col);
    }
    NccPeak *out = staged + (size_t)slot * band_cap;
    int total = 0;
    float res[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) res[c] = 0.f;

    for (int j = 0; j < n_batch; ++j) {
        const int zb = r0 - 1 + kNccBatch * j;      // first NCC row of the batch
        if (vok) {
#pragma unroll
            for (int i = 0; i < kNccBatch; ++i) {
                // the template's taps are symmetric: H + 1 values
                float sg = prm.gz[0] * col[i], s1 = col[i], s2 = col[i] * col[i];
#pragma unroll
                for (int a = 1; a < S; ++a) {
                    const float x = col[i + a];
                    sg = fmaf(prm.gz[a <= H ? a : S - 1 - a], x, sg);
                    s1 += x;
                    s2 = fmaf(x, x, s2);
                }
                vdst[i * VS] = sg;
                vdst[(kNccBatch + i) * VS] = s1;
                vdst[(2 * kNccBatch + i) * VS] = s2;
            }
        }
        __syncthreads();
        if (j + 1 < n_batch) {
#pragma unroll
            for (int i = 0; i < 2 * H; ++i) col[i] = col[i + kNccBatch];
            const int z = zt + NW + kNccBatch * j;
            envelope(nx, z, col + 2 * H);
#pragma unroll
            for (int i = 0; i < kNccBatch; ++i) nx[i] = load(z + kNccBatch + i);
        }
        if (item) {
            // the previous batch's last two rows become the carried rows
            if (ir >= kNccBatch - 2) {
                float4 *d = reinterpret_cast<float4 *>(ncc + (ir - (kNccBatch - 2)) * NS + 8 * ig);
                d[0] = make_float4(res[0], res[1], res[2], res[3]);
                d[1] = make_float4(res[4], res[5], res[6], res[7]);
            }
            float sums[3][8];
#pragma unroll
            for (int kind = 0; kind < 3; ++kind) {
                float v[4 * NV];
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    *reinterpret_cast<float4 *>(&v[4 * q]) =
                        *reinterpret_cast<const float4 *>(V + kind * kNccBatch * VS + voff[q]);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    float s = kind == 0 ? prm.gu[0] * v[c] : v[c];
#pragma unroll
                    for (int b = 1; b < S; ++b) 
                        s = kind == 0 ? fmaf(prm.gu[b <= H ? b : S - 1 - b], v[c + b], s) : s + v[c + b];
                    sums[kind][c] = s;
                }
            }
            float num[8], var[8], low = FLT_MAX;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                num[c] = fmaf(-prm.kbar, sums[1][c], sums[0][c]) * prm.inv_sk;
                var[c] = fmaf(-(sums[1][c] * sums[1][c]), prm.inv_w, sums[2][c]);
                low = fminf(low, var[c]);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) res[c] = num[c] * __builtin_amdgcn_rsqf(var[c]);
            // rsqrtf is the hardware's reciprocal root but for denormals, which it scales
            if (__ballot(low < FLT_MIN)) {
#pragma unroll
                for (int c = 0; c < 8; ++c) res[c] = num[c] * rsqrtf(var[c]);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) res[c] = var[c] > 1e-6f * sums[2][c] ? res[c] : 0.f;
            // outside the image: ignored by the peak test
            if ((unsigned)(zb + ir) >= (unsigned)nz) {
#pragma unroll
                for (int c = 0; c < 8; ++c) res[c] = -INFINITY;
            }
            if (ig == 0) res[0] = -INFINITY;
            if (8 * ig + 7 > nu) {
#pragma unroll
                for (int c = 0; c < 8; ++c) res[c] = 8 * ig + c > nu ? -INFINITY : res[c];
            }
            float4 *d = reinterpret_cast<float4 *>(ncc + (2 + ir) * NS + 8 * ig);
            d[0] = make_float4(res[0], res[1], res[2], res[3]);
            d[1] = make_float4(res[4], res[5], res[6], res[7]);
        }
        __syncthreads();
        // peaks of NCC rows zb - 1 .. zb + 6 (LDS rows 1 .. 8): at or above the
        // threshold, 3x3 regional maximum (raster tie-break)
        unsigned bits = 0;
        const int zp = zb - 1 + ir;
        const float *row = ncc + (1 + ir) * NS + 8 * ig;
        if (item && zp >= r0 && zp < r1) {
            const float4 a = reinterpret_cast<const float4 *>(row)[0];
            const float4 b = reinterpret_cast<const float4 *>(row)[1];
            const float n8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int c = 0; c < 8; ++c) bits |= n8[c] >= prm.tau ? 1u << c : 0u;
            if (ig == 0) bits &= ~1u;                            // columns -1 and nu
            const int over = 8 * ig + 8 - (nu + 1);
            if (over > 0) bits &= over < 8 ? 0xffu >> over : 0u;
        }
        unsigned todo = bits;
        bits = 0;
        while (todo) {
            const int c = __ffs((int)todo) - 1;
            todo &= todo - 1;
            const float *mid = row + c, *up = mid - NS, *dn = mid + NS;
            const float n0 = mid[0];
            if (n0 > up[-1] && n0 > up[0] && n0 > up[1] && n0 > mid[-1] && n0 >= mid[1] &&
                n0 >= dn[-1] && n0 >= dn[0] && n0 >= dn[1])
                bits |= 1u << c;
        }
        // offsets: at most four maxima among eight neighbours, so three ballots
        // give the wave's prefix sums
        const int cnt = __popc(bits);
        int off = 0, wt = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const unsigned long long bal = __ballot((cnt >> k) & 1);
            off += __popcll(bal & ((1ull << lane) - 1ull)) << k;
            wt += __popcll(bal) << k;
        }
        if (lane == 0) wave_tot[j & 1][wv] = wt;
        __syncthreads();
        int batch = 0;
        for (int q = 0; q < nw; ++q) {
            const int w = wave_tot[j & 1][q];
            if (q < wv) off += w;
            batch += w;
        }
        off += total;
        total += batch;
        while (bits) {
            const int c = __ffs((int)bits) - 1;
            bits &= bits - 1;
            const float *mid = row + c;
            NccPeak pk;
            pk.iz = zp;
            pk.iu = 8 * ig + c - 1;
            pk.up = mid[-NS];
            pk.dn = mid[NS];
            pk.left = mid[-1];
            pk.right = mid[1];
            pk.n0 = mid[0];
            out[off++] = pk;
        }
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane == 0) wave_max[wv] = m;
    __syncthreads();
    if (t == 0) {
        for (int q = 1; q < nw; ++q) m = fmaxf(m, wave_max[q]);
        band_max[slot] = m;
        band_cnt[slot] = total;
    }
}

// The intensity threshold of an image: alpha times the maximum of its bands'
// maxima (work-groups of 256 threads; every thread gets it).
__device__ inline float ncc_threshold(const float *__restrict__ band_max, int img, int bands,
                                      float alpha) {
    float m = 0.f;
    for (int b = threadIdx.x & 63; b < bands; b += 64) m = fmaxf(m, band_max[(size_t)img * bands + b]);
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    return alpha * m;
}

// One work-group per image, a wave per band in turn: the intensity of each band's
// maxima, and the number of those that reach the threshold, as offsets within the
// image.
__global__ __launch_bounds__(256) void ncc_count_kernel(const float2 *__restrict__ P,
                                                        NccPeak *__restrict__ staged,
                                                        const float *__restrict__ band_max,
                                                        const int *__restrict__ band_cnt,
                                                        int *__restrict__ band_off,
                                                        int *__restrict__ img_cnt, float alpha,
                                                        int nz, int nu, int bands, int band_cap)
{
    const int img = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float thr = ncc_threshold(band_max, img, bands, alpha);
    for (int b = wv; b < bands; b += 4) {
        const size_t slot = (size_t)img * bands + b;
        const int n = band_cnt[slot];
        NccPeak *pk = staged + slot * band_cap;
        int c = 0;
        for (int i = lane; i < n; i += 64) {
            const float v = ncc_mag(P[((size_t)img * nz + pk[i].iz) * nu + pk[i].iu]);
            pk[i].intensity = v;
            c += v >= thr ? 1 : 0;
        }
        for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
        if (lane == 0) band_off[slot] = c;
    }
    __syncthreads();
    // exclusive scan of the image's bands by the first wave
    if (wv != 0) return;
    int carry = 0;
    for (int b0 = 0; b0 < bands; b0 += 64) {
        const int b = b0 + lane;
        const int c = b < bands ? band_off[(size_t)img * bands + b] : 0;
        int incl = c;
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        if (b < bands) band_off[(size_t)img * bands + b] = carry + incl - c;
        carry += __shfl(incl, 63);
    }
    if (lane == 0) img_cnt[img] = carry;
}

// One work-group per image, a wave per band in turn: the records of the maxima
// that reach the threshold, in order, with the sub-pixel fit (here, where every
// lane has one, rather than where they are found).
__global__ __launch_bounds__(256) void ncc_write_kernel(const NccPeak *__restrict__ staged,
                                                        const float *__restrict__ band_max,
                                                        const int *__restrict__ band_cnt,
                                                        const int *__restrict__ band_off,
                                                        const int *__restrict__ img_off,
                                                        ulm_loc_t *__restrict__ locs, int capacity,
                                                        float alpha, int nz, int nu, int F, int bands,
                                                        int band_cap)
{
    const int img = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float thr = ncc_threshold(band_max, img, bands, alpha);
    for (int b = wv; b < bands; b += 4) {
        const size_t slot = (size_t)img * bands + b;
        const int n = band_cnt[slot];
        const NccPeak *src = staged + slot * band_cap;
        int o = img_off[img] + band_off[slot];
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            NccPeak pk = src[min(i, n - 1)];
            const bool keep = i < n && pk.intensity >= thr;
            const unsigned long long bal = __ballot(keep);
            const int at = o + __popcll(bal & ((1ull << lane) - 1ull));
            o += __popcll(bal);
            if (!keep || at >= capacity) continue;
            const float dz = (pk.iz > 0 && pk.iz < nz - 1) ? subpix(pk.up, pk.n0, pk.dn) : 0.f;
            const float du = (pk.iu > 0 && pk.iu < nu - 1) ? subpix(pk.left, pk.n0, pk.right) : 0.f;
            ulm_loc_t rec;
            rec.plane = img / F;
            rec.frame = img % F;
            rec.iz = pk.iz;
            rec.iu = pk.iu;
            rec.z = (float)pk.iz + dz;
            rec.u = (float)pk.iu + du;
            rec.ncc = pk.n0;
            rec.intensity = pk.intensity;
            locs[at] = rec;
        }
    }
}

// Exclusive scan of n counts by one work-group; writes the total to *count.
__global__ __launch_bounds__(1024) void loc_scan_kernel(const int *__restrict__ cnt,
                                                        int *__restrict__ off, int n,
                                                        int *__restrict__ count)
{
    // passes of 4096 counts, 4 consecutive ones per thread: each wave scans its
    // threads' sums with lane shuffles, the 16 wave totals meet in LDS (double-
    // buffered by pass parity: one barrier per pass), and a running carry links
    // the passes; the next pass's counts are loaded during this one
    __shared__ int wtot[2][16];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    auto load4 = [&](int b0, int (&v)[4]) {
        const int i0 = b0 + 4 * t;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = i0 + q < n ? cnt[i0 + q] : 0;
    };
    int cur[4], nxt[4];
    load4(0, cur);
    int carry = 0, par = 0;
    for (int b0 = 0; b0 < n; b0 += 4096) {
        load4(b0 + 4096, nxt);
        const int sum = cur[0] + cur[1] + cur[2] + cur[3];
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        if (lane == 63) wtot[par][wv] = incl;
        __syncthreads();
        int base = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int x = wtot[par][q];
            if (q < wv) base += x;
            tot += x;
        }
        int run = carry + base + incl - sum;
        const int i0 = b0 + 4 * t;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (i0 + q < n) off[i0 + q] = run;
            run += cur[q];
        }
        carry += tot;
        par ^= 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) cur[q] = nxt[q];
    }
    if (t == 0) *count = carry;
}

__global__ __launch_bounds__(256) void loc_scatter_kernel(
    const ulm_loc_t *__restrict__ staged, const int *__restrict__ cnt, const int *__restrict__ off,
    ulm_loc_t *__restrict__ locs, int capacity, int band_cap)
{
    const int slot = blockIdx.x;
    const int n = cnt[slot], o = off[slot];
    const ulm_loc_t *src = staged + (size_t)slot * band_cap;
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        if (o + i < capacity) locs[o + i] = src[i];
}

__global__ void density_kernel(const ulm_loc_t *__restrict__ locs, const int *__restrict__ count,
                               int capacity, int up, int nz, int nu, int planes,
                               uint32_t *__restrict__ dens)
{
    const int n = min(*count, capacity);
    const int W = nu * up, H = nz * up;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const ulm_loc_t r = locs[i];
        const int bz = (int)floorf((r.z + 0.5f) * up);
        const int bu = (int)floorf((r.u + 0.5f) * up);
        if (r.plane < 0 || r.plane >= planes || bz < 0 || bz >= H || bu < 0 || bu >= W) continue;
        atomicAdd(&dens[((size_t)r.plane * H + bz) * W + bu], 1u);
    }
}

// LDS of the band kernel, and the limit on the plane's width: what a band of 16
// rows takes whole (envelope with halo and three vertical sums), so that a width
// is accepted or refused independently of the batch shape.
static size_t ncc_stream_lds(int nu, int half) {
    return sizeof(float) * ((size_t)3 * kNccBatch * ncc_vstride(nu, half) +
                            (size_t)(2 + kNccBatch) * ncc_nstride(nu));
}

size_t ncc_lds_bytes(int nu, int half) {
    const size_t R_out = 16 + 2, R_in = R_out + 2 * half, W_in = nu + 2 + 2 * half;
    const size_t img = std::max(R_in * W_in, R_out * (size_t)(nu + 2));
    return (img + 3 * R_out * W_in) * sizeof(float);
}

// Rows per band: 8 m - 2, so that a band is m whole batches.  The tallest that
// leaves eight work-groups per CU: taller bands read and root fewer halo rows
// (2H + 2 per band), shorter ones keep the chip filled on small ensembles.
int ncc_band_rows(int n_img, int nz) {
    for (int r : {38, 22})
        if ((long)n_img * cdiv(nz, r) >= 2048) return r;
    return 14;
}

NccParams make_ncc_params(const ulm_ctx *ctx) {
    const ulm_config_t &c = ctx->cfg;
    NccParams p{};
    const int h = (c.ncc_size - 1) / 2;
    p.half = h;
    double sz = 0, su = 0;
    double gz[2 * kNccMaxHalf + 1], gu[2 * kNccMaxHalf + 1];
    for (int a = -h; a <= h; ++a) {
        gz[a + h] = exp(-(double)a * a / (2.0 * c.sigma_z * c.sigma_z));
        gu[a + h] = exp(-(double)a * a / (2.0 * c.sigma_u * c.sigma_u));
        sz += gz[a + h];
        su += gu[a + h];
        if (a <= 0) {
            p.gz[a + h] = (float)gz[a + h];
            p.gu[a + h] = (float)gu[a + h];
        }
    }
    const double W = (double)c.ncc_size * c.ncc_size;
    const double kbar = sz * su / W;
    double sk = 0;
    for (int a = 0; a < c.ncc_size; ++a)
        for (int b = 0; b < c.ncc_size; ++b) {
            const double d = gz[a] * gu[b] - kbar;
            sk += d * d;
        }
    p.kbar = (float)kbar;
    p.inv_w = (float)(1.0 / W);
    p.inv_sk = (float)(1.0 / sqrt(sk));
    p.tau = (float)c.tau_ncc;
    p.alpha = (float)c.alpha;
    return p;
}

hipError_t launch_localize(const ulm_ctx *ctx, const float2 *filt, ulm_loc_t *locs, int capacity,
                           int *count, char *ws, hipStream_t st)
{
    const Geometry &g = ctx->geo;
    const Workspace &w = ctx->ws;
    const int F = g.n_frames, planes = g.n_planes;
    const int n_img = planes * F;
    float *bmax = (float *)(ws + w.band_max);
    int *bcnt = (int *)(ws + w.band_cnt);
    int *boff = (int *)(ws + w.band_off);
    int *icnt = (int *)(ws + w.img_cnt), *ioff = (int *)(ws + w.img_off);
    NccPeak *staged = (NccPeak *)(ws + w.staged);
    const NccParams prm = make_ncc_params(ctx);
    const int W_in = g.nu + 2 + 2 * prm.half;
    const int threads = 64 * cdiv(W_in, 64);                // one per input column
    if (threads > kNccMaxThreads) return hipErrorInvalidValue;
    const size_t lds = ncc_stream_lds(g.nu, prm.half);
#define ULM_NCC_BAND(HH)                                                                          \
    case HH:                                                                                      \
        hipLaunchKernelGGL(ncc_stream_kernel<HH>, dim3(n_img * w.bands), dim3(threads), lds, st,  \
                           filt, bmax, staged, bcnt, prm, g.nz, g.nu, w.bands, w.band_rows,       \
                           w.band_cap);                                                           \
        break;
    switch (prm.half) {
        ULM_NCC_BAND(1)
        ULM_NCC_BAND(2)
        ULM_NCC_BAND(3)
        ULM_NCC_BAND(4)
        ULM_NCC_BAND(5)
        ULM_NCC_BAND(6)
        ULM_NCC_BAND(7)
        default: return hipErrorInvalidValue;
    }
#undef ULM_NCC_BAND
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ncc_count_kernel, dim3(n_img), dim3(256), 0, st, filt, staged, bmax, bcnt, boff,
                       icnt, prm.alpha, g.nz, g.nu, w.bands, w.band_cap);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(loc_scan_kernel, dim3(1), dim3(1024), 0, st, icnt, ioff, n_img, count);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(ncc_write_kernel, dim3(n_img), dim3(256), 0, st, staged, bmax, bcnt, boff, ioff,
                       locs, capacity, prm.alpha, g.nz, g.nu, F, w.bands, w.band_cap);
    return hipGetLastError();
}

hipError_t launch_frame_max(const float2 *P, float *fmax, int n_img, int npix, hipStream_t st)
{
    hipLaunchKernelGGL(frame_max_kernel, dim3(n_img), dim3(256), 0, st, P, fmax, npix);
    return hipGetLastError();
}

// Exclusive scan of n counts into off, the total into *count.
hipError_t launch_scan(const int *cnt, int *off, int n, int *count, hipStream_t st)
{
    hipLaunchKernelGGL(loc_scan_kernel, dim3(1), dim3(1024), 0, st, cnt, off, n, count);
    return hipGetLastError();
}

// Exclusive scan of per-slot counts, then each slot's records to its offset.
hipError_t launch_compact(const int *cnt, int *off, int nslots, int *count, const ulm_loc_t *staged,
                          int cap, ulm_loc_t *locs, int capacity, hipStream_t st)
{
    hipLaunchKernelGGL(loc_scan_kernel, dim3(1), dim3(1024), 0, st, cnt, off, nslots, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(loc_scatter_kernel, dim3(nslots), dim3(256), 0, st, staged, cnt, off, locs,
                       capacity, cap);
    return hipGetLastError();
}

hipError_t launch_density(const ulm_ctx *ctx, const ulm_loc_t *locs, const int *count,
                          int capacity, int up, uint32_t *dens, hipStream_t st)
{
    const Geometry &g = ctx->geo;
    hipLaunchKernelGGL(density_kernel, dim3(1024), dim3(256), 0, st, locs, count, capacity, up,
                       g.nz, g.nu, g.n_planes, dens);
    return hipGetLastError();
}


}  // namespace ulm

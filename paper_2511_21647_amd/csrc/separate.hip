// MB separation of the filtered planes into flow sub-populations (paper Section
// II-A5): at every pixel, the F-point DFT of the slow-time signal, an ideal
// band-pass mask per subset (up = positive-frequency bins 1..H, down = the
// negative ones, H = (F - 1) / 2, each direction split by |frequency| into S
// contiguous speed ranges), and the inverse DFT of each masked spectrum.
//
// sep_two_kernel: frame counts that split into two radices (all but five of those
// supported); two passes with the butterflies in registers (see below).
// sep_kernel: the others; one work-group per (plane, 8 consecutive pixels).  The frames
// of those pixels are staged in LDS ([frame][pixel], pixels fastest, so the
// global loads and stores are 64-byte rows and the butterflies read
// consecutive banks), transformed by a mixed-radix Stockham FFT (radices 4, 2,
// 3, 5, 7) that ping-pongs between two LDS buffers, and the spectrum is kept in
// registers; each subset then rewrites its masked spectrum to LDS, runs the
// inverse transform and streams the result out.  HBM traffic is one read of
// the planes and one write per subset.
#include "common.h"

#include <math.h>

#include <cmath>
#include <utility>
#include <vector>

namespace ulm {

constexpr int kSepPix = 8;                  // pixels per work-group
constexpr int kSepThreads = 256;
constexpr int kSepMaxFrames = 512;
constexpr int kSepMaxPass = 12;
constexpr int kSepMaxSub = 16;              // 2 S subsets, S <= 8
constexpr int kSepRegs = (kSepMaxFrames * kSepPix + kSepThreads - 1) / kSepThreads;

struct SepArgs {
    int F, npix, planes, n_sub, H;
    int n_pass;
    int radix[kSepMaxPass];
    int tw_off[kSepMaxPass];                // offset of each pass's twiddles in the table
    unsigned pmag[kSepMaxPass];             // floor(2^32 / p) + 1 for the pass's p (0 when p = 1)
    int n_tw;                               // twiddle entries (all passes)
    const float2 *twt;                      // [n_tw + 21] twiddles, then the radix roots
    const float2 *twf;                      // [2][F] exp(-2 pi i n / F), and over F, for the two-pass form
    int lo[kSepMaxSub], hi[kSepMaxSub];     // |k| range of each subset
};

__device__ inline float2 cmulf(float2 a, float2 b) {
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ inline float2 cmulf_conj(float2 a, float2 b) {   // a * conj(b)
    return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// -i z (forward) or +i z (inverse)
template <bool INV>
__device__ inline float2 mul_mi(float2 z) { return INV ? make_float2(-z.y, z.x) : make_float2(z.y, -z.x); }

// In-place R-point DFT of u, u_out[m] = sum_q u[q] exp(-+2 pi i q m / R).
// Radices 2, 3, 4 and 5 use the usual symmetric forms; 7 the direct sum with
// the roots wr[] (exp(-2 pi i q / 7)).
template <int R, bool INV>
__device__ inline void sep_dft(float2 (&u)[R], const float2 *wr)
{
    auto add = [](float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); };
    auto sub = [](float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); };
    auto scl = [](float2 a, float s) { return make_float2(a.x * s, a.y * s); };
    if constexpr (R == 2) {
        const float2 a = u[0], b = u[1];
        u[0] = add(a, b);
        u[1] = sub(a, b);
    } else if constexpr (R == 4) {
        const float2 s02 = add(u[0], u[2]), d02 = sub(u[0], u[2]);
        const float2 s13 = add(u[1], u[3]), d13 = mul_mi<INV>(sub(u[1], u[3]));
        u[0] = add(s02, s13);
        u[2] = sub(s02, s13);
        u[1] = add(d02, d13);
        u[3] = sub(d02, d13);
    } else if constexpr (R == 3) {
        constexpr float h = 0.866025403784438646763723f;     // sin(2 pi / 3)
        const float2 t1 = add(u[1], u[2]);
        const float2 t2 = sub(u[0], scl(t1, 0.5f));
        const float2 t3 = mul_mi<INV>(scl(sub(u[1], u[2]), h));
        u[0] = add(u[0], t1);
        u[1] = add(t2, t3);
        u[2] = sub(t2, t3);
    } else if constexpr (R == 5) {
        constexpr float c1 = 0.309016994374947424102293f;     // cos(2 pi / 5)
        constexpr float c2 = -0.809016994374947424102293f;    // cos(4 pi / 5)
        constexpr float s1 = 0.951056516295153572116439f;     // sin(2 pi / 5)
        constexpr float s2 = 0.587785252292473129168706f;     // sin(4 pi / 5)
        const float2 t1 = add(u[1], u[4]), t2 = add(u[2], u[3]);
        const float2 t3 = sub(u[1], u[4]), t4 = sub(u[2], u[3]);
        auto even = [&](float p, float q) {
            return make_float2(fmaf(t2.x, q, fmaf(t1.x, p, u[0].x)), fmaf(t2.y, q, fmaf(t1.y, p, u[0].y)));
        };
        const float2 a1 = even(c1, c2), a2 = even(c2, c1);
        const float2 b1 = mul_mi<INV>(add(scl(t3, s1), scl(t4, s2)));
        const float2 b2 = mul_mi<INV>(sub(scl(t3, s2), scl(t4, s1)));
        u[0] = add(u[0], add(t1, t2));
        u[1] = add(a1, b1);
        u[4] = sub(a1, b1);
        u[2] = add(a2, b2);
        u[3] = sub(a2, b2);
    } else {
        float2 o[R];
#pragma unroll
        for (int qo = 0; qo < R; ++qo) {
            float2 acc = u[0];
#pragma unroll
            for (int q = 1; q < R; ++q) {
                const float2 w = wr[(q * qo) % R];
                const float2 t = INV ? cmulf_conj(u[q], w) : cmulf(u[q], w);
                acc.x += t.x;
                acc.y += t.y;
            }
            o[qo] = acc;
        }
#pragma unroll
        for (int qo = 0; qo < R; ++qo) u[qo] = o[qo];
    }
}

// One Stockham pass of radix R over every pixel: x -> y.  p = product of the
// radices of the earlier passes; tw[k R + q] = exp(-2 pi i q k / (p R)) for
// k < p; wr[q] = exp(-2 pi i q / R).  INV uses the conjugates.  i mod p comes
// from a multiply-high by pmag = floor(2^32 / p) + 1, exact for i, p < 2^16.
template <int R, bool INV>
__device__ void sep_pass(const float2 *__restrict__ x, float2 *__restrict__ y, int F, int p,
                         unsigned pmag, const float2 *tw, const float2 *wr)
{
    const int nb = F / R;                                  // butterflies per pixel
    for (int e = threadIdx.x; e < nb * kSepPix; e += kSepThreads) {
        const int i = e / kSepPix, px = e % kSepPix;
        const int k = p == 1 ? 0 : i - (int)__umulhi((unsigned)i, pmag) * p;
        float2 u[R];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            float2 v = x[(i + q * nb) * kSepPix + px];
            if (q > 0) v = INV ? cmulf_conj(v, tw[k * R + q]) : cmulf(v, tw[k * R + q]);
            u[q] = v;
        }
        const int j = (i - k) * R + k;
        sep_dft<R, INV>(u, wr);
#pragma unroll
        for (int qo = 0; qo < R; ++qo) y[(j + qo * p) * kSepPix + px] = u[qo];
    }
}

// All passes; returns the buffer that holds the result.
template <bool INV>
__device__ float2 *sep_fft(float2 *a, float2 *b, const SepArgs &g, const float2 *tw,
                           const float2 *wr)
{
    int p = 1;
    for (int s = 0; s < g.n_pass; ++s) {
        const int R = g.radix[s];
        const float2 *t = tw + g.tw_off[s];
        switch (R) {
            case 2: sep_pass<2, INV>(a, b, g.F, p, g.pmag[s], t, wr + 0); break;
            case 3: sep_pass<3, INV>(a, b, g.F, p, g.pmag[s], t, wr + 2); break;
            case 4: sep_pass<4, INV>(a, b, g.F, p, g.pmag[s], t, wr + 5); break;
            case 5: sep_pass<5, INV>(a, b, g.F, p, g.pmag[s], t, wr + 9); break;
            default: sep_pass<7, INV>(a, b, g.F, p, g.pmag[s], t, wr + 14); break;
        }
        __syncthreads();
        float2 *c = a;
        a = b;
        b = c;
        p *= R;
    }
    return a;
}

__global__ __launch_bounds__(kSepThreads) void sep_kernel(const float2 *__restrict__ P,
                                                          float2 *__restrict__ out, SepArgs g)
{
    extern __shared__ float2 sm[];
    float2 *buf0 = sm;                                     // [F][kSepPix]
    float2 *buf1 = sm + (size_t)g.F * kSepPix;
    float2 *tw = buf1 + (size_t)g.F * kSepPix;             // [n_tw]
    float2 *wr = tw + g.n_tw;                              // radix roots: 2, 3, 4, 5, 7 -> 21
    const int groups = cdiv(g.npix, kSepPix);
    const int plane = blockIdx.x / groups, px0 = (blockIdx.x % groups) * kSepPix;
    const int t = threadIdx.x;

    // twiddles of every pass and the roots of unity of every radix, from the
    // context's table (tw and wr are contiguous, as in the table)
    for (int e = t; e < g.n_tw + 21; e += kSepThreads) tw[e] = g.twt[e];
    const float2 *src = P + (size_t)plane * g.F * g.npix + px0;
    const int npx = min(kSepPix, g.npix - px0);
    for (int e = t; e < g.F * kSepPix; e += kSepThreads) {
        const int f = e / kSepPix, px = e % kSepPix;
        buf0[e] = px < npx ? src[(size_t)f * g.npix + px] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    const float2 *X = sep_fft<false>(buf0, buf1, g, tw, wr);
    // the spectrum stays in registers: element e = t + 256 r
    float2 xr[kSepRegs];
    int nreg = 0;
#pragma unroll
    for (int r = 0; r < kSepRegs; ++r) {
        const int e = t + r * kSepThreads;
        if (e < g.F * kSepPix) {
            xr[r] = X[e];
            nreg = r + 1;
        }
    }
    const float scale = 1.0f / (float)g.F;
    const size_t sub_stride = (size_t)g.planes * g.F * g.npix;
    for (int s = 0; s < g.n_sub; ++s) {
        const bool up = s < g.n_sub / 2;
        const int lo = g.lo[s], hi = g.hi[s];
        __syncthreads();                                    // previous subset's reads done
#pragma unroll
        for (int r = 0; r < kSepRegs; ++r) {
            if (r < nreg) {
                const int e = t + r * kSepThreads;
                if (e < g.F * kSepPix) {
                    const int k = e / kSepPix;
                    const int m = up ? k : g.F - k;
                    const bool keep = (up ? (k >= 1 && k <= g.H) : (k >= g.F - g.H)) && m >= lo && m < hi;
                    buf0[e] = keep ? xr[r] : make_float2(0.f, 0.f);
                }
            }
        }
        __syncthreads();
        const float2 *Y = sep_fft<true>(buf0, buf1, g, tw, wr);
        float2 *dst = out + s * sub_stride + (size_t)plane * g.F * g.npix + px0;
        for (int e = t; e < g.F * kSepPix; e += kSepThreads) {
            const int f = e / kSepPix, px = e % kSepPix;
            if (px < npx) {
                const float2 v = Y[e];
                dst[(size_t)f * g.npix + px] = make_float2(v.x * scale, v.y * scale);
            }
        }
    }
}

// ---------------------------------------------------------------- two-pass form
// F = R1 R2 with both factors among sep_is_radix: the transform is two passes whose
// butterflies stay in registers.  With n = i + R2 q and k = m1 + R1 m2,
//   X[k] = sum_i w_F^{i m1} [sum_q x[n] w_R1^{q m1}] w_R2^{i m2},
// so thread (i, pixel) takes the R1 frames i + R2 q straight from memory, thread
// (m1, pixel) ends with the R2 spectrum values m1 + R1 m2 and keeps them, and a
// subset's inverse runs the same way back: its masked values through the R2-point
// inverse in the registers that hold them, one exchange through LDS, the twiddles and
// the R1-point inverse, and the frames straight to memory.  One LDS exchange a
// transform (the general kernel: one a radix and the staging).
// Bound by the stores: six subsets of 2 x 300 frames of 68500 pixels 1189 -> 546 us, of
// which the loads and stores alone take 560 and all but the stores 380 (one or two
// work-groups a CU overlap the two; consecutive work-groups on one XCD, whose L2 joins
// the lines they share, 946 us without).  20 frames of 64 x 64 pixels 25 -> 11 us, 512 of
// 150 x 200 1066 -> 450 us.
// Rounding: the error against 64 bits is 0.90 of the general kernel's form on average over
// the frame counts, at 12 frames 1.03 and elsewhere at most 1.01 (300: 1.32e-7 against
// 1.49e-7), because the coprime factors of a radix have no twiddles, and 1 / F comes with
// the inverse's twiddles instead of as a rounding of its own.

// cos and sin of 2 pi q / R at compile time (Taylor series about the nearest octant's
// multiple, in double)
constexpr double sep_series(double x, bool odd) {
    double term = odd ? x : 1.0, sum = term;
    for (int n = odd ? 2 : 1; n < 40; n += 2) {
        term *= -x * x / (double)(n * (n + 1));
        sum += term;
    }
    return sum;
}
constexpr double kSepPi = 3.14159265358979323846264338327950288;
constexpr double sep_cos(int q, int R) {
    q %= R;
    if (2 * q > R) return sep_cos(R - q, R);
    if (4 * q > R) return -sep_cos(R - 2 * q, 2 * R);
    if (8 * q > R) return sep_series(kSepPi * (R - 4 * q) / (2.0 * R), true);
    return sep_series(2.0 * kSepPi * q / R, false);
}
constexpr double sep_sin(int q, int R) {
    q %= R;
    if (2 * q > R) return -sep_sin(R - q, R);
    if (4 * q > R) return sep_sin(R - 2 * q, 2 * R);
    if (8 * q > R) return sep_series(kSepPi * (R - 4 * q) / (2.0 * R), false);
    return sep_series(2.0 * kSepPi * q / R, true);
}

// cos and sin of 2 pi q / R, what their rounding leaves over in the l arrays.
template <int R> struct SepRoots {
    float c[R], s[R], cl[R], sl[R];
    constexpr SepRoots() : c(), s(), cl(), sl() {
        for (int q = 0; q < R; ++q) {
            c[q] = (float)sep_cos(q, R);
            s[q] = (float)sep_sin(q, R);
            cl[q] = (float)(sep_cos(q, R) - (double)c[q]);
            sl[q] = (float)(sep_sin(q, R) - (double)s[q]);
        }
    }
};

// z (c - i s), or z (c + i s) for INV; c and s one float each, or the sum of two.
template <bool INV>
__device__ inline float2 sep_turn(float2 z, float c, float s)
{
    const float t = INV ? -s : s;
    return make_float2(fmaf(z.x, c, z.y * t), fmaf(z.y, c, -z.x * t));
}
template <bool INV>
__device__ inline float2 sep_turn(float2 z, float c, float s, float cl, float sl)
{
    const float t = INV ? -s : s, tl = INV ? -sl : sl;
    return make_float2(fmaf(z.x, c, fmaf(z.y, t, fmaf(z.x, cl, z.y * tl))),
                       fmaf(z.y, c, fmaf(-z.x, t, fmaf(z.y, cl, -z.x * tl))));
}

// The smallest factor A of R that has none in common with R / A (R if there is none).
constexpr int sep_coprime(int R) {
    for (int a = 2; a < R; ++a) {
        int x = a, y = R / a;
        while (y != 0) {
            const int t = x % y;
            x = y;
            y = t;
        }
        if (R % a == 0 && x == 1) return a;
    }
    return R;
}

// In-place R-point DFT in registers, as sep_dft.  R = A B with coprime factors goes by
// the prime-factor algorithm (Good and Thomas): with n = (B n1 + A n2) mod R,
//   X[k] = sum_n1 w_A^{n1 k} sum_n2 w_B^{n2 k} x[n],
// A-point and B-point DFTs without twiddles between them.  Powers of one prime have
// twiddles between the two: 9 and 16 as a pass's whole radix of two floats, as one float's
// rounding makes the transform less exact than radix by radix there (81, 256 and 512 frames
// by 3-4%) and not elsewhere (324 by 1%), and in 27 and 18 two take 405 and 486 frames past
// 128 registers (382 -> 444 and 435 -> 515 us).
template <int R, bool INV, bool TOP = true>
__device__ inline void sep_reg_dft(float2 (&u)[R])
{
    if constexpr (R <= 5) {
        sep_dft<R, INV>(u, nullptr);
    } else if constexpr (R == 7) {
        constexpr SepRoots<R> w;
        float2 a[3], b[3], o[R];
        o[0] = u[0];
#pragma unroll
        for (int q = 1; q <= 3; ++q) {
            a[q - 1] = make_float2(u[q].x + u[R - q].x, u[q].y + u[R - q].y);
            b[q - 1] = make_float2(u[q].x - u[R - q].x, u[q].y - u[R - q].y);
            o[0].x += a[q - 1].x;
            o[0].y += a[q - 1].y;
        }
#pragma unroll
        for (int m = 1; m <= 3; ++m) {
            float2 re = u[0], im = make_float2(0.f, 0.f);
#pragma unroll
            for (int q = 1; q <= 3; ++q) {
                re.x = fmaf(w.c[q * m % R], a[q - 1].x, re.x);
                re.y = fmaf(w.c[q * m % R], a[q - 1].y, re.y);
                im.x = fmaf(w.s[q * m % R], b[q - 1].x, im.x);
                im.y = fmaf(w.s[q * m % R], b[q - 1].y, im.y);
            }
            const float2 t = mul_mi<INV>(im);
            o[m] = make_float2(re.x + t.x, re.y + t.y);
            o[R - m] = make_float2(re.x - t.x, re.y - t.y);
        }
#pragma unroll
        for (int q = 0; q < R; ++q) u[q] = o[q];
    } else if constexpr (sep_coprime(R) < R) {
        constexpr int A = sep_coprime(R), B = R / A;
        float2 v[A][B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) {
            float2 x[A];
#pragma unroll
            for (int n1 = 0; n1 < A; ++n1) x[n1] = u[(B * n1 + A * n2) % R];
            sep_reg_dft<A, INV, TOP>(x);
#pragma unroll
            for (int k = 0; k < A; ++k) v[k][n2] = x[k];
        }
#pragma unroll
        for (int k = 0; k < A; ++k) sep_reg_dft<B, INV, TOP>(v[k]);
#pragma unroll
        for (int k = 0; k < R; ++k) u[k] = v[k % A][k % B];
    } else {
        constexpr int A = R % 4 == 0 ? 4 : (R % 5 == 0 ? 5 : 3);
        constexpr int B = R / A;
        constexpr SepRoots<R> w;
        float2 v[A][B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            float2 x[A];
#pragma unroll
            for (int q = 0; q < A; ++q) x[q] = u[i + B * q];
            sep_reg_dft<A, INV, false>(x);
#pragma unroll
            for (int m = 0; m < A; ++m) {
                // exp(-+ 2 pi i (i m) / R)
                const int j = i * m;
                if (j == 0) v[m][i] = x[m];
                else if (TOP && (R == 9 || R == 16)) v[m][i] = sep_turn<INV>(x[m], w.c[j], w.s[j], w.cl[j], w.sl[j]);
                else v[m][i] = sep_turn<INV>(x[m], w.c[j], w.s[j]);
            }
        }
#pragma unroll
        for (int m = 0; m < A; ++m) {
            sep_reg_dft<B, INV, false>(v[m]);
#pragma unroll
            for (int m2 = 0; m2 < B; ++m2) u[m + A * m2] = v[m][m2];
        }
    }
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Pixels of a work-group: rows of 256 bytes (128-byte rows: 777 us where these took 605),
// but 128 where a thread's second butterfly leaves too few registers for 32 pixels'
// threads (512 frames, R2 = 32: 824 us with 256-byte rows, 450 so; R2 = 25 still 561
// against 647, though its 800 threads leave 128 registers and 14, 15, 18 and 20 beside it
// spill 3 to 10).
constexpr int sep_pixels(int r2) { return r2 <= 25 ? 32 : 16; }
constexpr int sep_threads(int r2) { return (r2 * sep_pixels(r2) + 63) / 64 * 64; }

template <int R1, int R2>
__global__ __launch_bounds__(sep_threads(R2)) void sep_two_kernel(
    const float2 *__restrict__ P, float2 *__restrict__ out, SepArgs g)
{
    constexpr int F = R1 * R2, kPix = sep_pixels(R2), kRow = R2 * kPix;
    __shared__ float2 ex[R1][kRow];               // [m1][i][pixel]
    const int groups = cdiv(g.npix, kPix);
    const int lin = xcd_remap(blockIdx.x, groups * g.planes);
    const int plane = lin / groups, px = threadIdx.x % kPix, i = threadIdx.x / kPix;
    const int p = lin % groups * kPix + px;
    const bool first = i < R2, second = i < R1;   // i is m1 in the second pass
    // a plane through a descriptor: the frame's offset is scalar; pixels past the plane
    // lie outside it, read as zero and are not stored
    const int row = g.npix * (int)sizeof(float2);
    const int off = p < g.npix && first ? i * row + p * (int)sizeof(float2) : -16;
    const size_t at = (size_t)plane * F * g.npix;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float2 *>(P + at), 0, F * row, 0x00027000);

    // exp(-2 pi i n / F), and over F for the inverses (side by side: one address)
    __shared__ float2 tw[F][2];
    for (int e = threadIdx.x; e < F; e += sep_threads(R2)) {
        tw[e][0] = g.twf[e];
        tw[e][1] = g.twf[F + e];
    }
    lds_barrier();
    if (first) {
        float2 u[R1];
#pragma unroll
        for (int q = 0; q < R1; ++q) {
            const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(src, off, R2 * q * row, 0));
            u[q] = make_float2(v[0], v[1]);
        }
        sep_reg_dft<R1, false>(u);
#pragma unroll
        for (int m = 0; m < R1; ++m) ex[m][i * kPix + px] = m == 0 ? u[m] : cmulf(u[m], tw[i * m][0]);
    }
    lds_barrier();
    float2 X[R2];
    if (second) {
#pragma unroll
        for (int n = 0; n < R2; ++n) X[n] = ex[i][n * kPix + px];
        sep_reg_dft<R2, false>(X);
    }
    // 1 / F for the terms without a twiddle, as the sum of two floats
    constexpr float s_hi = (float)(1.0 / F), s_lo = (float)(1.0 / F - (double)s_hi);
    const size_t sub_stride = (size_t)g.planes * F * g.npix;
    for (int s = 0; s < g.n_sub; ++s) {
        // bins [k0, k0 + n): lo.. up, or F - hi + 1.. down
        const bool up = s < g.n_sub / 2;
        const int n = g.hi[s] - g.lo[s], k0 = up ? g.lo[s] : F - g.hi[s] + 1;
        lds_barrier();                          // the reads of the exchange before
        if (second) {
            float2 y[R2];
#pragma unroll
            for (int m = 0; m < R2; ++m) {
                const bool keep = (unsigned)(i + R1 * m - k0) < (unsigned)n;
                y[m] = keep ? X[m] : make_float2(0.f, 0.f);
            }
            sep_reg_dft<R2, true>(y);
#pragma unroll
            for (int m = 0; m < R2; ++m) ex[i][m * kPix + px] = y[m];
        }
        lds_barrier();
        if (first) {
            float2 u[R1];
#pragma unroll
            for (int m = 0; m < R1; ++m) {
                const float2 v = ex[m][i * kPix + px];
                u[m] = m == 0 ? make_float2(fmaf(v.x, s_hi, v.x * s_lo), fmaf(v.y, s_hi, v.y * s_lo))
                              : cmulf_conj(v, tw[i * m][1]);
            }
            sep_reg_dft<R1, true>(u);
            const __amdgpu_buffer_rsrc_t dst =
                __builtin_amdgcn_make_buffer_rsrc(out + s * sub_stride + at, 0, F * row, 0x00027000);
#pragma unroll
            for (int q = 0; q < R1; ++q)
                __builtin_amdgcn_raw_buffer_store_b64(
                    __builtin_bit_cast(u32x2, f32x2{u[q].x, u[q].y}), dst, off, R2 * q * row, 0);
        }
    }
}

// The larger radices a butterfly is made for, and the smaller factor of the most even
// split of F into two of them (0 if there is none).
constexpr bool sep_is_radix(int r) {
    constexpr int set[] = {2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16, 18, 20, 21, 24, 25, 27, 28, 32, 35};
    for (int x : set)
        if (x == r) return true;
    return false;
}
constexpr int sep_split(int F) {
    int best = 0;
    for (int r = 2; r * r <= F; ++r)
        if (F % r == 0 && sep_is_radix(r) && sep_is_radix(F / r)) best = r;
    return best;
}
using SepKernel = void (*)(const float2 *, float2 *, SepArgs);
template <int F> constexpr SepKernel sep_two_of() {
    if constexpr (sep_split(F) != 0) return sep_two_kernel<sep_split(F), F / sep_split(F)>;
    else return nullptr;
}
struct SepTable { SepKernel k[kSepMaxFrames + 1]; };
template <int... Fs> constexpr SepTable sep_two_table(std::integer_sequence<int, Fs...>) {
    return {{sep_two_of<Fs>()...}};
}

// Radices for F (4 first, then 2, 3, 5, 7); false if F has another prime factor.
static bool sep_factor(int F, SepArgs &g) {
    g.n_pass = 0;
    int n = F, off = 0, p = 1;
    const int order[5] = {4, 2, 3, 5, 7};
    for (int r : order) {
        while (n % r == 0) {
            if (g.n_pass == kSepMaxPass) return false;
            g.radix[g.n_pass] = r;
            g.tw_off[g.n_pass] = off;
            g.pmag[g.n_pass] = p == 1 ? 0u : (unsigned)((1ull << 32) / (unsigned)p + 1ull);
            off += p * r;
            p *= r;
            ++g.n_pass;
            n /= r;
        }
    }
    g.n_tw = off;
    return n == 1;
}

bool separate_supported(int F) {
    SepArgs g;
    return F >= 2 && F <= kSepMaxFrames && sep_factor(F, g);
}

// The kernel's table for F frames: tw[tw_off[s] + k R + q] = exp(-2 pi i q k /
// (p R)) for every pass s (radix R, p = product of the earlier radices), then
// the roots exp(-2 pi i q / R) of R = 2, 3, 4, 5, 7 (2 + 3 + 4 + 5 + 7 = 21
// entries), then for the two-pass form exp(-2 pi i n / F) of n < F, and the same over F;
// FP64, rounded to FP32.  Empty if F is not supported.
std::vector<float2> separate_twiddles(int F) {
    SepArgs g;
    if (!separate_supported(F)) return {};
    sep_factor(F, g);
    std::vector<float2> t((size_t)g.n_tw + 21);
    auto root = [](double turns) {      // exp(2 pi i turns)
        return make_float2((float)std::cos(2.0 * M_PI * turns), (float)std::sin(2.0 * M_PI * turns));
    };
    int p = 1;
    for (int s = 0; s < g.n_pass; ++s) {
        const int R = g.radix[s];
        for (int e = 0; e < p * R; ++e) {
            const int k = e / R, q = e % R;
            t[g.tw_off[s] + e] = root(-(double)((long)q * k % (p * R)) / (double)(p * R));
        }
        p *= R;
    }
    const int rad[5] = {2, 3, 4, 5, 7};
    int o = g.n_tw;
    for (int r : rad)
        for (int q = 0; q < r; ++q) t[o++] = root(-(double)q / (double)r);
    for (int n = 0; n < F; ++n) t.push_back(root(-(double)n / (double)F));
    for (int n = 0; n < F; ++n) {
        const double a = 2.0 * M_PI * (double)n / (double)F;
        t.push_back(make_float2((float)(std::cos(a) / F), (float)(-std::sin(a) / F)));
    }
    return t;
}

size_t separate_lds_bytes(int F) {
    SepArgs g;
    sep_factor(F, g);
    return sizeof(float2) * ((size_t)2 * F * kSepPix + g.n_tw + 21);
}

hipError_t launch_separate(const ulm_ctx *ctx, const float2 *P, int n_speed, float2 *out,
                           hipStream_t st)
{
    const Geometry &geo = ctx->geo;
    SepArgs g;
    if (!sep_factor(geo.n_frames, g)) return hipErrorInvalidValue;
    g.F = geo.n_frames;
    g.npix = geo.nz * geo.nu;
    g.planes = geo.n_planes;
    g.n_sub = 2 * n_speed;
    g.H = (g.F - 1) / 2;
    for (int d = 0; d < 2; ++d)
        for (int s = 0; s < n_speed; ++s) {
            g.lo[d * n_speed + s] = 1 + (s * g.H) / n_speed;
            g.hi[d * n_speed + s] = 1 + ((s + 1) * g.H) / n_speed;
        }
    g.twt = ctx->tab.sep_tw;
    if (!g.twt) return hipErrorInvalidValue;
    g.twf = g.twt + g.n_tw + 21;
    // two passes where the frames split into two radices and a plane fits a descriptor's
    // 31-bit offsets; the general kernel otherwise (2, 3, 5, 7 and 343 frames)
    static constexpr auto two = sep_two_table(std::make_integer_sequence<int, kSepMaxFrames + 1>());
    const int r1 = sep_split(g.F);
    if (r1 && (size_t)g.F * g.npix * sizeof(float2) < (1ull << 31) - 4096) {
        const int r2 = g.F / r1;
        hipLaunchKernelGGL(two.k[g.F], dim3(cdiv(g.npix, sep_pixels(r2)) * g.planes), dim3(sep_threads(r2)), 0,
                           st, P, out, g);
        return hipGetLastError();
    }
    const int groups = cdiv(g.npix, kSepPix);
    hipLaunchKernelGGL(sep_kernel, dim3(groups * g.planes), dim3(kSepThreads),
                       separate_lds_bytes(g.F), st, P, out, g);
    return hipGetLastError();
}

}  // namespace ulm

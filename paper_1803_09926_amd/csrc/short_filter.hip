// Filter gradient of short launches in one kernel, depthwise and group, either layout, 3x3, 5x5 and 7x7, any stride, padding and multiplier.
//
// What bounds a short filter gradient is not its sums but its two launches: a second kernel that adds a few partials takes the host 2.9 us and
// the GPU 2.5 to 3.5, as much as the first.  Here a block owns its filter entries alone: a lane takes one pair of output and input channel and
// every step-th output position, keeps the sums of all taps, and the lanes of a pair are added up in the block, over a wavefront by butterfly and over the
// four wavefronts through LDS.  A position's values are all loaded before the first is used, and a tap outside the image adds nothing (its
// product is never formed, so that no infinity meets a zero).  Lanes: NCHW 64 or 256 positions of one pair, so that they read along
// the rows; NHWC cw consecutive pairs by 256 / cw positions.
#include "gconv.hpp"
#include "short_filter.hpp"

namespace dwc {

namespace {

struct ShortGeom {
    int C, H, W, s, p, O, Cg, Og, Ho, Wo;
    int npix, npairs;        // output positions of all images; (output, input channel of its group)
    int cw, lcw, ws;         // pairs of a wavefront (2^lcw), wavefronts that share them (1 or 4)
    float rHo, rWo;
};

// n / d for 0 <= n < 2^21, r = 1.0f / d
__device__ __forceinline__ int over(int n, float r) { return (int)(((float)n + 0.5f) * r); }

template <typename T, int LAYOUT, int K>
__global__ __launch_bounds__(256) void k_short_bwd_filter(ShortGeom g, const T *__restrict__ x, const T *__restrict__ dy, float *__restrict__ dw)
{
    extern __shared__ float red[];                           // [wavefront][tap][pair]
    constexpr bool NHWC = LAYOUT == LAYOUT_NHWC;
    constexpr int KK = K * K, U = K == 3 ? 2 : 1;            // positions of a lane at a time
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = lane & (g.cw - 1), groups = 4 / g.ws;
    const int pair = min((int)(blockIdx.x * groups + (g.ws == 1 ? wv : 0)) * g.cw + c, g.npairs - 1);
    const int o = NHWC ? pair % g.O : pair / g.Cg, ci = NHWC ? pair / g.O : pair - o * g.Cg, ch = o / g.Og * g.Cg + ci;
    const int per = 64 >> g.lcw, step = per * g.ws;
    float acc[KK];
#pragma unroll
    for (int t = 0; t < KK; ++t) acc[t] = 0.f;
    const int xw = NHWC ? g.C : 1, xh = g.W * xw, plane = g.H * g.W;      // elements between columns and rows of x
#pragma unroll 1
    for (int p0 = (lane >> g.lcw) + (g.ws == 4 ? wv * per : 0); p0 < g.npix; p0 += step * U) {
        T d[U], v[U][K][K];
        bool rows[U][K], cols[U][K];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool there = p0 + u * step < g.npix;
            const int q = there ? p0 + u * step : 0, r = over(q, g.rWo), ow = q - r * g.Wo, n = over(r, g.rHo), oh = r - n * g.Ho;
            d[u] = dy[NHWC ? q * g.O + o : (n * g.O + o) * (g.Ho * g.Wo) + oh * g.Wo + ow];
            const int h0 = oh * g.s - g.p, w0 = ow * g.s - g.p;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                rows[u][k] = there && (unsigned)(h0 + k) < (unsigned)g.H;
                cols[u][k] = (unsigned)(w0 + k) < (unsigned)g.W;
            }
            const int at = NHWC ? n * plane * g.C + ch : (n * g.C + ch) * plane;
#pragma unroll
            for (int kh = 0; kh < K; ++kh)
#pragma unroll
                for (int kw = 0; kw < K; ++kw) v[u][kh][kw] = x[at + (rows[u][kh] ? h0 + kh : 0) * xh + (cols[u][kw] ? w0 + kw : 0) * xw];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < KK; ++t) {
                const float sum = fmaf(ldf(&d[u]), ldf(&v[u][t / K][t % K]), acc[t]);
                acc[t] = rows[u][t / K] && cols[u][t % K] ? sum : acc[t];
            }
    }
    // (a step of all sums together: 49 sums one after the other took 20 us)
    for (int off = 32; off >= g.cw; off >>= 1)
#pragma unroll
        for (int t = 0; t < KK; ++t) acc[t] += __shfl_xor(acc[t], off, 64);
    if (lane < g.cw)
#pragma unroll
        for (int t = 0; t < KK; ++t) red[(wv * KK + t) * g.cw + c] = acc[t];
    __syncthreads();
    for (int e = threadIdx.x; e < groups * KK * g.cw; e += 256) {
        const int r = e >> g.lcw, grp = r / KK, t = r - grp * KK, pr = (int)(blockIdx.x * groups + grp) * g.cw + (e & (g.cw - 1));
        if (pr >= g.npairs) continue;
        const int n = KK * g.cw;
        // (the largest sums, whose rounding counts most, in 64 bits: error of 0.83 to 0.95 of the two launches', no longer)
        const float sum = g.ws == 4 ? (float)(((double)red[e] + (double)red[e + n]) + ((double)red[e + 2 * n] + (double)red[e + 3 * n])) : red[e];
        dw[NHWC ? t * g.npairs + pr : pr * KK + t] = sum;
    }
}

bool short_geom(const GGeom &q, int layout, ShortGeom *g)
{
    const long long npix = (long long)q.N * q.Ho * q.Wo, npairs = (long long)q.O * q.Cg;
    if ((q.K != 3 && q.K != 5 && q.K != 7) || npix >= 1 << 21 || npairs >= 1 << 24) return false;
    *g = {q.C, q.H, q.W, q.s, q.p, q.O, q.Cg, q.Og, q.Ho, q.Wo, (int)npix, (int)npairs, 1, 0, 4, 1.0f / (float)q.Ho, 1.0f / (float)q.Wo};
    if (layout == LAYOUT_NCHW) {
        if (npix <= 64 || (npix <= 256 && npairs >= 1024)) g->ws = 1;
    } else {
        // four pairs of consecutive channels, more where that leaves blocks enough or positions for all lanes
        for (g->lcw = 2; g->lcw < 4 && npairs >> g->lcw > 512; ) ++g->lcw;
        while (g->lcw < 6 && 256 >> g->lcw > npix) ++g->lcw;
        g->cw = 1 << g->lcw;
    }
    return true;
}

template <typename T, int LAYOUT>
hipError_t short_go(const ShortGeom &g, int K, const void *x, const void *dy, float *dw, hipStream_t st)
{
    const int per = g.cw * (4 / g.ws);
    const unsigned blocks = (unsigned)((g.npairs + per - 1) / per), lds = (unsigned)(4 * K * K * g.cw * sizeof(float));
    auto kernel = K == 3 ? k_short_bwd_filter<T, LAYOUT, 3> : K == 5 ? k_short_bwd_filter<T, LAYOUT, 5> : k_short_bwd_filter<T, LAYOUT, 7>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), lds, st, g, (const T *)x, (const T *)dy, dw);
    return hipGetLastError();
}

}  // namespace

// Estimated time in us: the launch with the sums of a block, the rounds of a lane's loads, all loads of a compute unit, its blocks, and what the loads touch: NCHW
// the lines of a wavefront's positions in x (those of small or strided planes lie far apart), NHWC all of x, of which a block takes a part of every
// line.  Fitted to 110 000 random layers of up to 13 us: nine of ten between 0.9 and 1.1 times the measured time, one in a hundred
// longer by 1.25 (without the lines 1.3 to 1.5, and 2.2 in planes of 2 x 2 outputs).
static double short_us(const ShortGeom &g, int K, int layout, int dtype, double xelems)
{
    static const float fit[2][3][5] = {{{2.87f, 1.12f, 0.375f, 1.59f, 0.0168f}, {4.02f, 0.54f, 0.417f, 4.38f, 0.0457f}, {4.59f, 1.18f, 0.161f, 11.95f, 0.0802f}},
                                       {{2.92f, 1.14f, 0.669f, 0.45f, 0.68f}, {3.54f, 0.666f, 0.559f, 1.65f, 0.68f}, {5.25f, 1.92f, 0.f, 6.9f, 0.81f}}};
    const float *c = fit[layout == LAYOUT_NHWC][K / 2 - 1];
    const int U = K == 3 ? 2 : 1, step = (64 >> g.lcw) * g.ws * U, per = g.cw * (4 / g.ws), esz = dtype == DT_F32 ? 4 : 2;
    const double rounds = (g.npix + step - 1) / step, blocks = (g.npairs + per - 1) / per;
    double touched = xelems * esz * 1e-6;
    if (layout == LAYOUT_NCHW) {
        const double planes = 64.0 / ((double)g.Ho * g.Wo), lines = planes * g.H * g.W * esz / 128 + (planes > 1 ? planes : 1);
        touched = (blocks > 256 ? blocks / 256 : 1) * rounds * U * lines;
    }
    return c[0] + c[1] * rounds + c[2] * blocks * rounds * U * K * K / (256 * 64) + c[3] * blocks / 1024 + c[4] * touched;
}

// One launch of the generic kernels (a single partial, written where the gradient goes), fitted to 30 000 random layers: 0.9 to 1.3 of the time.
static double generic_one_us(const ShortGeom &g, int K, int layout)
{
    if (layout == LAYOUT_NCHW) {
        const double steps = (g.npix + 255) / 256, blocks = (double)g.npairs * K * K / 2048;
        return 3.2 + 0.29 * steps + blocks * (0.8 * steps + 1.0);
    }
    const double steps = (g.npix + 3) / 4, blocks = (double)((g.O + 63) / 64) * K * K * g.Cg / 2048;
    return 2.2 + 0.3 * steps + 0.53 * blocks * steps;
}

// Instead of two launches up to the estimates below, over 66 000 random layers in a loop of calls, in brackets the share longer by more than 8 %: 3x3 0.63 to
// 0.67 of the time [0.04 %], instead of the small-plane kernels, whose two launches take 5.6 us, 0.65 [0.1 %]; 5x5 NCHW 0.63 [0.2 %], small planes 0.72 [0 %], NHWC
// 0.56 and 0.70 [0.05 and 0.3 %]; 7x7 NCHW 0.75 [0.8 %], NHWC no shorter; instead of the matrix instructions 3x3 0.67 [0.1 %] and 0.61 [0.8 %], 5x5
// 0.67 [0.3 %] and 0.59 [0.8 %].  An estimate of half a us more is where 3 to 10 % are longer.  Instead of one launch of the generic
// kernels where its own estimate is that much below theirs: 0.40 to 0.73 of the time, 1 % longer.
bool short_bwd_filter_shorter(const GGeom &q, int layout, int dtype, FilterWay way)
{
    ShortGeom g;
    if (!short_geom(q, layout, &g)) return false;
    if (tune_active()) {                                         // forced tilings are those of the other kernels
        const char *e = tune_env("DWCONV_TUNE_SHORT");
        return e && atoi(e) != 0;
    }
    const bool nhwc = layout == LAYOUT_NHWC;
    const double us = short_us(g, q.K, layout, dtype, (double)q.N * q.C * q.H * q.W);
    switch (way) {
    case FILTER_GENERIC_ONE: return us < 0.85 * generic_one_us(g, q.K, layout);
    case FILTER_MATRIX: return us < (q.K == 3 ? (nhwc ? 8.0 : 10.0) : (nhwc ? 9.0 : 12.0));
    case FILTER_SMALL_PLANES: return us < (q.K == 3 ? 6.0 : 6.5);
    default: return us < (q.K == 3 ? 7.25 : q.K == 5 ? (nhwc ? 8.0 : 9.0) : (nhwc ? 0.0 : 11.0));
    }
}

hipError_t short_bwd_filter(const GGeom &q, int layout, int dtype, const void *x, const void *dy, float *dw, hipStream_t st)
{
    ShortGeom g;
    if (!short_geom(q, layout, &g)) return hipErrorInvalidValue;
    if (layout == LAYOUT_NCHW) return dtype == DT_F32 ? short_go<float, LAYOUT_NCHW>(g, q.K, x, dy, dw, st) : short_go<bf16_t, LAYOUT_NCHW>(g, q.K, x, dy, dw, st);
    return dtype == DT_F32 ? short_go<float, LAYOUT_NHWC>(g, q.K, x, dy, dw, st) : short_go<bf16_t, LAYOUT_NHWC>(g, q.K, x, dy, dw, st);
}

}  // namespace dwc

// Group convolution behind the C ABI (gconv_* in include/dwconv.h): argument validation, variant
// selection, and the generic kernels that are correct for any K, stride, pad and group size in both
// layouts and storage types (one thread per output element; not tuned).  Groups of one input channel
// are the depthwise layer and run on its kernels.
#include "../../include/dwconv.h"
#include "gconv.hpp"
#include "short_filter.hpp"
#include <math.h>

namespace dwc {

template <int LAYOUT>
__device__ __forceinline__ int gat(int CH, int HH, int WW, int n, int ch, int h, int w)
{
    if (LAYOUT == LAYOUT_NCHW) return ((n * CH + ch) * HH + h) * WW + w;
    return ((n * HH + h) * WW + w) * CH + ch;
}
// filter entry (o, ci, kh, kw): [O,Cg,K,K] or [K,K,Cg,O]
template <int LAYOUT>
__device__ __forceinline__ int gwat(const GGeom &g, int o, int ci, int kh, int kw)
{
    if (LAYOUT == LAYOUT_NCHW) return ((o * g.Cg + ci) * g.K + kh) * g.K + kw;
    return ((kh * g.K + kw) * g.Cg + ci) * g.O + o;
}
template <int LAYOUT>
__device__ __forceinline__ void gunflat(int idx, int CH, int HH, int WW, int &n, int &ch, int &h, int &w)
{
    if (LAYOUT == LAYOUT_NCHW) {
        w = idx % WW; idx /= WW; h = idx % HH; idx /= HH; ch = idx % CH; n = idx / CH;
    } else {
        ch = idx % CH; idx /= CH; w = idx % WW; idx /= WW; h = idx % HH; n = idx / HH;
    }
}

template <typename T, int LAYOUT>
__global__ __launch_bounds__(256) void k_gconv_generic_fwd(GGeom g, const T *__restrict__ x, const T *__restrict__ w,
                                                           T *__restrict__ y, int total)
{
    const unsigned uidx = blockIdx.x * 256u + threadIdx.x;   // the last block may reach past 2^31
    if (uidx >= (unsigned)total) return;
    int idx = (int)uidx;
    int n, o, oh, ow;
    gunflat<LAYOUT>(idx, g.O, g.Ho, g.Wo, n, o, oh, ow);
    const int c0 = (o / g.Og) * g.Cg;
    float acc = 0.f;
    for (int ci = 0; ci < g.Cg; ++ci)
        for (int kh = 0; kh < g.K; ++kh) {
            const int ih = oh * g.s - g.p + kh;
            if (ih < 0 || ih >= g.H) continue;
            for (int kw = 0; kw < g.K; ++kw) {
                const int iw = ow * g.s - g.p + kw;
                if (iw < 0 || iw >= g.W) continue;
                acc = fmaf(ldf(w + gwat<LAYOUT>(g, o, ci, kh, kw)), ldf(x + gat<LAYOUT>(g.C, g.H, g.W, n, c0 + ci, ih, iw)), acc);
            }
        }
    stf(y + idx, acc);
}

template <typename T, int LAYOUT>
__global__ __launch_bounds__(256) void k_gconv_generic_bwd_data(GGeom g, const T *__restrict__ dy,
                                                                const T *__restrict__ w, T *__restrict__ dx, int total)
{
    const unsigned uidx = blockIdx.x * 256u + threadIdx.x;   // the last block may reach past 2^31
    if (uidx >= (unsigned)total) return;
    int idx = (int)uidx;
    int n, c, ih, iw;
    gunflat<LAYOUT>(idx, g.C, g.H, g.W, n, c, ih, iw);
    const int o0 = (c / g.Cg) * g.Og, ci = c % g.Cg;
    float acc = 0.f;
    for (int oi = 0; oi < g.Og; ++oi) {
        const int o = o0 + oi;
        for (int kh = 0; kh < g.K; ++kh) {
            const int th = ih + g.p - kh;
            if (th < 0 || th % g.s != 0) continue;
            const int oh = th / g.s;
            if (oh >= g.Ho) continue;
            for (int kw = 0; kw < g.K; ++kw) {
                const int tw = iw + g.p - kw;
                if (tw < 0 || tw % g.s != 0) continue;
                const int ow = tw / g.s;
                if (ow >= g.Wo) continue;
                acc = fmaf(ldf(w + gwat<LAYOUT>(g, o, ci, kh, kw)), ldf(dy + gat<LAYOUT>(g.O, g.Ho, g.Wo, n, o, oh, ow)), acc);
            }
        }
    }
    stf(dx + idx, acc);
}

// Stage 1, NCHW: block (weight entry j = ((o*Cg+ci)*K+kh)*K+kw, part); threads stride over the pixels of
// the part; wavefront butterfly, then LDS across the 4 waves.
template <typename T>
__global__ __launch_bounds__(256) void k_gconv_generic_bwd_filter_nchw(GGeom g, const T *__restrict__ x,
                                                                       const T *__restrict__ dy, float *__restrict__ ws,
                                                                       int per_part, int J)
{
    __shared__ float red[4];
    const int j = blockIdx.x, part = blockIdx.y;
    const int kw = j % g.K, kh = (j / g.K) % g.K, ci = (j / (g.K * g.K)) % g.Cg, o = j / (g.K * g.K * g.Cg);
    const int c = (o / g.Og) * g.Cg + ci;
    const int npix = g.N * g.Ho * g.Wo;
    const int lo = part * per_part, hi = min(npix, lo + per_part);
    float acc = 0.f;
    for (int pix = lo + (int)threadIdx.x; pix < hi; pix += 256) {
        const int ow = pix % g.Wo, t = pix / g.Wo, oh = t % g.Ho, n = t / g.Ho;
        const int ih = oh * g.s - g.p + kh, iw = ow * g.s - g.p + kw;
        if (ih < 0 || ih >= g.H || iw < 0 || iw >= g.W) continue;
        acc = fmaf(ldf(dy + gat<LAYOUT_NCHW>(g.O, g.Ho, g.Wo, n, o, oh, ow)),
                   ldf(x + gat<LAYOUT_NCHW>(g.C, g.H, g.W, n, c, ih, iw)), acc);
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) ws[(size_t)part * J + j] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Stage 1, NHWC: block (tile of 64 output channels x one (kh,kw,ci), part); lane = channel, the 4 waves
// stride over pixels; LDS across the waves.
template <typename T>
__global__ __launch_bounds__(256) void k_gconv_generic_bwd_filter_nhwc(GGeom g, const T *__restrict__ x,
                                                                       const T *__restrict__ dy, float *__restrict__ ws,
                                                                       int per_part, int J, int notiles)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int otile = blockIdx.x % notiles, e = blockIdx.x / notiles;     // e = (kh*K + kw)*Cg + ci
    const int part = blockIdx.y;
    const int ci = e % g.Cg, kw = (e / g.Cg) % g.K, kh = e / (g.Cg * g.K);
    const int o = otile * 64 + lane;
    const int npix = g.N * g.Ho * g.Wo;
    const int lo = part * per_part, hi = min(npix, lo + per_part);
    float acc = 0.f;
    if (o < g.O) {
        const int c = (o / g.Og) * g.Cg + ci;
        for (int pix = lo + wv; pix < hi; pix += 4) {
            const int ow = pix % g.Wo, t = pix / g.Wo, oh = t % g.Ho, n = t / g.Ho;
            const int ih = oh * g.s - g.p + kh, iw = ow * g.s - g.p + kw;
            if (ih < 0 || ih >= g.H || iw < 0 || iw >= g.W) continue;
            acc = fmaf(ldf(dy + (size_t)pix * g.O + o), ldf(x + gat<LAYOUT_NHWC>(g.C, g.H, g.W, n, c, ih, iw)), acc);
        }
    }
    red[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && o < g.O)
        ws[(size_t)part * J + (size_t)e * g.O + o] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

hipError_t gconv_generic_fwd(const GGeom &g, int layout, int dtype, const void *x, const void *w, void *y, hipStream_t st)
{
    const int total = g.N * g.O * g.Ho * g.Wo;
    dim3 grid((unsigned)(((long long)total + 255) / 256)), block(256);
#define LAUNCH(T, L) hipLaunchKernelGGL((k_gconv_generic_fwd<T, L>), grid, block, 0, st, g, (const T *)x, (const T *)w, (T *)y, total)
    if (dtype == DT_F32) { if (layout == LAYOUT_NCHW) LAUNCH(float, LAYOUT_NCHW); else LAUNCH(float, LAYOUT_NHWC); }
    else                 { if (layout == LAYOUT_NCHW) LAUNCH(bf16_t, LAYOUT_NCHW); else LAUNCH(bf16_t, LAYOUT_NHWC); }
#undef LAUNCH
    return hipGetLastError();
}

hipError_t gconv_generic_bwd_data(const GGeom &g, int layout, int dtype, const void *dy, const void *w, void *dx,
                                  hipStream_t st)
{
    const int total = g.N * g.C * g.H * g.W;
    dim3 grid((unsigned)(((long long)total + 255) / 256)), block(256);
#define LAUNCH(T, L) hipLaunchKernelGGL((k_gconv_generic_bwd_data<T, L>), grid, block, 0, st, g, (const T *)dy, (const T *)w, (T *)dx, total)
    if (dtype == DT_F32) { if (layout == LAYOUT_NCHW) LAUNCH(float, LAYOUT_NCHW); else LAUNCH(float, LAYOUT_NHWC); }
    else                 { if (layout == LAYOUT_NCHW) LAUNCH(bf16_t, LAYOUT_NCHW); else LAUNCH(bf16_t, LAYOUT_NHWC); }
#undef LAUNCH
    return hipGetLastError();
}

int gconv_generic_bwd_filter_parts(const GGeom &g)
{
    // about 8192 pixels per part, at most 64 parts (the launch's second grid dimension), and never more
    // than 32 MiB of partials
    const long long npix = (long long)g.N * g.Ho * g.Wo;
    long long parts = (npix + 8191) / 8192;
    if (parts > 64) parts = 64;
    const long long J = (long long)g.O * g.Cg * g.K * g.K;
    while (parts > 1 && parts * J * 4 > (32ll << 20)) parts >>= 1;
    if (parts < 1) parts = 1;
    return (int)parts;
}

hipError_t gconv_generic_bwd_filter(const GGeom &g, int layout, int dtype, const void *x, const void *dy, float *ws,
                                    int parts, hipStream_t st)
{
    const int npix = g.N * g.Ho * g.Wo;
    const int per_part = (npix + parts - 1) / parts;
    const int J = g.O * g.Cg * g.K * g.K;
    if (layout == LAYOUT_NCHW) {
        dim3 grid(J, parts), block(256);
        if (dtype == DT_F32)
            hipLaunchKernelGGL(k_gconv_generic_bwd_filter_nchw<float>, grid, block, 0, st, g, (const float *)x, (const float *)dy, ws, per_part, J);
        else
            hipLaunchKernelGGL(k_gconv_generic_bwd_filter_nchw<bf16_t>, grid, block, 0, st, g, (const bf16_t *)x, (const bf16_t *)dy, ws, per_part, J);
    } else {
        const int notiles = (g.O + 63) / 64;
        dim3 grid(notiles * g.K * g.K * g.Cg, parts), block(256);
        if (dtype == DT_F32)
            hipLaunchKernelGGL(k_gconv_generic_bwd_filter_nhwc<float>, grid, block, 0, st, g, (const float *)x, (const float *)dy, ws, per_part, J, notiles);
        else
            hipLaunchKernelGGL(k_gconv_generic_bwd_filter_nhwc<bf16_t>, grid, block, 0, st, g, (const bf16_t *)x, (const bf16_t *)dy, ws, per_part, J, notiles);
    }
    return hipGetLastError();
}

// ---- variant selection -------------------------------------------------------------------------------

// the same tensor shapes as a depthwise geometry (for the kernels shared with the depthwise layer; C == O)
static Geom as_geom(const GGeom &g)
{
    Geom q;
    q.N = g.N; q.C = g.C; q.H = g.H; q.W = g.W; q.K = g.K; q.s = g.s; q.p = g.p; q.m = 1; q.O = g.O; q.Ho = g.Ho; q.Wo = g.Wo;
    return q;
}

// Estimated time in us of the generic kernels.  Forward and input gradient: a lane's products one after the other, or all of them at a rate that
// is higher for larger filters and lower where the stride skips taps or lines; the filter gradient: blocks of (entry, part), each as
// long as its lanes' pixels.  Fitted to 30 000 random layers: four of five between 0.65 and 1.2 times the measured time.
static double generic_us(const GGeom &g, int layout, int pass)
{
    const bool nhwc = layout == LAYOUT_NHWC, strided = g.s > 1;
    if (pass == 2) {
        const double J = (double)g.O * g.Cg * g.K * g.K, pixels = (double)g.N * g.Ho * g.Wo, parts = gconv_generic_bwd_filter_parts(g);
        if (!nhwc) {
            const double steps = ceil(pixels / parts / 256), blocks = J * parts / 2048;
            return 6 + 0.29 * steps + blocks * (0.8 * steps + 1.0);
        }
        const double steps = ceil(pixels / parts / 4), blocks = (double)((g.O + 63) / 64) * g.K * g.K * g.Cg * parts / 2048;
        return 4.6 + 0.3 * steps + 0.53 * blocks * steps + 20e-6 * parts * J;
    }
    // rows (columns) of the filter that an output needs, or that the outputs of a wavefront need between them: the others of its lanes wait
    // for each; in NHWC they are channels of one pixel
    const bool together = !nhwc || (pass == 0 ? g.O : g.C) < 64;
    auto taps = [&](long long n, int in, int out) { n = together ? in + (out - 1LL) * g.s : n; return (double)(n < g.K ? n : g.K); };
    double products, latency, rate, outputs;                     // products of an output; M products in a us
    if (pass == 0) {
        products = g.Cg * taps(g.H, g.H, g.Ho) * taps(g.W, g.W, g.Wo);
        outputs = (double)g.N * g.O * g.Ho * g.Wo;
        latency = 4 + 0.15 * products;
        rate = (g.K == 1 ? 1.0 : g.K == 3 ? 1.95 : 2.3) * (strided ? 0.7 : 1.0);
    } else {
        const bool skips = nhwc && strided && g.K > 1;
        products = g.Og * taps((long long)g.Ho * g.s, g.H, g.Ho) * taps((long long)g.Wo * g.s, g.W, g.Wo);
        outputs = (double)g.N * g.C * g.H * g.W;
        latency = 4.3 + (skips ? 0.13 : 0.23) * products;
        rate = (g.K == 1 ? 0.6 : g.K == 3 ? 1.05 : 1.2) * (skips ? 1.8 : nhwc && g.K == 3 ? 0.65 : 1.0);
    }
    const double all = outputs * products * 1e-6 / rate;
    return sqrt(latency * latency + all * all);
}

// Laying out the filter and staging a tile are a fixed 5 to 12 us, and a filter that takes the LDS leaves small tiles: few products per output
// and few outputs, or few channels a group with a large filter, are shorter one output per thread.  Where the two are close, the estimate of the latter is a fifth above
// the measured time below 10 us and a sixth to a quarter below it from 20 us on (medians), hence the line.  Over 24 000 random layers 0.25 % of the forward passes and 0.16 % of the
// input gradients that go here are longer by more than 8 % than one output per thread, 6 and 17 % of the 900 and 450 that stay would be shorter here by as much, and
// the time is 1.002 of the shorter of the two throughout.  (0.95 of the estimate less 1 and 0.7 us: 0.05 and 0.08, 13 and 22 %, 1.003, and
// 149x18x35x32 in nine groups, 5x5, fp32 NHWC, 95 us in place of 57.)  Two kinds have a line of their own, over layers between it and the common one: NCHW input gradients of 2x2 filters and larger, of 4000
// layers 608 + 88 (fp32, bf16) longer here by more than 8 % with 1.3, 7 + 0 with 1.25, and 61 that stay would be shorter here by as much; NCHW 7x7 forward in fp32, of 1600 570
// with 1.3, 98 with 1.1, and 153 (48x103x103 in 16 groups, 30 us generic, 42 here).  The filter gradient, whose
// time here hardly depends on the layer as long as it is short: 1 % either way.
static bool gemm_over_generic(const GGeom &g, int layout, int dtype, int pass, GemmPlan *pl)
{
    const double generic = generic_us(g, layout, pass);
    if (pass == 2) return generic > (g.K == 1 ? 10.5 : g.K == 3 ? 12.5 : 16.0) && gconv_gemm_plan(g, layout, dtype, pass, pl);
    const double line = layout == LAYOUT_NHWC ? 1.3 : pass == 1 && g.K > 1 ? 1.25 : g.K == 7 && pass == 0 && dtype == DT_F32 ? 1.1 : 1.3;
    return gconv_gemm_plan(g, layout, dtype, pass, pl) && gconv_gemm_us(*pl, layout, dtype) < line * generic - 3.2;
}

// In place of the NCHW row walk: in fp32 not for the filter gradient of 16 channels a group on many pixels (1.03 times as long at the median of
// random layers, up to 1.8).  Forward and input gradient by the estimates of both: of 440 random layers of 16 to 64 channels a group none is longer here by
// more than 8 %, of 350 of 80 to 160 on many pixels 0.6 to 1.7 % (always here: 5 to 10 %, up to 2.4 times), and none stays that would be shorter.  us, row walk ->
// here: 128x21x20 in two groups, batch 148, 251 -> 146; 1024x18x18 in 16, batch 128, 964 -> 690; 480x18x18 in five, batch 213, 1080 -> 2330: stays.
static bool gemm_over_rowwalk(const GGeom &g, int layout, int dtype, int pass, GemmPlan *pl)
{
    if (dtype == DT_F32 && pass == 2 && g.Cg == 16 && (long long)g.N * g.Ho * g.Wo >= 16384) return false;
    if (!gconv_gemm_plan(g, layout, dtype, pass, pl)) return false;
    return dtype != DT_F32 || pass == 2 || gconv_gemm_us(*pl, layout, dtype) * (g.Cg > 64 ? 0.85 : 0.7) < gconv_nchw_s1_us(g, pass == 1);
}

// In place of the other row walks, whose lanes are few in short launches (a lane walks 7 to 28 rows of all its group's input channels) and, NHWC with eight channels
// a group, many registers; in bf16 they widen every value.  Measured over 13 000 random layers of 2 to 64 channels a group, up to 120 M outputs in bf16, walk
// against these, the share in brackets longer by more than 8 %.  NCHW forward and input gradient: bf16 of eight channels 0.2 up to 0.7 at 120 M [0.3 %], of
// 3 to 5 0.45 up to 0.8 at 8 M [1 %], from 16 M on 0.98 to 1.15 [40 to 50 %, up to 2.3 times: 0.8 in rows of 16, 1.2 in rows of 60 and more], of two 0.6 to 0.9 up to
// 2 M, 1.0 at 3 M [20 %]; fp32 0.2 to 0.7 up to 2 M, of two channels up to 0.5 M, of others that the walk takes one output at a time (3, 5, 6, 10) up to 1 M, above those
// 0.9 to 2.  Filter gradient: bf16 0.57 to 0.8, of fewer than six channels from 16 M on 0.93 to 1.2 [22 to 72 %], of odd groups, whose walk takes one output channel at
// a time, 1.0 to 1.2 throughout, fp32 with four output channels at a time 0.63 to 0.87 up to 0.7 M [1 %], 0.92 at 1 M [8 %], then 1.06 to 1.25.  NHWC forward and input gradient with
// eight channels 0.4 to 0.87 in bf16, 0.7 to 0.83 in fp32 from 0.3 to 2.7 M; with two and four 0.8 to 1.8 and 1.0 to 2.5: they stay.  NHWC filter gradient in bf16 of
// four and eight 0.4 to 0.75 throughout, of two channels a group only where the walk's lanes are few: up to 32 channels in all and 3 M outputs 0.65 to 0.82 [1 %], 0.98 at 8 M
// [11 %], 1.1 to 1.35 above [50 %]; at stride 2 of eight 0.65 to 0.8, of four 0.72 to 0.85 from 0.1 to 1 M [5 %], 0.9 below [32 %]; fp32 with eight channels 0.8 to 0.86 up to 0.7 M
// [2 %], 0.93 at 0.9 M [10 %], 1.06 to 1.12 above.
static bool gemm_over_walk(const GGeom &g, int dtype, int pass, int variant, long long outputs)
{
    const bool f32 = dtype == DT_F32;
    if (tune_active()) return false;                             // forced tilings are those of the walks
    if (variant == GV_NCHW_K3S1) {
        // (16 output channels at a time, whether there are or not: 48x46x64 of four channels in two groups, fp32 10.5 on the walk, 15.9 here; 48x48x4 of two,
        // bf16 batch 202, input gradient 10.9 and 16.5.  In bf16, of 30 000 layers below the lines on outputs: two channels a group with 3.5 M padded outputs and more
        // 1.2 and 1.3 times as long here, forward and input gradient; three from 6 M on 0.96 and 1.0, up to 2.5 and 2.7; four from 8 M on 1.01 and 1.07)
        const long long padded = outputs / (pass == 1 ? g.C : g.O) * (((pass == 1 ? g.C : g.O) + 15) / 16 * 16);
        const int few = g.Cg < g.Og ? g.Cg : g.Og;
        const bool whole = g.Cg % 4 == 0 && g.Og % 4 == 0;       // the walk takes four output channels at a time
        if (pass < 2 && f32) return padded < (few == 2 ? 500000 : whole ? 2000000 : 1000000);
        if (pass < 2) return few == 2 ? outputs < 2000000 && padded < 3500000 : few < 6 ? padded < (few == 3 ? 6000000 : 8000000) : outputs < 1ll << 31;
        return g.Og % 4 == 0 || (!f32 && g.Og % 2 == 0 && g.Cg >= 6) ? outputs < (f32 ? 700000 : few < 6 ? 8000000 : 1ll << 31) : false;
    }
    if (variant == GV_NHWC_K3S1) {
        if (pass < 2) {
            // (a quarter of the output channels or more beside the tensor, on planes that are most of a tile: 24 channels in three groups, 4x4 to 6x6, 4.1 to 5.1 us on the
            // walk, 4.8 to 5.8 here; 13 % of such layers were longer by more than 8 %)
            if ((g.C + 15) / 16 * 16 * 3 >= g.C * 4 && g.H * g.W <= 36) return false;
            return g.Cg == 8 && g.Og == 8 && !gconv_nhwc_mfma_supported(g, dtype) && (!f32 || (outputs >= 300000 && outputs < 2700000));
        }
        return f32 ? g.Cg == 8 && outputs < 700000 : g.Cg > 2 || (g.C <= 32 && outputs < 3000000);
    }
    if (variant == GV_NHWC_BWD_FILTER_S2) return !f32 && (g.Cg == 8 ? outputs >= 8192 : g.C <= 64 && outputs >= 100000 && outputs < 1000000);
    return false;
}

static GPlan gplan(const GGeom &g, int layout, int dtype, int pass)
{
    GPlan pl = {GV_GENERIC, pass == 2 ? gconv_generic_bwd_filter_parts(g) : 0, 0, 0, 0, "group_generic", {}};
    if (tune_env("DWCONV_TUNE_GROUP_GENERIC")) return pl;
    // The filter gradient takes the small-plane form for groups of up to 4 on rows of up to 14, and on 28-wide rows in
    // bf16 (fp32 batch 128: 14x14 groups of 4 37 against 55 us, 28x28 groups of 4 83 against 85, groups of 8 122 against
    // 103; bf16 batch 256: 48 against 95, 83 against 107, 166 against 160)
    // Rows the row-walk kernels cannot take (7 elements) always go to the small-plane form instead of the generic one.
    const bool small_ok = pass < 2 || (g.Cg <= 4 && (g.W <= 14 || dtype == DT_BF16)) || !gconv_nchw_supported(g);      // (stride 2: always)
    if (layout == LAYOUT_NCHW && pass < 2 && gconv_nchws_mfma_fwd_supported(g)) {
        pl.variant = GV_NCHWS_MFMA_FWD;
        pl.name = pass == 0 ? "group_nchw_smallplane_mfma_k3s1" : "group_nchw_smallplane_mfma_k3s1_flip";
    } else if (layout == LAYOUT_NCHW && pass == 2 && gconv_nchws_mfma_bwd_filter_supported(g, dtype, false)) {
        pl.variant = GV_NCHWS_MFMA_BWD_FILTER;
        pl.name = "group_nchw_smallplane_mfma_bwd_filter_k3s1";
        pl.parts = gconv_nchws_mfma_bwd_filter_parts(g, dtype);
    } else if (layout == LAYOUT_NCHW && g.Cg == g.Og && small_ok && nchws_group_supported(as_geom(g), g.Cg) &&
        !tune_env("DWCONV_TUNE_GNOSMALL")) {
        // small planes (rows of 7, 14 or 28): whole groups staged in LDS through flat 16-byte accesses
        pl.variant = GV_NCHWS_K3S1;
        if (g.s == 1)
            pl.name = pass == 0 ? "group_nchw_smallplane_k3s1" : pass == 1 ? "group_nchw_smallplane_k3s1_flip"
                                                                            : "group_nchw_smallplane_bwd_filter_k3s1";
        else
            pl.name = pass == 0 ? "group_nchw_smallplane_fwd_k3s2" : pass == 1 ? "group_nchw_smallplane_bwd_data_k3s2"
                                                                               : "group_nchw_smallplane_bwd_filter_k3s2";
        if (pass == 2) nchws_bwd_filter_tiling(as_geom(g), dtype, &pl.a, &pl.c, &pl.parts, g.Cg);
    } else if (layout == LAYOUT_NCHW && gconv_nchw_supported(g)) {
        pl.variant = GV_NCHW_K3S1;
        pl.name = pass == 0 ? "group_nchw_rowwalk_k3s1" : pass == 1 ? "group_nchw_rowwalk_k3s1_flip" : "group_nchw_bwd_filter_k3s1";
        if (pass == 2) pl.parts = gconv_nchw_bwd_filter_parts(g);
    } else if (layout == LAYOUT_NHWC && pass == 2 && gconv_nchws_mfma_bwd_filter_supported(g, dtype, true)) {
        pl.variant = GV_NHWC_LDS_MFMA_BWD_FILTER;
        pl.name = "group_nhwc_lds_mfma_bwd_filter_k3s1";
        pl.parts = gconv_nchws_mfma_bwd_filter_parts(g, dtype);
    } else if (layout == LAYOUT_NHWC && pass == 2 && gconv_nhwc_tr_bwd_filter_supported(g, dtype)) {
        pl.variant = GV_NHWC_TR_BWD_FILTER;
        pl.name = "group_nhwc_mfma_bwd_filter_k3s1";
        pl.parts = gconv_nhwc_tr_bwd_filter_parts(g, dtype);
    } else if (layout == LAYOUT_NHWC && pass < 2 && gconv_nhwc_mfma_s2_supported(g, dtype, pass)) {
        pl.variant = GV_NHWC_MFMA_S2;
        pl.name = pass == 0 ? "group_nhwc_mfma_fwd_k3s2" : "group_nhwc_mfma_bwd_data_k3s2";
    } else if (layout == LAYOUT_NHWC && pass == 2 && gconv_nhwc_bwd_filter_s2_supported(g)) {
        pl.variant = GV_NHWC_BWD_FILTER_S2;
        pl.name = "group_nhwc_bwd_filter_k3s2";
        pl.parts = gconv_nhwc_bwd_filter_s2_parts(g);
    } else if (layout == LAYOUT_NHWC && gconv_nhwc_supported(g)) {
        pl.variant = GV_NHWC_K3S1;
        const bool mm = pass < 2 && gconv_nhwc_mfma_supported(g, dtype);      // forward and backward-data on the matrix cores
        pl.name = pass == 0 ? (mm ? "group_nhwc_mfma_k3s1" : "group_nhwc_rowwalk_k3s1")
                : pass == 1 ? (mm ? "group_nhwc_mfma_k3s1_flip" : "group_nhwc_rowwalk_k3s1_flip") : "group_nhwc_bwd_filter_k3s1";
        if (pass == 2) pl.parts = gconv_nhwc_bwd_filter_parts(g, dtype);
    }
    // the one-launch filter gradient in place of two; a walk's line is below that of the kernels that may take its place, so it is asked first
    auto short_one = [&](FilterWay way) {
        if (pass != 2 || pl.variant == GV_NCHWS_MFMA_BWD_FILTER || !short_bwd_filter_shorter(g, layout, dtype, way)) return false;
        pl.variant = GV_SHORT_BWD_FILTER; pl.parts = 1;
        pl.name = layout == LAYOUT_NCHW ? "group_nchw_short_bwd_filter" : "group_nhwc_short_bwd_filter";
        return true;
    };
    const bool shorter = pl.variant != GV_GENERIC && short_one(pl.variant == GV_NCHWS_K3S1 ? FILTER_SMALL_PLANES : FILTER_TWO);
    // What no kernel above takes, and NCHW groups of a multiple of 16 channels in place of the row walk (14x14, 16 channels a
    // group, 512 channels, fp32 batch 64: 62 -> 45 us; 32 channels at batch 4: 53 -> 15): the 16x16 matrix instructions
    const bool rowwalk16 = pl.variant == GV_NCHW_K3S1 && g.Cg % 16 == 0 && g.Og % 16 == 0;
    const long long outputs = (long long)g.N * (pass == 1 ? (long long)g.C * g.H * g.W : (long long)g.O * g.Ho * g.Wo);
    // (fewer outputs: only of many products, which a lane of the generic kernels adds up one after the other: 4x4x96 in three groups, 5x5, 99 us)
    const bool enough = outputs >= 2048 || (pl.variant == GV_GENERIC && (pass == 1 ? g.Og : g.Cg) * g.K * g.K >= 256);
    bool walk = false;
    auto gemm = [&]() {
        if (shorter || !enough) return false;
        if ((pl.variant == GV_GENERIC || rowwalk16) && tune_env("DWCONV_TUNE_GROUP_GEMM")) return gconv_gemm_plan(g, layout, dtype, pass, &pl.gemm);
        if (pl.variant == GV_GENERIC) return gemm_over_generic(g, layout, dtype, pass, &pl.gemm);
        if (rowwalk16) return gemm_over_rowwalk(g, layout, dtype, pass, &pl.gemm);
        walk = gemm_over_walk(g, dtype, pass, pl.variant, outputs);
        return walk && gconv_gemm_plan(g, layout, dtype, pass, &pl.gemm);
    };
    if (gemm()) {
        pl.variant = GV_GEMM;
        pl.name = pass == 0 ? "group_mfma16" : pass == 1 ? "group_mfma16_bwd_data" : "group_mfma16_bwd_filter";
        if (pass == 2) { pl.parts = pl.gemm.nparts; pl.a = walk; }
        short_one(FILTER_MATRIX);
    } else if (pl.variant == GV_GENERIC) short_one(pl.parts == 1 ? FILTER_GENERIC_ONE : FILTER_TWO);
    // a tuned filter gradient whose partial sums would not fit in 64 MiB (very wide rows): the generic kernels
    if (pass == 2 && pl.variant != GV_GENERIC && (long long)pl.parts * g.O * g.Cg * g.K * g.K * 4 > (64ll << 20)) {
        const GPlan gen = {GV_GENERIC, gconv_generic_bwd_filter_parts(g), 0, 0, 0, "group_generic", {}};
        return gen;
    }
    return pl;
}

}  // namespace dwc

using namespace dwc;

static int gvalidate(const dwconv_group_desc *d, GGeom *g)
{
    if (!d) return DWCONV_ERR_NULL;
    if (d->layout != DWCONV_NCHW && d->layout != DWCONV_NHWC) return DWCONV_ERR_BAD_ENUM;
    if (d->dtype != DWCONV_F32 && d->dtype != DWCONV_BF16) return DWCONV_ERR_BAD_ENUM;
    if (d->N < 1 || d->C < 1 || d->H < 1 || d->W < 1 || d->K < 1 || d->stride < 1 || d->pad < 0 || d->groups < 1 ||
        d->O < 1)
        return DWCONV_ERR_BAD_DIM;
    if (d->C % d->groups != 0 || d->O % d->groups != 0) return DWCONV_ERR_BAD_DIM;
    if (d->K > DWCONV_MAX_K) return DWCONV_ERR_UNSUPPORTED;
    const long long sh = (long long)d->H + 2ll * d->pad - d->K, sw = (long long)d->W + 2ll * d->pad - d->K;
    if (sh < 0 || sw < 0) return DWCONV_ERR_BAD_DIM;
    const long long Ho = sh / d->stride + 1, Wo = sw / d->stride + 1;
    const long long lim = 1ll << 31;
    const long long Cg = d->C / d->groups;
    if ((long long)d->pad >= (1 << 20) || (long long)d->N * d->C * d->H * d->W >= lim ||
        (long long)d->N * d->O * Ho * Wo >= lim || (long long)d->O * Cg * d->K * d->K >= lim)
        return DWCONV_ERR_TOO_LARGE;
    if (g) {
        g->N = d->N; g->C = d->C; g->H = d->H; g->W = d->W;
        g->K = d->K; g->s = d->stride; g->p = d->pad;
        g->G = d->groups; g->O = d->O; g->Cg = (int)Cg; g->Og = d->O / d->groups;
        g->Ho = (int)Ho; g->Wo = (int)Wo;
    }
    return DWCONV_OK;
}

// one input channel per group: the depthwise layer with multiplier O/C
static inline dwconv_desc as_depthwise(const dwconv_group_desc *d)
{
    dwconv_desc q = {d->N, d->C, d->H, d->W, d->K, d->stride, d->pad, d->O / d->C, d->layout, d->dtype};
    return q;
}

static inline bool gmisaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

extern "C" {

int gconv_out_dims(const dwconv_group_desc *desc, int32_t *Ho, int32_t *Wo)
{
    GGeom g;
    const int rc = gvalidate(desc, &g);
    if (rc != DWCONV_OK) return rc;
    if (Ho) *Ho = g.Ho;
    if (Wo) *Wo = g.Wo;
    return DWCONV_OK;
}

size_t gconv_bwd_filter_workspace_bytes(const dwconv_group_desc *desc)
{
    GGeom g;
    if (gvalidate(desc, &g) != DWCONV_OK) return 0;
    if (g.Cg == 1) {
        const dwconv_desc q = as_depthwise(desc);
        return dwconv_bwd_filter_workspace_bytes(&q);
    }
    const GPlan pl = gplan(g, desc->layout, desc->dtype, 2);
    return (size_t)pl.parts * (size_t)g.O * g.Cg * g.K * g.K * sizeof(float);
}

int gconv_fwd(const dwconv_group_desc *desc, const void *x, const void *w, void *y, void *stream)
{
    GGeom g;
    const int rc = gvalidate(desc, &g);
    if (rc != DWCONV_OK) return rc;
    if (g.Cg == 1) {
        const dwconv_desc q = as_depthwise(desc);
        return dwconv_fwd(&q, x, w, y, stream);
    }
    if (!x || !w || !y) return DWCONV_ERR_NULL;
    if (gmisaligned(x) || gmisaligned(w) || gmisaligned(y)) return DWCONV_ERR_ALIGN;
    const GPlan pl = gplan(g, desc->layout, desc->dtype, 0);
    hipError_t e;
    if (pl.variant == GV_NCHWS_MFMA_FWD) e = gconv_nchws_mfma_fwd(g, desc->dtype, x, w, y, false, (hipStream_t)stream);
    else if (pl.variant == GV_NCHWS_K3S1) e = nchws_group_fwd(as_geom(g), g.Cg, desc->dtype, x, w, y, false, (hipStream_t)stream);
    else if (pl.variant == GV_NCHW_K3S1) e = gconv_nchw_s1(g, desc->dtype, x, w, y, false, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_K3S1) e = gconv_nhwc_s1(g, desc->dtype, x, w, y, false, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_MFMA_S2) e = gconv_nhwc_mfma_s2(g, desc->dtype, x, w, y, false, (hipStream_t)stream);
    else if (pl.variant == GV_GEMM) e = gconv_gemm(pl.gemm, desc->layout, desc->dtype, x, w, y, (hipStream_t)stream);
    else e = gconv_generic_fwd(g, desc->layout, desc->dtype, x, w, y, (hipStream_t)stream);
    return e == hipSuccess ? DWCONV_OK : DWCONV_ERR_LAUNCH;
}

int gconv_bwd_data(const dwconv_group_desc *desc, const void *dy, const void *w, void *dx, void *stream)
{
    GGeom g;
    const int rc = gvalidate(desc, &g);
    if (rc != DWCONV_OK) return rc;
    if (g.Cg == 1) {
        const dwconv_desc q = as_depthwise(desc);
        return dwconv_bwd_data(&q, dy, w, dx, stream);
    }
    if (!dy || !w || !dx) return DWCONV_ERR_NULL;
    if (gmisaligned(dy) || gmisaligned(w) || gmisaligned(dx)) return DWCONV_ERR_ALIGN;
    const GPlan pl = gplan(g, desc->layout, desc->dtype, 1);
    hipError_t e;
    if (pl.variant == GV_NCHWS_MFMA_FWD) e = gconv_nchws_mfma_fwd(g, desc->dtype, dy, w, dx, true, (hipStream_t)stream);
    else if (pl.variant == GV_NCHWS_K3S1 && g.s == 2) e = nchws_group_bwd_data_s2(as_geom(g), g.Cg, desc->dtype, dy, w, dx, (hipStream_t)stream);
    else if (pl.variant == GV_NCHWS_K3S1) e = nchws_group_fwd(as_geom(g), g.Cg, desc->dtype, dy, w, dx, true, (hipStream_t)stream);
    else if (pl.variant == GV_NCHW_K3S1) e = gconv_nchw_s1(g, desc->dtype, dy, w, dx, true, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_K3S1) e = gconv_nhwc_s1(g, desc->dtype, dy, w, dx, true, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_MFMA_S2) e = gconv_nhwc_mfma_s2(g, desc->dtype, dy, w, dx, true, (hipStream_t)stream);
    else if (pl.variant == GV_GEMM) e = gconv_gemm(pl.gemm, desc->layout, desc->dtype, dy, w, dx, (hipStream_t)stream);
    else e = gconv_generic_bwd_data(g, desc->layout, desc->dtype, dy, w, dx, (hipStream_t)stream);
    return e == hipSuccess ? DWCONV_OK : DWCONV_ERR_LAUNCH;
}

int gconv_bwd_filter(const dwconv_group_desc *desc, const void *x, const void *dy, void *dw, void *workspace,
                     size_t workspace_bytes, void *stream)
{
    GGeom g;
    const int rc = gvalidate(desc, &g);
    if (rc != DWCONV_OK) return rc;
    if (g.Cg == 1) {
        const dwconv_desc q = as_depthwise(desc);
        return dwconv_bwd_filter(&q, x, dy, dw, workspace, workspace_bytes, stream);
    }
    if (!x || !dy || !dw) return DWCONV_ERR_NULL;
    if (gmisaligned(x) || gmisaligned(dy) || gmisaligned(dw)) return DWCONV_ERR_ALIGN;
    const GPlan pl = gplan(g, desc->layout, desc->dtype, 2);
    const int J = g.O * g.Cg * g.K * g.K;
    const size_t need = (size_t)pl.parts * (size_t)J * sizeof(float);
    if (!workspace || workspace_bytes < need) return DWCONV_ERR_WORKSPACE;
    if (gmisaligned(workspace)) return DWCONV_ERR_ALIGN;
    hipError_t e;
    const bool final = pl.parts == 1 && pl.variant != GV_GEMM;             // a kernel without products of padding: its sums are the gradient
    if (final) workspace = dw;
    if (pl.variant == GV_SHORT_BWD_FILTER) e = short_bwd_filter(g, desc->layout, desc->dtype, x, dy, (float *)workspace, (hipStream_t)stream);
    else if (pl.variant == GV_NCHWS_K3S1) e = nchws_group_bwd_filter(as_geom(g), g.Cg, desc->dtype, x, dy, (float *)workspace, pl.a, pl.c, (hipStream_t)stream);
    else if (pl.variant == GV_NCHWS_MFMA_BWD_FILTER) e = gconv_nchws_mfma_bwd_filter(g, desc->dtype, false, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_TR_BWD_FILTER) e = gconv_nhwc_tr_bwd_filter(g, desc->dtype, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_LDS_MFMA_BWD_FILTER) e = gconv_nchws_mfma_bwd_filter(g, desc->dtype, true, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_BWD_FILTER_S2) e = gconv_nhwc_bwd_filter_s2(g, desc->dtype, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_NCHW_K3S1) e = gconv_nchw_bwd_filter(g, desc->dtype, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_NHWC_K3S1) e = gconv_nhwc_bwd_filter(g, desc->dtype, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    else if (pl.variant == GV_GEMM) e = gconv_gemm_bwd_filter(pl.gemm, desc->layout, desc->dtype, x, dy, (float *)workspace, (hipStream_t)stream);
    else e = gconv_generic_bwd_filter(g, desc->layout, desc->dtype, x, dy, (float *)workspace, pl.parts, (hipStream_t)stream);
    if (final || e != hipSuccess) return e == hipSuccess ? DWCONV_OK : DWCONV_ERR_LAUNCH;
    if (pl.variant == GV_GEMM) {
        FilterGradSrc src = {x, dy, desc->dtype, desc->layout, g.N, g.C, g.H, g.W, g.K, g.s, g.p, g.O, g.Cg, g.Og, g.Ho, g.Wo};
        gconv_gemm_filter_tiles(pl.gemm, &src);
        // (in place of a walk a partial is a longer chain of sums than the walks', 1.01 to 1.03 times their error against 64 bits in bf16, 1.09 in
        // fp32 NHWC; with the partials in 64 bits 0.69 to 0.82 and 0.84 to 0.93, in the same time.  Up to 16 384 entries that is as short as 32 bits or shorter, from there on
        // 0.2 us a launch longer (74 000 entries 4.2 -> 4.4), which the others need not pay.)
        e = reduce_partials((const float *)workspace, pl.parts, J, (float *)dw, src, pl.a != 0 || J < 16384, (hipStream_t)stream);
    } else e = reduce_partials((const float *)workspace, pl.parts, J, (float *)dw, (hipStream_t)stream);
    return e == hipSuccess ? DWCONV_OK : DWCONV_ERR_LAUNCH;
}

const char *gconv_variant_name(const dwconv_group_desc *desc, int pass)
{
    GGeom g;
    if (gvalidate(desc, &g) != DWCONV_OK || pass < 0 || pass > 2) return "invalid";
    if (g.Cg == 1) {
        const dwconv_desc q = as_depthwise(desc);
        return dwconv_variant_name(&q, pass);
    }
    return gplan(g, desc->layout, desc->dtype, pass).name;
}

}  // extern "C"

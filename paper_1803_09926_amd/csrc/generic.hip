// Generic fallback kernels: correct for any K, stride, pad and channel multiplier, both layouts,
// both storage types.  One thread per output element; not tuned.  Also holds the second stage of
// the filter-gradient reduction, which every bwd_filter variant shares.
#include "point.hpp"

namespace dwc {

// Decompose a flat element index of a [N,CH,HH,WW] / [N,HH,WW,CH] tensor.
template <int LAYOUT>
__device__ __forceinline__ void unflat(int idx, int CH, int HH, int WW, int &n, int &ch, int &h, int &w)
{
    if (LAYOUT == LAYOUT_NCHW) {
        w = idx % WW; idx /= WW; h = idx % HH; idx /= HH; ch = idx % CH; n = idx / CH;
    } else {
        ch = idx % CH; idx /= CH; w = idx % WW; idx /= WW; h = idx % HH; n = idx / HH;
    }
}

template <typename T, int LAYOUT>
__global__ __launch_bounds__(256) void k_generic_fwd(Geom g, const T *__restrict__ x, const T *__restrict__ w,
                                                     T *__restrict__ y, int total)
{
    const unsigned uidx = blockIdx.x * 256u + threadIdx.x;   // the last block may reach past 2^31
    if (uidx >= (unsigned)total) return;
    int idx = (int)uidx;
    int n, o, oh, ow;
    unflat<LAYOUT>(idx, g.O, g.Ho, g.Wo, n, o, oh, ow);
    stf(y + idx, point_fwd<T, LAYOUT>(g, x, w, n, o, oh, ow));
}

template <typename T, int LAYOUT>
__global__ __launch_bounds__(256) void k_generic_bwd_data(Geom g, const T *__restrict__ dy, const T *__restrict__ w,
                                                          T *__restrict__ dx, int total)
{
    const unsigned uidx = blockIdx.x * 256u + threadIdx.x;   // the last block may reach past 2^31
    if (uidx >= (unsigned)total) return;
    int idx = (int)uidx;
    int n, c, ih, iw;
    unflat<LAYOUT>(idx, g.C, g.H, g.W, n, c, ih, iw);
    stf(dx + idx, point_bwd_data<T, LAYOUT>(g, dy, w, n, c, ih, iw));
}

// Stage 1, NCHW: block (tap j = (o*K+kh)*K+kw, part).  Threads stride over the pixels
// (n, oh, ow) of the part with ow fastest; wavefront butterfly, then LDS across the 4 waves.
template <typename T>
__global__ __launch_bounds__(256) void k_generic_bwd_filter_nchw(Geom g, const T *__restrict__ x,
                                                                 const T *__restrict__ dy, float *__restrict__ ws,
                                                                 int parts, int per_part)
{
    __shared__ float red[4];
    const int j = blockIdx.x, part = blockIdx.y;
    const int kw = j % g.K, kh = (j / g.K) % g.K, o = j / (g.K * g.K);
    const int c = o / g.m;
    const int npix = g.N * g.Ho * g.Wo;
    const int lo = part * per_part, hi = min(npix, lo + per_part);
    float acc = 0.f;
    for (int pix = lo + (int)threadIdx.x; pix < hi; pix += 256) {
        int ow = pix % g.Wo, t = pix / g.Wo, oh = t % g.Ho, n = t / g.Ho;
        int ih = oh * g.s - g.p + kh, iw = ow * g.s - g.p + kw;
        if (ih < 0 || ih >= g.H || iw < 0 || iw >= g.W) continue;
        acc = fmaf(ldf(dy + at<LAYOUT_NCHW>(g.O, g.Ho, g.Wo, n, o, oh, ow)),
                   ldf(x + at<LAYOUT_NCHW>(g.C, g.H, g.W, n, c, ih, iw)), acc);
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) ws[(size_t)part * (g.O * g.K * g.K) + j] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Stage 1, NHWC: block (tile of 64 output channels, tap (kh,kw), part).  Lane = channel, the 4
// waves stride over pixels; LDS across the waves.
template <typename T>
__global__ __launch_bounds__(256) void k_generic_bwd_filter_nhwc(Geom g, const T *__restrict__ x,
                                                                 const T *__restrict__ dy, float *__restrict__ ws,
                                                                 int parts, int per_part)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int o = blockIdx.x * 64 + lane;
    const int tap = blockIdx.y, part = blockIdx.z;
    const int kw = tap % g.K, kh = tap / g.K;
    const int npix = g.N * g.Ho * g.Wo;
    const int lo = part * per_part, hi = min(npix, lo + per_part);
    float acc = 0.f;
    if (o < g.O) {
        const int c = o / g.m;
        for (int pix = lo + wv; pix < hi; pix += 4) {
            int ow = pix % g.Wo, t = pix / g.Wo, oh = t % g.Ho, n = t / g.Ho;
            int ih = oh * g.s - g.p + kh, iw = ow * g.s - g.p + kw;
            if (ih < 0 || ih >= g.H || iw < 0 || iw >= g.W) continue;
            acc = fmaf(ldf(dy + (size_t)pix * g.O + o), ldf(x + at<LAYOUT_NHWC>(g.C, g.H, g.W, n, c, ih, iw)), acc);
        }
    }
    red[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && o < g.O)
        ws[(size_t)part * (g.O * g.K * g.K) + tap * g.O + o] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Products of entry j inside the image over the outputs of one partial, added up by the block (see FilterGradSrc).  A NaN ends the
// sum: whatever is added stays a NaN.
__device__ __forceinline__ float partial_inside(const FilterGradSrc &f, int j, int partial, float *red)
{
    const bool nhwc = f.layout == LAYOUT_NHWC;
    const int KK = f.K * f.K, tap = nhwc ? j / (f.Cg * f.O) : j % KK, kh = tap / f.K, kw = tap - kh * f.K;
    const int o = nhwc ? j % f.O : j / KK / f.Cg, ci = (nhwc ? j / f.O : j / KK) % f.Cg, c = o / f.Og * f.Cg + ci;
    const int ntiles = f.tn * f.ta * f.tb, step = f.per ? 1 : f.nparts, npos = f.TN * f.TA * f.TB;
    const int first = f.per ? partial * f.per : partial, last = f.per && ntiles - first > f.per ? first + f.per : ntiles;
    float acc = 0.f;
    for (int tile = first; tile < last; tile += step) {
        const int tb = tile % f.tb, ta = tile / f.tb % f.ta, tn = tile / f.tb / f.ta;
        for (int q0 = 0; q0 < npos; q0 += 256 * 8) {
            // eight products of a lane on their way at a time
            float a[8], b[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int q = q0 + i * 256 + (int)threadIdx.x, r = q / f.TB, im = r / f.TA;
                const int ow = tb * f.TB + q - r * f.TB, oh = ta * f.TA + r - im * f.TA, n = tn * f.TN + im;
                const int ih = oh * f.s - f.p + kh, iw = ow * f.s - f.p + kw;
                a[i] = b[i] = 0.f;
                if (q >= npos || n >= f.N || oh >= f.Ho || ow >= f.Wo || (unsigned)ih >= (unsigned)f.H ||
                    (unsigned)iw >= (unsigned)f.W) continue;
                const size_t px = nhwc ? ((size_t)(n * f.H + ih) * f.W + iw) * f.C + c : ((size_t)(n * f.C + c) * f.H + ih) * f.W + iw;
                const size_t py = nhwc ? ((size_t)(n * f.Ho + oh) * f.Wo + ow) * f.O + o : ((size_t)(n * f.O + o) * f.Ho + oh) * f.Wo + ow;
                a[i] = f.dtype == DT_F32 ? ((const float *)f.dy)[py] : ldf((const bf16_t *)f.dy + py);
                b[i] = f.dtype == DT_F32 ? ((const float *)f.x)[px] : ldf((const bf16_t *)f.x + px);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) acc = fmaf(a[i], b[i], acc);
            if (__syncthreads_or(acc != acc)) return __builtin_nanf("");
        }
    }
    acc = wave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// Entry j again: its finite partials as they are, the others from the products inside the image, until the sum is a NaN.  What costs
// time is a partial that is not finite and whose products inside the image are no NaN, so that all of them are read: one such value
// per channel takes one partial per entry.  (64x147x147 3x3 NCHW fp32, batch 32, finite 0.09 ms: every dy a NaN 0.36 ms, one infinity per
// channel 2.4, in the first corner of every image and channel 21; with all of dy read for every such entry 60 to 90 in each case.)
__device__ float entry_inside(const FilterGradSrc &f, int j, const float *ws, int parts, int J, float *red, unsigned long long *flags)
{
    float total = 0.f, mine = 0.f;
    for (int p0 = 0; p0 < parts; p0 += 256) {
        const int p = p0 + (int)threadIdx.x;
        const float v = p < parts ? ws[(size_t)p * J + j] : 0.f;
        const bool finite = __builtin_fabsf(v) < __builtin_inff();
        mine += finite ? v : 0.f;
        const unsigned long long b = __ballot(!finite);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = b;
        __syncthreads();
        for (int w = 0; w < 4; ++w)
            for (unsigned long long m = flags[w]; m; m &= m - 1) {         // uniform
                total += partial_inside(f, j, p0 + w * 64 + __ffsll((long long)m) - 1, red);
                if (total != total) return total;
            }
    }
    mine = wave_sum(mine);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mine;
    __syncthreads();
    return ((red[0] + red[1]) + (red[2] + red[3])) + total;
}

// total[e]: the block's entries j0 + e < J, in LDS
template <int JT, bool CHECK, typename S>
__device__ __forceinline__ void store_entries(const FilterGradSrc &src, const S *total, int j0, const float *ws, int parts, int J, float *dw)
{
    const int t = threadIdx.x;
    const bool mine = t < JT && j0 + t < J;
    const float v = t < JT ? (float)total[t] : 0.f;
    const bool bad = CHECK && mine && !(__builtin_fabsf(v) < __builtin_inff());
    if (mine && !bad) dw[j0 + t] = v;
    if constexpr (CHECK) {
        if (!__syncthreads_or(bad)) return;
        __shared__ float red[4];
        __shared__ unsigned long long flags[4];
#pragma unroll 1
        for (int e = 0; e < JT && j0 + e < J; ++e) {
            if (__builtin_fabsf((float)total[e]) < __builtin_inff()) continue;
            const float s = entry_inside(src, j0 + e, ws, parts, J, red, flags);
            if (t == 0) dw[j0 + e] = s;
        }
    }
}

// Stage 2: dw[j] = sum_p ws[p*J + j].  A block owns JT consecutive j; PT = 256/JT threads per j
// take the partials p = r, r+PT, r+2PT, ... eight at a time.  All eight loads of a batch are issued
// before the first is used, also in the last, partly filled batch (clamped index, value dropped):
// the kernel is a few microseconds of pure load latency, so one latency per batch is what counts.
// The batch is added in a fixed tree, then the PT sub-sums in a fixed tree, in S: 32 bits through LDS; 64 bits (wide: 0.6 to 0.9 of the
// error of a whole gradient) over the wavefront first, which is a barrier instead of two to six (as short as 32 bits through LDS up to 16 000 entries, 0.97 to 0.99 of a gradient below 9 us).
template <int JT, bool CHECK, typename S>
__global__ __launch_bounds__(256) void k_reduce_partials(const float *__restrict__ ws, int parts, int J,
                                                         float *__restrict__ dw, FilterGradSrc src)
{
    constexpr int PT = 256 / JT;
    __shared__ S red[PT][JT + 1];
    const int jj = threadIdx.x % JT, r = threadIdx.x / JT;
    const int j = blockIdx.x * JT + jj;
    S acc = 0;
    if (j < J) {
        const float *p0 = ws + j;
        for (int p = r; p < parts; p += 8 * PT) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int q = p + i * PT;
                const float t = p0[(size_t)min(q, parts - 1) * J];
                v[i] = q < parts ? t : 0.f;
            }
            acc += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        }
    }
    if constexpr (sizeof(S) == 8) {
#pragma unroll
        for (int off = 32; off >= JT; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((threadIdx.x & 63) < JT) red[threadIdx.x >> 6][jj] = acc;
        __syncthreads();
        if (r == 0) red[0][jj] = (red[0][jj] + red[1][jj]) + (red[2][jj] + red[3][jj]);
        __syncthreads();
    } else {
        red[r][jj] = acc;
        __syncthreads();
        // tree over the PT sub-sums: thread (r, jj) adds red[r + half]
        for (int half = PT / 2; half >= 1; half >>= 1) {
            if (r < half) red[r][jj] += red[r + half][jj];
            __syncthreads();
        }
    }
    store_entries<JT, CHECK>(src, red[0], blockIdx.x * JT, ws, parts, J, dw);
}

// The same for J a multiple of 4: a lane takes four consecutive j, so that a wavefront reads 256 to 1024 consecutive bytes of a
// partial row instead of 32 to 256; JT / 4 lanes across j, the others across the partials.
template <typename S> struct Sum4 { S x, y, z, w; };
template <int JT, bool CHECK, typename S>
__global__ __launch_bounds__(256) void k_reduce_partials4(const float *__restrict__ ws, int parts, int J, float *__restrict__ dw,
                                                          FilterGradSrc src)
{
    constexpr int JL = JT / 4, PT = 256 / JL;
    __shared__ Sum4<S> red[PT][JL];
    const int jj = threadIdx.x % JL, r = threadIdx.x / JL;
    const int j = blockIdx.x * JT + jj * 4;
    Sum4<S> acc = {0, 0, 0, 0};
    auto add = [](auto a, auto b) { a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w; return a; };
    if (j < J) {
        const float *p0 = ws + j;
        for (int p = r; p < parts; p += 8 * PT) {
            float4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int q = p + i * PT;
                const float4 t = *reinterpret_cast<const float4 *>(p0 + (size_t)min(q, parts - 1) * J);
                v[i] = q < parts ? t : make_float4(0.f, 0.f, 0.f, 0.f);
            }
            acc = add(acc, add(add(add(v[0], v[1]), add(v[2], v[3])), add(add(v[4], v[5]), add(v[6], v[7]))));
        }
    }
    if constexpr (sizeof(S) == 8) {
#pragma unroll
        for (int off = 32; off >= JL; off >>= 1)
            acc = add(acc, Sum4<S>{__shfl_xor(acc.x, off, 64), __shfl_xor(acc.y, off, 64), __shfl_xor(acc.z, off, 64), __shfl_xor(acc.w, off, 64)});
        if ((threadIdx.x & 63) < JL) red[threadIdx.x >> 6][jj] = acc;
        __syncthreads();
        if (r == 0) red[0][jj] = add(add(red[0][jj], red[1][jj]), add(red[2][jj], red[3][jj]));
        __syncthreads();
    } else {
        red[r][jj] = acc;
        __syncthreads();
        for (int half = PT / 2; half >= 1; half >>= 1) {
            if (r < half) red[r][jj] = add(red[r][jj], red[r + half][jj]);
            __syncthreads();
        }
    }
    if constexpr (CHECK) store_entries<JT, true>(src, &red[0][0].x, blockIdx.x * JT, ws, parts, J, dw);
    else if (r == 0 && j < J) *reinterpret_cast<float4 *>(dw + j) = make_float4(red[0][jj].x, red[0][jj].y, red[0][jj].z, red[0][jj].w);
}

// ---- host side --------------------------------------------------------------------------------

hipError_t generic_fwd(const Geom &g, int layout, int dtype, const void *x, const void *w, void *y, hipStream_t st)
{
    const int total = g.N * g.O * g.Ho * g.Wo;
    dim3 grid((unsigned)(((long long)total + 255) / 256)), block(256);
#define LAUNCH(T, L) hipLaunchKernelGGL((k_generic_fwd<T, L>), grid, block, 0, st, g, (const T *)x, (const T *)w, (T *)y, total)
    if (dtype == DT_F32) { if (layout == LAYOUT_NCHW) LAUNCH(float, LAYOUT_NCHW); else LAUNCH(float, LAYOUT_NHWC); }
    else                 { if (layout == LAYOUT_NCHW) LAUNCH(bf16_t, LAYOUT_NCHW); else LAUNCH(bf16_t, LAYOUT_NHWC); }
#undef LAUNCH
    return hipGetLastError();
}

hipError_t generic_bwd_data(const Geom &g, int layout, int dtype, const void *dy, const void *w, void *dx, hipStream_t st)
{
    const int total = g.N * g.C * g.H * g.W;
    dim3 grid((unsigned)(((long long)total + 255) / 256)), block(256);
#define LAUNCH(T, L) hipLaunchKernelGGL((k_generic_bwd_data<T, L>), grid, block, 0, st, g, (const T *)dy, (const T *)w, (T *)dx, total)
    if (dtype == DT_F32) { if (layout == LAYOUT_NCHW) LAUNCH(float, LAYOUT_NCHW); else LAUNCH(float, LAYOUT_NHWC); }
    else                 { if (layout == LAYOUT_NCHW) LAUNCH(bf16_t, LAYOUT_NCHW); else LAUNCH(bf16_t, LAYOUT_NHWC); }
#undef LAUNCH
    return hipGetLastError();
}

int generic_bwd_filter_parts(const Geom &g)
{
    // about 8192 pixels per part, at most 64 parts, and never more than 32 MiB of partials
    long long npix = (long long)g.N * g.Ho * g.Wo;
    long long parts = (npix + 8191) / 8192;
    if (parts > 64) parts = 64;
    long long J = (long long)g.O * g.K * g.K;
    while (parts > 1 && parts * J * 4 > (32ll << 20)) parts >>= 1;
    if (parts < 1) parts = 1;
    return (int)parts;
}

hipError_t generic_bwd_filter(const Geom &g, int layout, int dtype, const void *x, const void *dy, float *ws,
                              int parts, hipStream_t st)
{
    const int npix = g.N * g.Ho * g.Wo;
    const int per_part = (npix + parts - 1) / parts;
    if (layout == LAYOUT_NCHW) {
        dim3 grid(g.O * g.K * g.K, parts), block(256);
        if (dtype == DT_F32)
            hipLaunchKernelGGL(k_generic_bwd_filter_nchw<float>, grid, block, 0, st, g, (const float *)x, (const float *)dy, ws, parts, per_part);
        else
            hipLaunchKernelGGL(k_generic_bwd_filter_nchw<bf16_t>, grid, block, 0, st, g, (const bf16_t *)x, (const bf16_t *)dy, ws, parts, per_part);
    } else {
        dim3 grid((g.O + 63) / 64, g.K * g.K, parts), block(256);
        if (dtype == DT_F32)
            hipLaunchKernelGGL(k_generic_bwd_filter_nhwc<float>, grid, block, 0, st, g, (const float *)x, (const float *)dy, ws, parts, per_part);
        else
            hipLaunchKernelGGL(k_generic_bwd_filter_nhwc<bf16_t>, grid, block, 0, st, g, (const bf16_t *)x, (const bf16_t *)dy, ws, parts, per_part);
    }
    return hipGetLastError();
}

template <bool CHECK, typename S>
static hipError_t reduce_go(const float *ws, int parts, int J, float *dw, const FilterGradSrc &src, hipStream_t st)
{
    // threads per output chosen so that one batch of eight loads per thread covers the partials
    // (PT = 256/JT about parts/8), but enough blocks to spread small J over the chip
    // From 2048 entries on four a lane: a lane's loads then span whole lines of a partial (6400 entries x 448 partials 9.5 -> 5 us,
    // 18432 x 128 6.8 -> 5); below that the narrower lanes spread better (288 x 15: 2.7 us against 3.1).
    if (J % 4 == 0 && J >= 2048) {
        int jt = 16;
        while (jt < 64 && (256 / (jt / 4)) * 8 > parts && (J + 2 * jt - 1) / (2 * jt) >= 128) jt *= 2;
#define GO(JT) hipLaunchKernelGGL((k_reduce_partials4<JT, CHECK, S>), dim3((J + JT - 1) / JT), dim3(256), 0, st, ws, parts, J, dw, src)
        if (jt == 16) GO(16);
        else if (jt == 32) GO(32);
        else GO(64);
#undef GO
        return hipGetLastError();
    }
    int jt = 4;
    while (jt < 64 && (256 / jt) * 8 > parts && (J + 2 * jt - 1) / (2 * jt) >= 8) jt *= 2;
#define GO(JT) hipLaunchKernelGGL((k_reduce_partials<JT, CHECK, S>), dim3((J + JT - 1) / JT), dim3(256), 0, st, ws, parts, J, dw, src)
    switch (jt) {
    case 4: GO(4); break;
    case 8: GO(8); break;
    case 16: GO(16); break;
    case 32: GO(32); break;
    default: GO(64); break;
    }
#undef GO
    return hipGetLastError();
}

hipError_t reduce_partials(const float *ws, int parts, int J, float *dw, hipStream_t st)
{
    return reduce_go<false, float>(ws, parts, J, dw, FilterGradSrc{}, st);
}
hipError_t reduce_partials(const float *ws, int parts, int J, float *dw, const FilterGradSrc &src, bool wide, hipStream_t st)
{
    return (wide ? reduce_go<true, double> : reduce_go<true, float>)(ws, parts, J, dw, src, st);
}

}  // namespace dwc

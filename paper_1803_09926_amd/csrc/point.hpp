// One output at a time, tap by tap, any K, stride, pad and multiplier: the generic kernels, and what the kernels of nchw_flat.hip
// and nhwc_any.hip fall back to for a channel whose filter holds an infinity or NaN.  The tiled kernels multiply the zeros of the
// padding (and of columns and rows that are none) like any value; against a non-finite factor that product is a NaN where no
// product belongs.  (In the filter gradient the second stage does this, see FilterGradSrc: in the walk the addresses of the
// products would cost a third of the wavefronts.)  The check costs a pass about 1%: 19x19x480 3x3 fp32 18.6 -> 18.9 us.
#pragma once
#include "kernels.hpp"

namespace dwc {

template <int LAYOUT>
__device__ __forceinline__ int at(int CH, int HH, int WW, int n, int ch, int h, int w)
{
    if (LAYOUT == LAYOUT_NCHW) return ((n * CH + ch) * HH + h) * WW + w;
    return ((n * HH + h) * WW + w) * CH + ch;
}
template <int LAYOUT>
__device__ __forceinline__ int wat(int O, int K, int o, int kh, int kw)
{
    if (LAYOUT == LAYOUT_NCHW) return (o * K + kh) * K + kw;
    return (kh * K + kw) * O + o;
}

template <typename T, int LAYOUT>
__device__ __forceinline__ float point_fwd(const Geom &g, const T *x, const T *w, int n, int o, int oh, int ow)
{
    const int c = o / g.m;
    float acc = 0.f;
#pragma unroll 1
    for (int kh = 0; kh < g.K; ++kh) {
        int ih = oh * g.s - g.p + kh;
        if (ih < 0 || ih >= g.H) continue;
#pragma unroll 1
        for (int kw = 0; kw < g.K; ++kw) {
            int iw = ow * g.s - g.p + kw;
            if (iw < 0 || iw >= g.W) continue;
            acc = fmaf(ldf(w + wat<LAYOUT>(g.O, g.K, o, kh, kw)), ldf(x + at<LAYOUT>(g.C, g.H, g.W, n, c, ih, iw)), acc);
        }
    }
    return acc;
}

template <typename T, int LAYOUT>
__device__ __forceinline__ float point_bwd_data(const Geom &g, const T *dy, const T *w, int n, int c, int ih, int iw)
{
    float acc = 0.f;
#pragma unroll 1
    for (int q = 0; q < g.m; ++q) {
        const int o = c * g.m + q;
#pragma unroll 1
        for (int kh = 0; kh < g.K; ++kh) {
            int th = ih + g.p - kh;
            if (th < 0 || th % g.s != 0) continue;
            int oh = th / g.s;
            if (oh >= g.Ho) continue;
#pragma unroll 1
            for (int kw = 0; kw < g.K; ++kw) {
                int tw = iw + g.p - kw;
                if (tw < 0 || tw % g.s != 0) continue;
                int ow = tw / g.s;
                if (ow >= g.Wo) continue;
                acc = fmaf(ldf(w + wat<LAYOUT>(g.O, g.K, o, kh, kw)), ldf(dy + at<LAYOUT>(g.O, g.Ho, g.Wo, n, o, oh, ow)), acc);
            }
        }
    }
    return acc;
}

// Whether an infinity or NaN has been added: half an instruction per value (v_maximum3_f32 keeps a NaN).
struct NonFinite {
    float most = 0.f;
    __device__ __forceinline__ void add(float v) { most = __builtin_elementwise_maximum(most, __builtin_fabsf(v)); }
    __device__ __forceinline__ bool any() const { return !(most < __builtin_inff()); }
};

}  // namespace dwc

// Group convolution on the 16x16 matrix instructions: either layout, any group size and padding, strides up to 4, K up to 7 (filter gradient:
// 5), where the filter entries of 16 outputs and the smallest tile fit 64 KiB of LDS.  Where they do not, one output per thread is left, in
// the forward pass and, at stride 1, the input gradient: fp32 5x5 with 24 channels a group, and with 32 on rows of 16 and more (at stride 2
// both on all rows); fp32 7x7 with 16 and fewer on rows of 28 and more; fp32 NCHW 3x3 stride 2 with 24 and 32 on rows from 75 on; bf16 5x5
// with 24, and NCHW stride 2 with 32, on most rows from 56 on.
//
// Forward (and the input gradient): D[o][pixel] += sum over (tap, input channel) W[o][tap, ci] * X[tap, ci][pixel], 16 output
// channels x 16 pixels per instruction.  A block owns up to a few times 16 output channels and a tile of positions; the
// input pixels its taps reach sit in LDS as [pixel][channel] with the zero padding written out, so that for any stride and
// tap a lane's operand is four consecutive channels of one pixel: one 8-byte (bf16) or 16-byte (fp32) LDS read.  The filter
// entries are laid out in LDS once per block in operand order.  With fewer than 16 channels per group the 16 outputs span
// several groups and the entries that pair different groups are zeros; a tile that holds an infinity or NaN is then
// computed without them, so that it stays inside its group.
// Input gradient at stride s: with h + p = s*a + f and w + p = s*b + e the taps kh = f + s*k, kw = e + s*l read dy[a - k][b - l]:
// s*s classes (f, e) of output pixels, each a stride-1 convolution over the same staged dy tile.
// Filter gradient: D[o][ci] += dy[o][pixel] * X[ci][pixel + tap], the contraction over pixels, all taps in registers.
//
// What bounds it: not the matrix cores (the three passes of the 14x14 layer below need 2 us of them) but the latency of a short
// block: filter, tile and outputs are three rounds to memory, so every lane issues its loads of a round together (with one load
// at a time the same passes took 20, 20 and 40 us).  us on one MI355X, one output per thread -> these kernels, forward / input
// gradient / filter gradient: 14x14x512, 16 channels a group, bf16 NHWC batch 32 207 / 777 / 888 -> 14 / 16 / 20; 56x56x256
// stride 2, 8 channels a group, bf16 NCHW batch 16 183 / 893 / 396 -> 24 / 22 / 31; 57x57x128, 4 channels a group, fp32 NCHW
// batch 64 629 / 950 / 1730 -> 155 / 154 / 145 (there 3 of 4 products are zeros).
#include "gconv.hpp"

namespace dwc {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));

// four consecutive channels of one pixel, or of one output's filter entries, in the storage type
template <typename T> struct Frag;
template <> struct Frag<float> { float4 v; };
template <> struct Frag<bf16_t> { uint2 v; };

__device__ __forceinline__ v4f mma16(const Frag<float> &a, const Frag<float> &b, v4f d)
{
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.x, b.v.x, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.y, b.v.y, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.z, b.v.z, d, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.w, b.v.w, d, 0, 0, 0);
}
__device__ __forceinline__ v4f mma16(const Frag<bf16_t> &a, const Frag<bf16_t> &b, v4f d)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, a.v), __builtin_bit_cast(v4s, b.v), d, 0, 0, 0);
}

__device__ __forceinline__ void gather4(Frag<float> &f, const float *a, const float *b, const float *c, const float *d)
{
    f.v = make_float4(*a, *b, *c, *d);
}
__device__ __forceinline__ void gather4(Frag<bf16_t> &f, const bf16_t *a, const bf16_t *b, const bf16_t *c, const bf16_t *d)
{
    f.v = make_uint2((uint32_t)*a | (uint32_t)*b << 16, (uint32_t)*c | (uint32_t)*d << 16);
}

template <typename T> __device__ __forceinline__ bool nonfinite(T v);
template <> __device__ __forceinline__ bool nonfinite<float>(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }
template <> __device__ __forceinline__ bool nonfinite<bf16_t>(bf16_t v) { return (v & 0x7f80u) == 0x7f80u; }

// One launch: the convolution from `in` (CI channels, Hi x Wi) to `out` (CO channels, Ho x Wo).  Position (a, b) of a tile
// reads input row IS*a - ip + roff and writes output row OS*a + f - op; roff = kh forward, -k for tap kh = f + OS*k backward.
struct GemmGeom {
    int N, CI, CO, Hi, Wi, Ho, Wo;
    int Cgi, Cgo;          // channels per group, input and output side
    int K, IS, OS, ip, op;
    int a0, na, b0, nb;    // positions of the whole image
    int bwd;
    // tile
    int TN, TA, TB;        // images, rows and columns of positions
    int tn, ta, tb;        // tiles in each direction
    int LH, LW;            // input pixels of a tile, per image
    int lo;                // lowest roff (backward: -(taps per class - 1))
    int NS, nk, CL, pitch; // 16-channel output blocks, 16-channel input chunks of each, channels in LDS, elements between pixels
    int nchb;              // channel blocks
    int packed;            // output blocks span groups
    int FO, FCg;           // filter dims: output channels, input channels per group (of the forward layer)
    float rCgi, rCgo, rKK, rnk;   // reciprocals for fdiv
};

// n / d for 0 <= n < 2^21 and d with reciprocal r = 1.0f / d: the half keeps the product away from the integers by more than
// its rounding error (0.5 / d against n / d * 2^-22), four instructions instead of the twenty of an integer division.
__device__ __forceinline__ int fdiv(int n, float r) { return (int)(((float)n + 0.5f) * r); }

__device__ __forceinline__ int cin_first(int o0, const GemmGeom &g) { return fdiv(o0, g.rCgo) * g.Cgi & ~3; }

// Input pixels of a tile to LDS as [image][row][column][channel]; what lies outside the image or the tensor's channels is
// written as zero.  Returns whether the lane staged an infinity or NaN.
// FAST: NHWC channel counts that are whole 16-byte vectors; NCHW tiles that span the rows.
template <typename T, bool NHWC, bool FAST>
__device__ __forceinline__ bool stage_pixels(const T *__restrict__ in, T *lx, int N, int C, int H, int W, int n0, int nimg, int h0, int w0,
                                             int LH, int LW, int ca, int CL, int pitch, bool check)
{
    [[maybe_unused]] constexpr int VE = 16 / (int)sizeof(T);
    bool bad = false;
    const int npix = nimg * LH * LW;
    const float rLW = 1.0f / (float)LW, rLH = 1.0f / (float)LH;
    // image, row and column of a staged pixel; false if it lies outside
    auto locate = [&](int pix, int &n, int &h, int &w) {
        const int r = fdiv(pix, rLW), im = fdiv(r, rLH);
        n = n0 + im; h = r - im * LH + h0; w = pix - r * LW + w0;
        return n < N && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W;
    };
    // every lane has B loads in flight before its first LDS write
    if constexpr (NHWC && FAST) {
        // a lane copies 16 bytes of channels of one pixel; ca is a multiple of VE
        constexpr int B = 8;
        const int nv = CL / VE, total = npix * nv;
        const float rnv = 1.0f / (float)nv;
        for (int i0 = threadIdx.x; i0 < total; i0 += B * 256) {
            u4v_t q[B];
            int at[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int i = i0 + b * 256, pix = fdiv(i, rnv), v = i - pix * nv, c = ca + v * VE;
                int n, h, w;
                const bool ok = locate(pix, n, h, w) && i < total && c < C;
                at[b] = i < total ? pix * pitch + v * VE : -1;
                q[b] = u4v_t{0u, 0u, 0u, 0u};
                if (ok) q[b] = *reinterpret_cast<const u4v_t *>(in + (unsigned)(((n * H + h) * W + w) * C + c));
            }
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (check) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        bad |= (sizeof(T) == 2 && (q[b][k] & 0x7f80u) == 0x7f80u) || (q[b][k] & 0x7f800000u) == 0x7f800000u;
                }
                if (at[b] >= 0) *reinterpret_cast<u4v_t *>(lx + at[b]) = q[b];
            }
        }
        return bad;
    }
    if constexpr (!NHWC && FAST) {
        // whole rows: a lane copies four channels of four consecutive pixels of a row, transposed in registers; the columns
        // beside the row are zero from the start and stay so
        constexpr int B = 2;
        const int nq = CL / 4, nr = (W + 3) / 4, rows = nimg * LH, total = nr * rows * nq;
        const float rnr = 1.0f / (float)nr, rrows = 1.0f / (float)rows;
        const unsigned end = (unsigned)(N * C * H * W), plane = (unsigned)(H * W);
        for (int i0 = threadIdx.x; i0 < total; i0 += B * 256) {
            T e[B][4][4];
            int at[B], len[B], col[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int i = i0 + b * 256, t = fdiv(i, rnr), run = i - t * nr, qd = fdiv(t, rrows), r = t - qd * rows;
                const int im = fdiv(r, rLH), h = r - im * LH + h0, n = n0 + im, c = ca + qd * 4;
                const bool ok = n < N && (unsigned)h < (unsigned)H && i < total;
                col[b] = run * 4 - w0;
                at[b] = (r * LW + col[b]) * pitch + qd * 4;
                len[b] = i < total ? min(4, W - run * 4) : 0;
                const unsigned p0 = (unsigned)(((n * C + c) * H + h) * W + run * 4);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) e[b][k][j] = T(0);
                    if (ok && c + k < C) {
                        const T *p = in + p0 + k * plane;
                        if (p0 + k * plane + 4 <= end) __builtin_memcpy(e[b][k], p, 4 * sizeof(T));      // any alignment
                        else {
#pragma unroll
                            for (int j = 0; j < 4; ++j) if (j < len[b]) e[b][k][j] = p[j];
                        }
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j >= len[b] || (unsigned)(col[b] + j) >= (unsigned)LW) continue;      // a column that no tap reaches
                    if (check) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) bad |= nonfinite<T>(e[b][k][j]);
                    }
                    Frag<T> f;
                    if constexpr (sizeof(T) == 4) f.v = make_float4(e[b][0][j], e[b][1][j], e[b][2][j], e[b][3][j]);
                    else f.v = make_uint2((uint32_t)e[b][0][j] | (uint32_t)e[b][1][j] << 16, (uint32_t)e[b][2][j] | (uint32_t)e[b][3][j] << 16);
                    *reinterpret_cast<Frag<T> *>(lx + at[b] + j * pitch) = f;
                }
        }
        return bad;
    }
    // a lane gathers four channels of one pixel; consecutive lanes take consecutive pixels of the plane (NCHW) or
    // consecutive channels (NHWC with a channel count that is no whole number of vectors)
    constexpr int B = 4;
    const int nq = CL / 4, total = npix * nq, per = NHWC ? nq : npix;
    const float rper = 1.0f / (float)per;
    const int cstep = NHWC ? 1 : H * W;
    for (int i0 = threadIdx.x; i0 < total; i0 += B * 256) {
        T e[B][4];
        int at[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int i = i0 + b * 256, hi = fdiv(i, rper), lo = i - hi * per, pix = NHWC ? hi : lo, c = ca + (NHWC ? lo : hi) * 4;
            int n, h, w;
            const bool ok = locate(pix, n, h, w) && i < total;
            at[b] = i < total ? pix * pitch + c - ca : -1;
            const T *p = in + (unsigned)(NHWC ? ((n * H + h) * W + w) * C + c : ((n * C + c) * H + h) * W + w);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e[b][k] = T(0);
                if (ok && c + k < C) e[b][k] = p[k * cstep];
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            if (check) {
#pragma unroll
                for (int k = 0; k < 4; ++k) bad |= nonfinite<T>(e[b][k]);
            }
            Frag<T> f;
            if constexpr (sizeof(T) == 4) f.v = make_float4(e[b][0], e[b][1], e[b][2], e[b][3]);
            else f.v = make_uint2((uint32_t)e[b][0] | (uint32_t)e[b][1] << 16, (uint32_t)e[b][2] | (uint32_t)e[b][3] << 16);
            if (at[b] >= 0) *reinterpret_cast<Frag<T> *>(lx + at[b]) = f;
        }
    }
    return bad;
}

// A tile that holds an infinity or NaN where 16 outputs span several groups, or whose filter does: one output per lane, its own
// group's channels and the taps inside the image only.
template <typename T, bool NHWC>
__device__ __forceinline__ void own_group_only(const GemmGeom &g, const Frag<T> *lw, const T *lx, T *__restrict__ out, int n0, int a0,
                                                         int b0, int ob, int ca)
{
    const int npos = g.TN * g.TA * g.TB, nch = g.NS * 16, KK = g.K * g.K;
#pragma unroll 1
    for (int i = threadIdx.x; i < g.OS * g.OS * npos * nch; i += 256) {
        const int oc = i % nch, q = i / nch % npos, cls = i / nch / npos;
        const int f = cls / g.OS, e = cls - f * g.OS, im = q / (g.TA * g.TB), da = q / g.TB % g.TA, db = q % g.TB;
        const int o = ob + oc, row = g.OS * (a0 + da) + f - g.op, col = g.OS * (b0 + db) + e - g.op;
        if (o >= g.CO || n0 + im >= g.N || a0 + da >= g.a0 + g.na || b0 + db >= g.b0 + g.nb || (unsigned)row >= (unsigned)g.Ho ||
            (unsigned)col >= (unsigned)g.Wo) continue;
        const int s = oc / 16, c0 = o / g.Cgo * g.Cgi, cs = cin_first(ob + s * 16, g);
        float acc = 0.f;
#pragma unroll 1
        for (int kh = f, k = 0; kh < g.K; kh += g.OS, ++k)
#pragma unroll 1
            for (int kw = e, l = 0; kw < g.K; kw += g.OS, ++l) {
                const int ro = g.bwd ? -k : kh, co = g.bwd ? -l : kw;
                if ((unsigned)(g.IS * (a0 + da) - g.ip + ro) >= (unsigned)g.Hi || (unsigned)(g.IS * (b0 + db) - g.ip + co) >= (unsigned)g.Wi) continue;
                const T *px = lx + ((im * g.LH + g.IS * da + ro - g.lo) * g.LW + g.IS * db + co - g.lo) * g.pitch;
#pragma unroll 1
                for (int c = c0; c < c0 + g.Cgi; ++c) {
                    const int j = c - cs;
                    const T *pw = reinterpret_cast<const T *>(&lw[((s * KK + kh * g.K + kw) * g.nk + j / 16) * 64 + j % 16 / 4 * 16 + oc % 16]);
                    acc = fmaf(ldf(pw + j % 4), ldf(px + c - ca), acc);
                }
            }
        stf(out + (NHWC ? (((size_t)(n0 + im) * g.Ho + row) * g.Wo + col) * g.CO + o : (((size_t)(n0 + im) * g.CO + o) * g.Ho + row) * g.Wo + col), acc);
    }
}

// ---------------------------------------------------------------------------------------------
// Forward and input gradient.  P: 16-pixel tiles that a wavefront computes at a time against one read of the filter.
// ---------------------------------------------------------------------------------------------
template <typename T, bool NHWC, bool FAST, int P>
__global__ __launch_bounds__(256) void k_gconv_gemm(GemmGeom g, const T *__restrict__ in, const T *__restrict__ w, T *__restrict__ out,
                                                    int nparts, unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int chb = (int)(lb % (unsigned)g.nchb), part = (int)(lb / (unsigned)g.nchb);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int K = g.K, KK = K * K, ob = chb * g.NS * 16;
    constexpr int VE = 16 / (int)sizeof(T);
    const int ca = cin_first(ob, g) & ~(VE - 1);
    Frag<T> *lw = reinterpret_cast<Frag<T> *>(smem);                       // [sub-block][tap][chunk][lane]
    T *lx = reinterpret_cast<T *>(lw + (size_t)g.NS * KK * g.nk * 64);
    const int npos = g.TN * g.TA * g.TB, npt = (npos + 15) / 16;

    // the filter entries in operand order, WB fragments of a lane loaded at a time; the first ones (all of a 3x3
    // filter with up to 16 input channels a group) are on their way while the first tile is staged (NHWC: 14x14
    // 16 channels a group 14.4 -> 13.3 us; in NCHW the registers they take cost a wavefront per SIMD: 57x57 bf16 67 -> 74)
    constexpr int WB = 3;
    const int nfrag = g.NS * KK * g.nk * 64;
    auto load_filter = [&](int i0, T (&e)[WB][4]) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
            const int i = i0 + b * 256, ln = i & 63, f = i >> 6, t = fdiv(f, g.rnk), kc = f - t * g.nk, s = fdiv(t, g.rKK), tap = t - s * KK;
            const int o = ob + s * 16 + (ln & 15), c0 = cin_first(ob + s * 16, g) + kc * 16 + (ln >> 4) * 4, grp = fdiv(o, g.rCgo);
            // the input channels of the output's group
            const int cg0 = grp * g.Cgi, cg1 = o < g.CO && i < nfrag ? min(cg0 + g.Cgi, g.CI) : cg0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = c0 + k;
                const int fo = g.bwd ? c : o, fc = g.bwd ? o - grp * g.Cgo : c - cg0;
                e[b][k] = T(0);
                if (c >= cg0 && c < cg1) e[b][k] = w[(unsigned)(NHWC ? (tap * g.FCg + fc) * g.FO + fo : (fo * g.FCg + fc) * KK + tap)];
            }
        }
    };
    bool wbad = false;
    auto put_filter = [&](int i0, const T (&e)[WB][4]) {
#pragma unroll
        for (int b = 0; b < WB; ++b) {
#pragma unroll
            for (int k = 0; k < 4; ++k) wbad |= nonfinite<T>(e[b][k]);
            const int i = i0 + b * 256;
            if (i >= nfrag) continue;
            if constexpr (sizeof(T) == 4) lw[i].v = make_float4(e[b][0], e[b][1], e[b][2], e[b][3]);
            else lw[i].v = make_uint2((uint32_t)e[b][0] | (uint32_t)e[b][1] << 16, (uint32_t)e[b][2] | (uint32_t)e[b][3] << 16);
        }
    };
    [[maybe_unused]] T wfirst[WB][4];
    if constexpr (NHWC) load_filter(threadIdx.x, wfirst);
    else
        for (int i0 = threadIdx.x; i0 < nfrag; i0 += WB * 256) {
            T e[WB][4];
            load_filter(i0, e);
            put_filter(i0, e);
        }

    if (!NHWC && FAST)
        for (int i = threadIdx.x; i < g.TN * g.LH * g.LW * g.pitch / VE; i += 256) reinterpret_cast<u4v_t *>(lx)[i] = u4v_t{0u, 0u, 0u, 0u};
    const int ntiles = g.tn * g.ta * g.tb, ncls = g.OS * g.OS;
    for (int tile = part; tile < ntiles; tile += nparts) {
        const int tb = tile % g.tb, ta = tile / g.tb % g.ta, tn = tile / g.tb / g.ta;
        const int n0 = tn * g.TN, a0 = g.a0 + ta * g.TA, b0 = g.b0 + tb * g.TB;
        __syncthreads();                                     // the previous tile has been read (first: nothing to wait for)
        const bool bad = stage_pixels<T, NHWC, FAST>(in, lx, g.N, g.CI, g.Hi, g.Wi, n0, g.TN, g.IS * a0 - g.ip + g.lo, g.IS * b0 - g.ip + g.lo,
                                         g.LH, g.LW, ca, g.CL, g.pitch, g.packed != 0);
        if (NHWC && tile == part) {
            put_filter(threadIdx.x, wfirst);
            for (int i0 = threadIdx.x + WB * 256; i0 < nfrag; i0 += WB * 256) {
                T e[WB][4];
                load_filter(i0, e);
                put_filter(i0, e);
            }
        }
        // One barrier behind the staging of every tile, whatever the filter and the tile hold: both paths below read pixels that other
        // wavefronts staged.  (wbad: what this lane laid out of the filter, so it counts for every tile of the block.)
        if (__builtin_expect(__syncthreads_or(wbad || bad), 0)) {
            own_group_only<T, NHWC>(g, lw, lx, out, n0, a0, b0, ob, ca);
            continue;
        }

        const int ngrp = (npt + P - 1) / P;
        const float rTA = 1.0f / (float)g.TA, rTB = 1.0f / (float)g.TB;
        for (int item = wv; item < g.NS * ngrp; item += 4) {
            const int s = item % g.NS, pg = item / g.NS;
            if (ob + s * 16 >= g.CO) continue;
            const int cl = cin_first(ob + s * 16, g) - ca + lk * 4;
            int base[P], row0[P], col0[P], img[P];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int q0 = (pg * P + p) * 16 + li, q = q0 < npos ? q0 : 0;
                const int r = fdiv(q, rTB), im = fdiv(r, rTA), da = r - im * g.TA, db = q - r * g.TB;
                base[p] = ((im * g.LH + g.IS * da - g.lo) * g.LW + g.IS * db - g.lo) * g.pitch + cl;
                img[p] = n0 + im;
                row0[p] = g.OS * (a0 + da) - g.op;
                col0[p] = g.OS * (b0 + db) - g.op;
                if (q0 >= npos || a0 + da >= g.a0 + g.na || b0 + db >= g.b0 + g.nb) img[p] = g.N;      // not a position of the image
            }
            for (int cls = 0; cls < ncls; ++cls) {
                const int f = cls / g.OS, e = cls - f * g.OS;
                v4f acc[P];
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p] = v4f{0.f, 0.f, 0.f, 0.f};
                auto tap = [&](int kh, int kw, int ro, int co) {
                    const int toff = (ro * g.LW + co) * g.pitch;
                    const Frag<T> *pw = lw + ((s * KK + kh * K + kw) * g.nk) * 64 + lane;
                    for (int kc = 0; kc < g.nk; ++kc) {
                        const Frag<T> a = pw[kc * 64];
#pragma unroll
                        for (int p = 0; p < P; ++p) {
                            const Frag<T> b = *reinterpret_cast<const Frag<T> *>(lx + base[p] + toff + kc * 16);
                            acc[p] = mma16(a, b, acc[p]);
                        }
                    }
                };
                for (int kh = f, k = 0; kh < K; kh += g.OS, ++k)
                    for (int kw = e, l = 0; kw < K; kw += g.OS, ++l) tap(kh, kw, g.bwd ? -k : kh, g.bwd ? -l : kw);
                const int o = ob + s * 16 + lk * 4;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int row = row0[p] + f, col = col0[p] + e;
                    if (img[p] >= g.N || (unsigned)row >= (unsigned)g.Ho || (unsigned)col >= (unsigned)g.Wo || o >= g.CO) continue;
                    if constexpr (NHWC) {
                        T *po = out + (unsigned)(((img[p] * g.Ho + row) * g.Wo + col) * g.CO + o);
                        const float r[4] = {acc[p][0], acc[p][1], acc[p][2], acc[p][3]};
                        if (g.CO % 4 == 0) Vec<T, 4>::store(po, r);
                        else {
#pragma unroll
                            for (int k = 0; k < 4; ++k) if (o + k < g.CO) stf(po + k, r[k]);
                        }
                    } else {
                        T *po = out + (unsigned)(((img[p] * g.CO + o) * g.Ho + row) * g.Wo + col);
#pragma unroll
                        for (int k = 0; k < 4; ++k) if (o + k < g.CO) stf(po + (unsigned)(k * g.Ho * g.Wo), acc[p][k]);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Filter gradient, stage 1.  A wavefront owns one pair of 16 output channels and 16 input channels (a "pair") and every
// WS-th step of 16 positions; a block holds NPAIR pairs and 4 / NPAIR = WS position splits, each of which is a partial.
// ---------------------------------------------------------------------------------------------
template <typename T, bool NHWC, bool FAST, int K>
__global__ __launch_bounds__(256) void k_gconv_gemm_filter(GemmGeom g, const T *__restrict__ x, const T *__restrict__ dy, float *__restrict__ ws,
                                                           int npair, int CLy, int pitchy, int nparts, int J, unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    constexpr int VE = 16 / (int)sizeof(T), KK = K * K;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int chb = (int)(lb % (unsigned)g.nchb), part = (int)(lb / (unsigned)g.nchb);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int WS = 4 / npair, pair = chb * npair + wv % npair, split = wv / npair;
    const int s = pair / g.nk, kc = pair - s * g.nk;                       // 16-channel output block, input chunk
    const int s0 = chb * npair / g.nk;
    const int cxa = (cin_first(s0 * 16, g) + (chb * npair - s0 * g.nk) * 16) & ~(VE - 1), cya = s0 * 16;
    const int cx = cin_first(s * 16, g) + kc * 16 - cxa + li, cy = s * 16 - cya + li;
    const int npos = g.TN * g.TA * g.TB, steps = (npos + 15) / 16;
    int *tab = reinterpret_cast<int *>(smem);                              // position -> LDS element of its input pixel
    T *lx = reinterpret_cast<T *>(tab + steps * 16);
    T *ly = lx + (size_t)g.TN * g.LH * g.LW * g.pitch;
    const float rTA = 1.0f / (float)g.TA, rTB = 1.0f / (float)g.TB;
    for (int p = threadIdx.x; p < steps * 16; p += 256) {
        const int q = min(p, npos - 1), r = fdiv(q, rTB), im = fdiv(r, rTA), da = r - im * g.TA, db = q - r * g.TB;
        tab[p] = ((im * g.LH + g.IS * da) * g.LW + g.IS * db) * g.pitch;
    }
    // beside the rows of x (NCHW) and behind the positions of dy: zeros
    if (!NHWC && FAST)
        for (int i = threadIdx.x; i < g.TN * g.LH * g.LW * g.pitch / VE; i += 256) reinterpret_cast<u4v_t *>(lx)[i] = u4v_t{0u, 0u, 0u, 0u};
    for (int i = threadIdx.x; i < (steps * 16 - npos) * pitchy; i += 256) ly[npos * pitchy + i] = T(0);
    // fp32: the 16 positions of a step are added up on their own before they join a sum.  A chain of n matrix instructions has a relative error of
    // about 2^-24 * sqrt(n / 6), and a 3x3 sum had up to twice the error of the kernels that these replaced (mean over random layers 1.65e-7
    // against the row walk's 1.12e-7, now 1.03e-7; 1.45e-7 against the generic kernels' 2.15e-7, now 1.02e-7), at 57x57x128 130 -> 141 us.  5x5 is
    // at 1.36e-7 against 2.38e-7 without, and has no registers for it (24 channels a group, 28x28, batch 64: 63 -> 95 us).
    constexpr bool FRESH = sizeof(T) == 4 && K <= 3;
    v4f acc[KK];
#pragma unroll
    for (int t = 0; t < KK; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    const bool live = s * 16 < g.CO;                                       // uniform: the last block may have pairs to spare

    const int ntiles = g.tn * g.ta * g.tb;
    for (int tile = part; tile < ntiles; tile += nparts) {
        const int tb = tile % g.tb, ta = tile / g.tb % g.ta, tn = tile / g.tb / g.ta;
        const int n0 = tn * g.TN, a0 = ta * g.TA, b0 = tb * g.TB;
        __syncthreads();
        stage_pixels<T, NHWC, FAST>(x, lx, g.N, g.CI, g.Hi, g.Wi, n0, g.TN, g.IS * a0 - g.ip, g.IS * b0 - g.ip, g.LH, g.LW, cxa, g.CL, g.pitch, false);
        stage_pixels<T, NHWC, FAST>(dy, ly, g.N, g.CO, g.Ho, g.Wo, n0, g.TN, a0, b0, g.TA, g.TB, cya, CLy, pitchy, false);
        __syncthreads();
        if (!live) continue;
        for (int st = split; st < steps; st += WS) {
            const int q = st * 16 + lk * 4;                                // the lane's four positions
            const int4 t4 = *reinterpret_cast<const int4 *>(tab + q);
            const T *py = ly + q * pitchy + cy, *px[4] = {lx + t4.x + cx, lx + t4.y + cx, lx + t4.z + cx, lx + t4.w + cx};
            Frag<T> d;
            gather4(d, py, py + pitchy, py + 2 * pitchy, py + 3 * pitchy);
#pragma unroll
            for (int kh = 0; kh < K; ++kh)
#pragma unroll
                for (int kw = 0; kw < K; ++kw) {
                    const int toff = (kh * g.LW + kw) * g.pitch;
                    Frag<T> b;
                    gather4(b, px[0] + toff, px[1] + toff, px[2] + toff, px[3] + toff);
                    if constexpr (FRESH) acc[kh * K + kw] += mma16(b, d, v4f{0.f, 0.f, 0.f, 0.f});
                    else acc[kh * K + kw] = mma16(b, d, acc[kh * K + kw]);
                }
        }
    }
    // lane: output s*16 + li against input channels kc*16 + lk*4 + r, so that 16 lanes write 16 consecutive outputs in NHWC
    // and a lane consecutive entries in NCHW; entries that pair different groups are dropped
    const int o = s * 16 + li, grp = fdiv(o, g.rCgo), c0 = cin_first(s * 16, g) + kc * 16 + lk * 4 - grp * g.Cgi;
    if (!live || o >= g.CO) return;
    float *dst = ws + (size_t)(part * WS + split) * J;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int ci = c0 + r;
        if ((unsigned)ci >= (unsigned)g.Cgi) continue;
        // (consecutive entries of a lane through one pointer, so that their stores merge)
        float *q = dst + (unsigned)(NHWC ? ci * g.FO + o : (o * g.FCg + ci) * KK);
        const unsigned tstep = NHWC ? (unsigned)(g.FCg * g.FO) : 1u;
#pragma unroll
        for (int t = 0; t < KK; ++t) q[NHWC ? t * tstep : t] = acc[t][r];
    }
}

// ---- host side --------------------------------------------------------------------------------

int cdivg(int a, int b) { return (a + b - 1) / b; }

// channel chunks of 16 that the inputs of any 16 consecutive outputs span, and the channels in LDS of `ns` such blocks
void channel_span(GemmGeom &g, int ns, int VE, int *CL)
{
    int nk = 1;
    auto first = [&](int o) { return o / g.Cgo * g.Cgi & ~3; };
    for (int o = 0; o < g.CO; o += 16) {
        const int end = ((o + 15 < g.CO ? o + 15 : g.CO - 1) / g.Cgo + 1) * g.Cgi;
        if (cdivg(end - first(o), 16) > nk) nk = cdivg(end - first(o), 16);
    }
    g.nk = nk;
    int cl = 0;
    for (int o = 0; o < g.CO; o += 16 * ns) {
        const int ca = first(o) & ~(VE - 1);
        for (int s = 0; s < ns && o + s * 16 < g.CO; ++s)
            if (first(o + s * 16) + nk * 16 - ca > cl) cl = first(o + s * 16) + nk * 16 - ca;
    }
    *CL = cdivg(cl, 8) * 8;
}

constexpr size_t GEMM_LDS = 64 << 10;

// positions of a tile: whole rows where they fit, several images of a small map
void pick_positions(GemmGeom &g, int want, int maxb)
{
    g.TB = g.nb < maxb ? g.nb : cdivg(g.nb, cdivg(g.nb, maxb));
    g.TA = want / g.TB;
    if (g.TA < 1) g.TA = 1;
    if (g.TA >= g.na) {
        g.TA = g.na;
        g.TN = want / (g.TA * g.TB);
        if (g.TN < 1) g.TN = 1;
        if (g.TN > g.N) g.TN = g.N;
    } else {
        g.TN = 1;
        g.TA = cdivg(g.na, cdivg(g.na, g.TA));
    }
    g.tn = cdivg(g.N, g.TN); g.ta = cdivg(g.na, g.TA); g.tb = cdivg(g.nb, g.TB);
}

struct GemmPlan { GemmGeom g; size_t lds; int nparts; unsigned nblocks; int npair, CLy, pitchy; bool fast; };

bool gemm_plan(const GGeom &q, int layout, int dtype, int pass, GemmPlan *pl)
{
    const int esz = dtype == DT_F32 ? 4 : 2, VE = 16 / esz;
    if (q.C > 65536 || q.O > 65536 || q.s > 4 || q.K > 7) return false;
    GemmGeom g = {};
    g.N = q.N; g.K = q.K; g.FO = q.O; g.FCg = q.Cg; g.bwd = pass == 1;
    if (pass != 1) {
        g.CI = q.C; g.CO = q.O; g.Hi = q.H; g.Wi = q.W; g.Ho = q.Ho; g.Wo = q.Wo; g.Cgi = q.Cg; g.Cgo = q.Og;
        g.IS = q.s; g.OS = 1; g.ip = q.p; g.op = 0; g.lo = 0;
        g.a0 = g.b0 = 0; g.na = q.Ho; g.nb = q.Wo;
    } else {
        g.CI = q.O; g.CO = q.C; g.Hi = q.Ho; g.Wi = q.Wo; g.Ho = q.H; g.Wo = q.W; g.Cgi = q.Og; g.Cgo = q.Cg;
        g.IS = 1; g.OS = q.s; g.ip = 0; g.op = q.p; g.lo = -((q.K + q.s - 1) / q.s - 1);
        g.a0 = g.b0 = q.p / q.s; g.na = (q.H - 1 + q.p) / q.s - g.a0 + 1; g.nb = (q.W - 1 + q.p) / q.s - g.b0 + 1;
    }
    const int reach = pass == 1 ? 1 - g.lo : q.K;                           // input rows of one position
    const int blocks16 = cdivg(g.CO, 16);
    if (pass < 2) {
        // output blocks of 16 per block: two where they read the same input channels (7x7 32 channels a group, batch 64, 1024
        // channels: bf16 NHWC 24 -> 21 us, fp32 NCHW 71 -> 54), otherwise one (14x14 16 channels a group, bf16 NHWC batch 32 15.6 us
        // with two, 14.4 with one; 56x56 24 channels a group 77 against 49)
        int ns = g.Cgo % 32 == 0 ? 2 : 1;
        if (ns > blocks16) ns = blocks16;
        for (;; ns = (ns + 1) / 2) {
            g.NS = ns;
            channel_span(g, ns, VE, &g.CL);
            g.packed = !(g.Cgo % 16 == 0 && g.Cgi % 16 == 0);
            g.pitch = g.CL + VE;
            for (int want = 256; want >= 16; want /= 2) {
                pick_positions(g, want, layout == LAYOUT_NHWC ? 32 : 64);
                g.LH = g.IS * (g.TA - 1) + reach; g.LW = g.IS * (g.TB - 1) + reach;
                pl->lds = (size_t)ns * q.K * q.K * g.nk * 64 * 4 * esz + (size_t)g.TN * g.LH * g.LW * g.pitch * esz;
                if (pl->lds <= GEMM_LDS) goto fits;
            }
            if (ns == 1) return false;
        }
    fits:
        g.nchb = cdivg(blocks16, g.NS);
        const long long tiles = (long long)g.tn * g.ta * g.tb;
        // the filter is laid out once per block: up to 2048 blocks, the tiles of a channel block shared among them
        long long parts = 2048 / g.nchb;
        if (parts < 1) parts = 1;
        if (parts > tiles) parts = tiles;
        parts = (tiles + (tiles + parts - 1) / parts - 1) / ((tiles + parts - 1) / parts);
        pl->nparts = (int)parts;
        pl->nblocks = (unsigned)(parts * g.nchb);
    } else {
        if (q.K > 5) return false;
        int dummy;
        channel_span(g, 1, VE, &dummy);
        const int pairs = blocks16 * g.nk;
        int npair = 4;
        while (npair > pairs) npair /= 2;
        bool fits = false;
        for (; npair >= 1 && !fits; npair /= 2) {
            pl->npair = npair;
            g.nchb = cdivg(pairs, npair);
            // channels in LDS of any block: its pairs run over (output block, chunk)
            int clx = 0, cly = 0;
            auto first = [&](int o) { return o / g.Cgo * g.Cgi & ~3; };
            for (int b = 0; b < g.nchb; ++b) {
                const int s0 = b * npair / g.nk, cxa = (first(s0 * 16) + (b * npair - s0 * g.nk) * 16) & ~(VE - 1);
                for (int j = 0; j < npair && b * npair + j < pairs; ++j) {
                    const int s = (b * npair + j) / g.nk, kc = b * npair + j - s * g.nk;
                    const int lowx = first(s * 16) + kc * 16;
                    if (lowx < cxa) { clx = 1 << 20; break; }
                    if (lowx + 16 - cxa > clx) clx = lowx + 16 - cxa;
                    if (s * 16 + 16 - s0 * 16 > cly) cly = s * 16 + 16 - s0 * 16;
                }
            }
            if (clx >= 1 << 20) continue;
            g.CL = cdivg(clx, 8) * 8; pl->CLy = cly;
            g.pitch = g.CL + VE; pl->pitchy = cly + VE;
            // tiles of fewer than 64 positions only if nothing else fits
            for (int want = 256; want >= (npair > 1 ? 64 : 16) && !fits; want /= 2) {
                pick_positions(g, want, layout == LAYOUT_NHWC ? 32 : 64);
                g.LH = g.IS * (g.TA - 1) + q.K; g.LW = g.IS * (g.TB - 1) + q.K;
                const int npos = g.TN * g.TA * g.TB, padded = (npos + 15) / 16 * 16;
                pl->lds = (size_t)padded * 4 + ((size_t)g.TN * g.LH * g.LW * g.pitch + (size_t)padded * pl->pitchy) * esz;
                fits = pl->lds <= GEMM_LDS;
            }
            if (fits) break;
        }
        if (!fits) return false;
        const long long tiles = (long long)g.tn * g.ta * g.tb, J = (long long)q.O * q.Cg * q.K * q.K;
        const int WS = 4 / npair;
        long long parts = 2048 / g.nchb;
        if (parts > tiles) parts = tiles;
        const long long most = (16ll << 20) / (WS * J * 4);
        if (parts > most) parts = most;
        if (parts < 1) parts = 1;
        if (WS * J * 4 > (64ll << 20)) return false;
        parts = (tiles + (tiles + parts - 1) / parts - 1) / ((tiles + parts - 1) / parts);
        pl->nparts = (int)parts;
        pl->nblocks = (unsigned)(parts * g.nchb);
    }
    g.rCgi = 1.0f / (float)g.Cgi; g.rCgo = 1.0f / (float)g.Cgo; g.rKK = 1.0f / (float)(q.K * q.K); g.rnk = 1.0f / (float)g.nk;
    pl->fast = layout == LAYOUT_NHWC ? q.C % VE == 0 && q.O % VE == 0 : g.tb == 1;
    pl->g = g;
    return true;
}

}  // namespace

bool gconv_gemm_supported(const GGeom &g, int layout, int dtype, int pass)
{
    GemmPlan pl;
    if (pass == 2 && g.K != 1 && g.K != 3 && g.K != 5) return false;
    return gemm_plan(g, layout, dtype, pass, &pl);
}

// Rounds of blocks, each as long as laying out the filter (three fragments of a lane at a time), then for every tile a fixed latency, the
// staging (16 bytes of a lane at a time) and the matrix instructions of its wavefronts.  Fitted to 36 000 random layers: four of five between
// 0.65 and 1.2 times the measured time.
double gconv_gemm_us(const GGeom &q, int layout, int dtype, int pass, int *positions, int *tiles)
{
    GemmPlan pl;
    if (!gemm_plan(q, layout, dtype, pass, &pl)) { *positions = *tiles = 0; return 1e30; }
    const GemmGeom &g = pl.g;
    const int npos = g.TN * g.TA * g.TB, ntiles = g.tn * g.ta * g.tb, esz = dtype == DT_F32 ? 4 : 2;
    *positions = npos;
    *tiles = cdivg(ntiles, pl.nparts);
    const size_t resident = pl.lds ? 163840 / pl.lds : 8;
    const double per_round = 256.0 * (double)(resident < 1 ? 1 : resident > 8 ? 8 : resident);
    const double rounds = pl.nblocks > per_round ? pl.nblocks / per_round : 1.0;
    const double layout_us = (layout == LAYOUT_NCHW ? 1.4 : 0.9) * cdivg(g.NS * g.K * g.K * g.nk * 64, 768);
    const double staging = (double)g.TN * g.LH * g.LW * g.CL * esz / 16 / 256;
    const double products = (double)cdivg(g.NS * cdivg(cdivg(npos, 16), 4), 4) * g.K * g.K * g.nk;
    return rounds * (layout_us + *tiles * ((pass == 0 ? 7.0 : 8.4) + 0.3 * staging + (dtype == DT_F32 ? 0.36 : 0.17) * products));
}

int gconv_gemm_parts(const GGeom &g, int layout, int dtype)
{
    GemmPlan pl;
    return gemm_plan(g, layout, dtype, 2, &pl) ? pl.nparts * (4 / pl.npair) : 0;
}

void gconv_gemm_filter_tiles(const GGeom &g, int layout, int dtype, FilterGradSrc *f)
{
    GemmPlan pl;
    gemm_plan(g, layout, dtype, 2, &pl);
    f->TN = pl.g.TN; f->TA = pl.g.TA; f->TB = pl.g.TB;
    f->tn = pl.g.tn; f->ta = pl.g.ta; f->tb = pl.g.tb;
    f->per = 0; f->nparts = pl.nparts; f->splits = 4 / pl.npair;
}

template <typename T, bool NHWC>
static hipError_t gemm_go(const GemmPlan &pl, const void *in, const void *w, void *out, hipStream_t st)
{
    auto kernel = pl.fast ? k_gconv_gemm<T, NHWC, true, 4> : k_gconv_gemm<T, NHWC, false, 4>;
    hipLaunchKernelGGL(kernel, dim3(pl.nblocks), dim3(256), pl.lds, st, pl.g, (const T *)in, (const T *)w, (T *)out,
                       pl.nparts, pl.nblocks);
    return hipGetLastError();
}
hipError_t gconv_gemm(const GGeom &q, int layout, int dtype, const void *in, const void *w, void *out, bool bwd, hipStream_t st)
{
    GemmPlan pl;
    if (!gemm_plan(q, layout, dtype, bwd ? 1 : 0, &pl)) return hipErrorInvalidValue;
    if (dtype == DT_F32) return layout == LAYOUT_NHWC ? gemm_go<float, true>(pl, in, w, out, st) : gemm_go<float, false>(pl, in, w, out, st);
    return layout == LAYOUT_NHWC ? gemm_go<bf16_t, true>(pl, in, w, out, st) : gemm_go<bf16_t, false>(pl, in, w, out, st);
}

template <typename T, bool NHWC>
static hipError_t gemm_filter_go(const GemmPlan &pl, const void *x, const void *dy, float *ws, hipStream_t st)
{
    const int J = pl.g.FO * pl.g.FCg * pl.g.K * pl.g.K;
    auto kernel = pl.fast ? (pl.g.K == 1 ? k_gconv_gemm_filter<T, NHWC, true, 1> : pl.g.K == 3 ? k_gconv_gemm_filter<T, NHWC, true, 3> : k_gconv_gemm_filter<T, NHWC, true, 5>)
                          : (pl.g.K == 1 ? k_gconv_gemm_filter<T, NHWC, false, 1> : pl.g.K == 3 ? k_gconv_gemm_filter<T, NHWC, false, 3> : k_gconv_gemm_filter<T, NHWC, false, 5>);
    hipLaunchKernelGGL(kernel, dim3(pl.nblocks), dim3(256), pl.lds, st, pl.g, (const T *)x, (const T *)dy, ws, pl.npair, pl.CLy, pl.pitchy,
                       pl.nparts, J, pl.nblocks);
    return hipGetLastError();
}
hipError_t gconv_gemm_bwd_filter(const GGeom &q, int layout, int dtype, const void *x, const void *dy, float *ws, hipStream_t st)
{
    GemmPlan pl;
    if (!gemm_plan(q, layout, dtype, 2, &pl)) return hipErrorInvalidValue;
    if (dtype == DT_F32) return layout == LAYOUT_NHWC ? gemm_filter_go<float, true>(pl, x, dy, ws, st) : gemm_filter_go<float, false>(pl, x, dy, ws, st);
    return layout == LAYOUT_NHWC ? gemm_filter_go<bf16_t, true>(pl, x, dy, ws, st) : gemm_filter_go<bf16_t, false>(pl, x, dy, ws, st);
}

}  // namespace dwc

// Group convolution on the 16x16 matrix instructions: either layout, any group size and padding, strides up to 4, K up to 7 (filter gradient:
// 5), where the filter entries of 16 outputs and the smallest tile fit the LDS of a compute unit.
//
// Forward (and the input gradient): D[o][pixel] += sum over (tap, input channel) W[o][tap, ci] * X[tap, ci][pixel], 16 output
// channels x 16 pixels per instruction, two taps or chunks of channels at a time in bf16.  A block owns up to a few times 16 output channels
// and tiles of positions; the input pixels a tile's taps reach sit in LDS as [pixel][channel] with the zero padding written out, so that for
// any stride and tap a lane's operand is four consecutive channels of one pixel: one 8-byte (bf16) or 16-byte (fp32) LDS read.  The filter
// entries are laid out in LDS once per block in operand order.  With fewer than 16 channels per group the 16 outputs span
// several groups and the entries that pair different groups are zeros; a tile that holds an infinity or NaN is then
// computed without them, so that it stays inside its group.
// Input gradient at stride s: with h + p = s*a + f and w + p = s*b + e the taps kh = f + s*k, kw = e + s*l read dy[a - k][b - l]:
// s*s classes (f, e) of output pixels, each a stride-1 convolution over the same staged dy tile.
// Filter gradient: D[o][ci] += dy[o][pixel] * X[ci][pixel + tap], the contraction over pixels, all taps in registers.
//
// What bounds it: not the matrix cores (the three passes of the 14x14 layer below need 2 us of them) nor the memory's latency (0.7 us of a
// block) but the instructions around them: laying out the filter one entry a load took a block 2 to 4 us, dividing out every staged pixel 3,
// positions of 16 lanes computed in all 64 a further one.  So the filter comes in whole vectors, a lane's place in the tile is found
// once, positions are looked up in a table, the loop over taps and chunks is one, and the next tile's loads are under way while a tile is
// computed.  us on one MI355X, one entry at a time -> now, forward / filter gradient (stage 1 and 2) / input gradient: 14x14x512, 16 channels
// a group, bf16 NHWC batch 32 15.0 / 19.7 / 17.0 -> 9.9 / 14.5 / 10.6; 56x56x256 stride 2, 8 channels a group, bf16 NCHW batch 16
// 24.9 / 31.5 / 21.8 -> 16.4 / 22.8 / 18.6; 57x57x128, 4 channels a group, fp32 NCHW batch 64 151 / 144 / 151 -> 116 / 134 / 116 (there 3 of 4
// products are zeros: 49 us of matrix instructions a pass).  A tile may take more than 64 KiB of LDS where the filter does: 28x28x512, 32
// channels a group at stride 2, fp32 NCHW batch 16, forward 81 -> 27.
// Any channel count and row width comes in vectors (16 bytes of channels at any alignment in NHWC; in NCHW tiles narrower than the rows, runs of
// four columns from the multiple of four before a tile), the NCHW filter by an entry's taps, so that a vector's place is found once, and two pairs of taps
// are read at a time: random layers 0.85 (bf16) and 0.875 (fp32) of the time in NCHW forward, 0.88 and 0.92 in the input gradient, NHWC 0.94 and 0.96,
// 0.93 and 0.98; 9x9x320 in ten groups, 5x5, bf16 NCHW batch 7, forward 15.3 -> 10.5;
// 16x16x160 in five, 5x5, fp32 NCHW batch 4, 17.6 -> 12.6.
#include "bounds.hpp"
#include "gconv.hpp"
#include <type_traits>

namespace dwc {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

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

// two fragments of each side: one instruction of 32 products in bf16
__device__ __forceinline__ v4f mma32(const Frag<float> &a0, const Frag<float> &a1, const Frag<float> &b0, const Frag<float> &b1, v4f d)
{
    return mma16(a1, b1, mma16(a0, b0, d));
}
__device__ __forceinline__ v4f mma32(const Frag<bf16_t> &a0, const Frag<bf16_t> &a1, const Frag<bf16_t> &b0, const Frag<bf16_t> &b1, v4f d)
{
    const u4v_t a = {a0.v.x, a0.v.y, a1.v.x, a1.v.y}, b = {b0.v.x, b0.v.y, b1.v.x, b1.v.y};
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a), __builtin_bit_cast(v8b, b), d, 0, 0, 0);
}

__device__ __forceinline__ void gather4(Frag<float> &f, const float *a, const float *b, const float *c, const float *d)
{
    f.v = make_float4(*a, *b, *c, *d);
}
template <typename T> __device__ __forceinline__ bool nonfinite(T v);
template <> __device__ __forceinline__ bool nonfinite<float>(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }
template <> __device__ __forceinline__ bool nonfinite<bf16_t>(bf16_t v) { return (v & 0x7f80u) == 0x7f80u; }

// Whether values, as stored, hold an infinity or NaN: their products with zero (fp32), or the largest exponent of two to a word (bf16).
template <typename T> struct Finite;
template <> struct Finite<float> {
    float m = 0.f;
    __device__ __forceinline__ void add(uint32_t q) { m = fmaf(__uint_as_float(q), 0.f, m); }
    __device__ __forceinline__ void add(const Frag<float> &f)
    {
        m = fmaf(f.v.x, 0.f, m); m = fmaf(f.v.y, 0.f, m); m = fmaf(f.v.z, 0.f, m); m = fmaf(f.v.w, 0.f, m);
    }
    __device__ __forceinline__ bool bad() const { return m != m; }
};
template <> struct Finite<bf16_t> {
    uint32_t m = 0;
    __device__ __forceinline__ void add(uint32_t q)
    {
        m = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, m), __builtin_bit_cast(u16x2, q & 0x7fff7fffu)));
    }
    __device__ __forceinline__ void add(const Frag<bf16_t> &f) { add(f.v.x); add(f.v.y); }
    __device__ __forceinline__ bool bad() const { return (m & 0xffffu) >= 0x7f80u || m >> 16 >= 0x7f80u; }
};

// V consecutive outputs at any alignment
template <typename T, int V, typename A> __device__ __forceinline__ void store_run(T *p, const A &v)
{
    if constexpr (sizeof(T) == 4) {
        float r[V];
#pragma unroll
        for (int i = 0; i < V; ++i) r[i] = v[i];
        __builtin_memcpy(p, r, sizeof r);
    } else {
        uint32_t r[V / 2];
#pragma unroll
        for (int i = 0; i < V / 2; ++i) r[i] = pack2_bf16(v[2 * i], v[2 * i + 1]);
        __builtin_memcpy(p, r, sizeof r);
    }
}

// n / d for 0 <= n < 2^21 and d with reciprocal r = 1.0f / d: the half keeps the product away from the integers by more than
// its rounding error (0.5 / d against n / d * 2^-22), four instructions instead of the twenty of an integer division.
__device__ __forceinline__ int fdiv(int n, float r) { return (int)(((float)n + 0.5f) * r); }

__device__ __forceinline__ int uniform_div(int n, float r) { return __builtin_amdgcn_readfirstlane(fdiv(n, r)); }

__device__ __forceinline__ int cin_first(int o0, const GemmGeom &g) { return fdiv(o0, g.rCgo) * g.Cgi & ~3; }

// Input pixels of a tile to LDS as [image][row][column][channel]; what lies outside the image or the tensor's channels is
// written as zero.  Any channel count, any width.  Returns whether the lane staged an infinity or NaN.
template <typename T, bool NHWC>
__device__ __forceinline__ bool stage_pixels(const T *__restrict__ in, T *lx, int N, int C, int H, int W, int n0, int nimg, int h0, int w0,
                                             int LH, int LW, int ca, int CL, int pitch, bool check)
{
    bool bad = false;
    const int npix = nimg * LH * LW;
    const float rLW = __builtin_amdgcn_rcpf((float)LW), rLH = __builtin_amdgcn_rcpf((float)LH);
    // image, row and column of a staged pixel; false if it lies outside
    auto locate = [&](int pix, int &n, int &h, int &w) {
        const int r = fdiv(pix, rLW), im = fdiv(r, rLH);
        n = n0 + im; h = r - im * LH + h0; w = pix - r * LW + w0;
        return n < N && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W;
    };
    // every lane has B loads in flight before its first LDS write
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

// The same where FAST holds, in two steps: load() sends out the loads of BT items of a lane, commit() writes them to LDS, so that the
// next tile is on its way while this one is computed.
// FAST: 1, channels of whole vectors (NHWC), tiles of whole rows (NCHW); 2, ragged channels, or tiles narrower than the rows.
// LATE: what the loads at a tensor's end need is done in commit() (not in the filter gradient: its registers are at the limit, 125 -> 131 in fp32 NCHW).
template <typename T, bool NHWC, int FAST, int BT, bool LATE> struct Stager;

// The elements of 16 (or eight) bytes from element n on.
template <int VE, typename Q> __device__ __forceinline__ Q later(Q q, int n)
{
    constexpr int WORDS = (int)sizeof(Q) / 4;
    if constexpr (VE == 4 && WORDS == 2) return __builtin_bit_cast(Q, __builtin_bit_cast(uint64_t, q) >> 16 * n);
    if constexpr (VE == WORDS) {
        if (n & 1) {
#pragma unroll
            for (int i = 0; i + 1 < WORDS; ++i) q[i] = q[i + 1];
        }
    } else if (n & 1) {
#pragma unroll
        for (int i = 0; i < WORDS; ++i) q[i] = q[i] >> 16 | (i + 1 < WORDS ? q[i + 1] << 16 : 0u);
    }
#pragma unroll
    for (int step = VE == WORDS ? 2 : 1; step < WORDS; step *= 2)          // words
        if (n & step * (VE / WORDS)) {
#pragma unroll
            for (int i = 0; i + step < WORDS; ++i) q[i] = q[i + step];
        }
    return q;
}

template <typename T, int FAST, int BT, bool LATE> struct Stager<T, true, FAST, BT, LATE> {
    static constexpr int VE = 16 / (int)sizeof(T);
    u4raw_t q[BT];
    uint32_t late;           // per item, how far behind the start of its load it begins: seen to in commit(), where the load has been waited for
    int rsub, csub, v;
    __device__ __forceinline__ Stager(const StageGeom &sg)
    {
        rsub = fdiv(threadIdx.x, sg.rper);
        const int rem = threadIdx.x - rsub * sg.per;
        csub = fdiv(rem, sg.rnv);
        v = (rem - csub * sg.nv) * VE;
    }
    // row and column of the lane's item `it` (uniform); false if it has none
    __device__ __forceinline__ bool locate(const StageGeom &sg, int it, int &r, int &col) const
    {
        col = csub;
        while (it >= sg.nrit) { it -= sg.nrit; col += sg.cols; }
        r = it * sg.RPI + rsub;
        return rsub < sg.RPI && r < sg.rows && col < sg.LW;
    }
    // nimg images from element `first` of `in` on, a tensor of `total` elements (VE and more, below 2^31): rows from h0, columns from w0, channels from ca.
    // Channels that are no whole number of vectors: unaligned loads, whose last elements are the next pixel's first (they meet zeros of
    // the filter), at the tensor's end those before it (`late`; shifted here, every load of a launch's last images, in a batch of one every load, was
    // waited for before the next was sent out: 926x102x27 in two groups to 5556 channels, fp32, input gradient 145 -> 116 us, NCHW 864x35x107 in nine
    // forward 192 -> 143, random layers of one image 0.98 at the mean, the shortest 0.72, the longest 1.05).
    __device__ __forceinline__ void load(const StageGeom &sg, const T *__restrict__ in, unsigned first, unsigned total, int nimg, int C, int H, int W,
                                         int h0, int w0, int ca, int it0)
    {
        const BufView view(in + first, (uint32_t)(nimg * C) * (uint32_t)(H * W) * (uint32_t)sizeof(T));
        [[maybe_unused]] const bool past = first + (unsigned)(nimg * C) * (unsigned)(H * W) + VE > total;
        late = 0u;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (it0 + b >= sg.iters) break;
            int h, w, im = 0;
            bool ok = locate(sg, it0 + b, h, w);
            if (sg.rows != sg.LH) { im = fdiv(h, sg.rLH); h -= im * sg.LH; }
            h += h0; w += w0;
            ok = ok && im < nimg && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W && ca + v < C;
            // (in range every factor is below 2^24)
            const uint32_t e = __umul24(__umul24(__umul24(im, H) + h, W) + w, C) + ca + v;
            if constexpr (FAST == 1) q[b] = view.b128(ok ? e * (uint32_t)sizeof(T) : BufView::OUTSIDE, 0);
            else {
                q[b] = u4raw_t{0u, 0u, 0u, 0u};
                if (ok) {
                    const unsigned p = first + e, at = min(p, total - VE);
                    __builtin_memcpy(&q[b], in + at, 16);
                    if (past) {
                        if constexpr (LATE) late |= (p - at) << 3 * b;
                        else q[b] = later<VE>(q[b], (int)(p - at));
                    }
                }
            }
        }
    }
    __device__ __forceinline__ void commit(const StageGeom &sg, T *lx, int, int, int it0, bool check, Finite<T> &seen)
    {
        if (FAST == 2 && LATE && late != 0u) {
#pragma unroll
            for (int b = 0; b < BT; ++b) q[b] = later<VE>(q[b], (int)(late >> 3 * b & 7u));
        }
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (it0 + b >= sg.iters) break;
            int r, col;
            const bool ok = locate(sg, it0 + b, r, col);
            if (check) {
#pragma unroll
                for (int k = 0; k < 4; ++k) seen.add(q[b][k]);
            }
            if (ok) *reinterpret_cast<u4raw_t *>(lx + __umul24(__umul24(r, sg.LW) + col, sg.pitch) + v) = q[b];
        }
    }
};

// Four channels of four consecutive columns of a row, transposed in registers.  Where a tile holds whole rows, the columns beside the row are
// zero from the start and stay so; where it is narrower, its runs of four start at the multiple of four before it and bring their own zeros.
template <typename T, int FAST, int BT, bool LATE> struct Stager<T, false, FAST, BT, LATE> {
    static constexpr int NW = (int)sizeof(T);      // 32-bit words of four columns
    typedef uint32_t word_t __attribute__((ext_vector_type(NW)));
    word_t e[BT][4];
    uint32_t late;           // per item and channel, as above
    int rsub, csub;
    __device__ __forceinline__ Stager(const StageGeom &sg)
    {
        rsub = fdiv(threadIdx.x, sg.rper);
        csub = threadIdx.x - rsub * sg.per;
    }
    // row of all channel quads and first column of the run of four; w0: the tile's first column
    __device__ __forceinline__ bool locate(const StageGeom &sg, int it, int W, int w0, int &r, int &col) const
    {
        int run = csub;
        while (it >= sg.nrit) { it -= sg.nrit; run += sg.cols; }
        r = it * sg.RPI + rsub;
        col = (FAST == 2 ? w0 & ~3 : 0) + run * 4;
        return rsub < sg.RPI && r < sg.rows && (FAST == 2 ? run < sg.width : col < W);
    }
    // nimg images from element `first` of `in` on, a tensor of `total` elements (four and more, below 2^31)
    __device__ __forceinline__ void load(const StageGeom &sg, const T *__restrict__ in, unsigned first, unsigned total, int nimg, int C, int H, int W,
                                         int h0, int w0, int ca, int it0)
    {
        const unsigned plane = (unsigned)(H * W);
        const bool past = W % 4 && runs_past(first + (unsigned)(nimg * C) * plane, total);        // of this tile or, up to two elements, the ones behind
        late = 0u;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (it0 + b >= sg.iters) break;
            int h, col, im = 0, qd = 0;
            bool ok = locate(sg, it0 + b, W, w0, h, col);
            if (sg.rows != sg.imrows) { qd = fdiv(h, sg.rimrows); h -= qd * sg.imrows; }
            if (sg.imrows != sg.LH) { im = fdiv(h, sg.rLH); h -= im * sg.LH; }
            h += h0;
            const int c = ca + qd * 4;
            ok = ok && im < nimg && (unsigned)h < (unsigned)H && (FAST == 1 || (unsigned)col < (unsigned)W) && c < C;
            unsigned p0 = first + (unsigned)(im * C + c) * plane + (unsigned)(h * W + col);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < NW; ++j) e[b][k][j] = 0u;
            if (ok) {
                // (channels behind the last one meet zeros of the filter: the last one again)
#pragma unroll
                for (int k = 0; k < 4; ++k, p0 += c + k < C ? plane : 0u) {
                    // any alignment; a run that passes the row's end reads the elements behind it, at the tensor's end those before it
                    const unsigned at = run_start(p0, total);
                    __builtin_memcpy(&e[b][k], in + at, 4 * sizeof(T));
                    if (past) {
                        if constexpr (LATE) late |= (p0 - at) << (b * 4 + k) * 2;
                        else e[b][k] = later<4>(e[b][k], (int)(p0 - at));
                    }
                }
            }
        }
    }
    // w0: the tile's first column
    __device__ __forceinline__ void commit(const StageGeom &sg, T *lx, int W, int w0, int it0, bool check, Finite<T> &seen)
    {
        if (LATE && late != 0u) {
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int k = 0; k < 4; ++k) e[b][k] = later<4>(e[b][k], (int)(late >> (b * 4 + k) * 2 & 3u));
        }
        const bool whole = FAST == 1 && W % 4 == 0 && w0 <= 0 && W - w0 <= sg.LW;                // every column of a run is one of the tile
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (it0 + b >= sg.iters) break;
            int r, col, qd = 0;
            const bool ok = locate(sg, it0 + b, W, w0, r, col);
            if (sg.rows != sg.imrows) { qd = fdiv(r, sg.rimrows); r -= qd * sg.imrows; }
            const int n = ok ? W - col : 0;                        // columns of the run inside the row
            col -= w0;
            T *at = lx + ((int)__umul24(r, sg.LW) + col) * sg.pitch + qd * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                Frag<T> f;
                if constexpr (sizeof(T) == 4)
                    f.v = make_float4(__uint_as_float(e[b][0][j]), __uint_as_float(e[b][1][j]), __uint_as_float(e[b][2][j]), __uint_as_float(e[b][3][j]));
                else {
                    const uint32_t sel = j & 1 ? 0x07060302u : 0x05040100u;
                    f.v = make_uint2(__builtin_amdgcn_perm(e[b][1][j / 2], e[b][0][j / 2], sel), __builtin_amdgcn_perm(e[b][3][j / 2], e[b][2][j / 2], sel));
                }
                if (FAST == 2 && j >= n) f.v = decltype(f.v){};
                if (whole ? n > 0 : (FAST == 2 ? ok : j < n) && (unsigned)(col + j) < (unsigned)sg.LW) {
                    if (check) {
                        seen.add(f);
                    }
                    *reinterpret_cast<Frag<T> *>(at + j * sg.pitch) = f;
                }
            }
        }
    }
};

// QUAD: fragments between quads of input channels.  NCHW: 17, one more than there are, where that costs no block on a compute unit, so that the entries that
// the lanes of a wavefront lay out (taps and channels of a few outputs) lie in different banks: bf16 0.955 of the time forward and 0.977 backward, fp32 0.987 and
// 1.003 (mean over random layers); always 17, a large filter left smaller tiles or fewer blocks (fp32 160x19x19 in one group, batch 30, 144 us with 16, 284
// with 17; 80 and more channels a group 25 % longer by more than 8 %, 7x7 9 %).  NHWC: 16, lanes write consecutive outputs (17: 1.00 in bf16, and 1.016 in fp32,
// whose tiles get smaller).

// A tile that holds an infinity or NaN where 16 outputs span several groups, or whose filter does: one output per lane, its own
// group's channels and the taps inside the image only.
template <typename T, bool NHWC, int QUAD>
__device__ __forceinline__ void own_group_only(const GemmGeom &g, const Frag<T> *lw, const int *slots, const T *lx, T *__restrict__ out, int n0, int a0,
                                                         int b0, int ob, int ca)
{
    const int npos = g.TN * g.TA * g.TB, nch = g.NS * 16, KK = g.K * g.K;
#pragma unroll 1
    for (int i = threadIdx.x; i < g.OS * g.OS * npos * nch; i += 256) {
        const int oc = i % nch, q = i / nch % npos, cls = i / nch / npos;
        const int f = cls / g.OS, e = cls - f * g.OS, im = q / (g.TA * g.TB), da = q / g.TB % g.TA, db = q % g.TB;
        const int sh = g.pairs && e == 0 ? g.shift : 0;
        const int o = ob + oc, row = g.OS * (a0 + da) + f - g.op, col = g.OS * (b0 + db + sh) + e - g.op;
        if (o >= g.CO || n0 + im >= g.N || a0 + da >= g.a0 + g.na || b0 + db >= g.b0 + g.nb || (unsigned)row >= (unsigned)g.Ho ||
            (unsigned)col >= (unsigned)g.Wo) continue;
        const int s = oc / 16, c0 = o / g.Cgo * g.Cgi, cs = cin_first(ob + s * 16, g);
        float acc = 0.f;
#pragma unroll 1
        for (int kh = f, k = 0; kh < g.K; kh += g.OS, ++k)
#pragma unroll 1
            for (int kw = e, l = 0; kw < g.K; kw += g.OS, ++l) {
                const int ro = g.bwd ? -k : kh, co = g.bwd ? -l : kw;
                if ((unsigned)(g.IS * (a0 + da) - g.ip + ro) >= (unsigned)g.Hi || (unsigned)(g.IS * (b0 + db + sh) - g.ip + co) >= (unsigned)g.Wi) continue;
                const T *px = lx + ((im * g.LH + g.IS * da + ro - g.lo) * g.LW + g.IS * (db + sh) + co - g.lo) * g.pitch;
#pragma unroll 1
                for (int c = c0; c < c0 + g.Cgi; ++c) {
                    const int j = c - cs;
                    const T *pw = reinterpret_cast<const T *>(&lw[((s * KK + (slots ? slots[kh * g.K + kw] : kh * g.K + kw)) * g.nk + j / 16) * (4 * QUAD) + j % 16 / 4 * QUAD + oc % 16]);
                    acc = fmaf(ldf(pw + j % 4), ldf(px + c - ca), acc);
                }
            }
        stf(out + (NHWC ? (((size_t)(n0 + im) * g.Ho + row) * g.Wo + col) * g.CO + o : (((size_t)(n0 + im) * g.CO + o) * g.Ho + row) * g.Wo + col), acc);
    }
}

// ---------------------------------------------------------------------------------------------
// The filter in LDS, in operand order: fragment [output block s][tap][chunk][lane] holds output s*16 + lane%16 against the input channels
// chunk*16 + lane/16*4 .. +3 from cin_first of the block on.  FAST: 16 bytes of the filter a lane and load, each entry then written where it
// belongs (one entry a load, gathered in operand order, cost a 14x14 layer of 16 channels a group 2 us forward and 4 us backward of its 13).
// ---------------------------------------------------------------------------------------------
template <typename T, bool NHWC, bool BWD, int FAST, int QUAD> struct FilterLoader {
    static constexpr int VE = 16 / (int)sizeof(T);
    const GemmGeom &g;
    int ob, KK;
    int g0, g1;              // groups of the block's outputs
    int fc0, X;              // the places in a group that are read (forward: all input channels, backward: those of the block's outputs)
    int nvr, nvec;           // vectors of a row (NCHW: of an entry's taps), of all rows
    float rnvr, rX;
    unsigned first, total;   // element that the first vector starts at; of the filter

    // Of the shapes that takes() admits, a block takes vectors where they are no more than its fragments (NCHW, where nine taps are three vectors in
    // fp32: half as many again).  Backward a block whose outputs lie in two
    // groups reads the groups' whole filter, which has no bound (12001 channels against 256: 27 million entries, beyond what fdiv divides) and
    // keeps the launch waiting: us, such blocks by vectors too -> not, bf16 NHWC 4x560x5x5 in two groups, 1x1, 36 -> 17.
    // NCHW needs at least a vector's taps, the filter a vector's entries.
    static __device__ __forceinline__ bool takes(const GemmGeom &g)
    {
        if (!NHWC) return g.K * g.K >= VE;
        return FAST != 2 || (unsigned)(g.FO * g.FCg * g.K * g.K) >= VE;
    }

    const int *slots;        // where a tap's entries go (null: in order)

    __device__ __forceinline__ FilterLoader(const GemmGeom &geom, int ob_, const int *slots_) : g(geom), ob(ob_), KK(geom.K * geom.K), slots(slots_)
    {
        const int olast = min(ob + g.NS * 16, g.CO) - 1;
        g0 = fdiv(ob, g.rCgo); g1 = fdiv(olast, g.rCgo);
        fc0 = 0; X = g.FCg;
        if (BWD && g0 == g1) { fc0 = ob - g0 * g.Cgo; X = olast + 1 - ob; }
        int rows;
        if (NHWC) {
            // rows of (tap, place in the group): forward the block's outputs, backward the groups' input channels
            first = BWD ? (unsigned)(g0 * g.Cgi) & ~(unsigned)(VE - 1) : (unsigned)ob;
            nvr = BWD ? (int)((g1 + 1) * g.Cgi - first + VE - 1) / VE : g.NS * 16 / VE;
            rows = KK * X;
        } else {
            // rows of (output or, backward, input channel; place in the group): its taps, the last vector ending with the last one
            first = (unsigned)((BWD ? g0 * g.Cgi : ob) * g.FCg + fc0) * KK;
            nvr = (KK + VE - 1) / VE;
            rows = (BWD ? (g1 - g0 + 1) * g.Cgi : olast + 1 - ob) * X;
        }
        total = (unsigned)(g.FO * g.FCg * KK);
        nvec = rows * nvr;
        rnvr = __builtin_amdgcn_rcpf((float)nvr); rX = __builtin_amdgcn_rcpf((float)X);
    }
    __device__ __forceinline__ u4raw_t load(const T *__restrict__ w, int i) const
    {
        u4raw_t q = u4raw_t{0u, 0u, 0u, 0u};
        if (i >= nvec) return q;
        const int row = fdiv(i, rnvr), v = (i - row * nvr) * VE;
        if constexpr (NHWC) {
            unsigned at = (unsigned)row;
            if (BWD) { const int tap = fdiv(row, rX); at = (unsigned)(tap * g.FCg + fc0 + row - tap * X); }
            // (a vector beyond a row's end holds the next row's first entries, which put() leaves out)
            if ((int)first + v < g.FO) {
                const unsigned p = at * (unsigned)g.FO + first + v;
                if constexpr (FAST == 1) q = *reinterpret_cast<const u4raw_t *>(w + p);
                else {
                    const unsigned from = min(p, total - VE);
                    __builtin_memcpy(&q, w + from, 16);
                    if (from != p) q = later<VE>(q, (int)(p - from));
                }
            }
        } else {
            const int r = fdiv(row, rX);
            __builtin_memcpy(&q, w + first + (unsigned)((r * g.FCg + row - r * X) * KK) + min(v, KK - VE), 16);               // any alignment
        }
        return q;
    }
    static __device__ __forceinline__ T entry(const u4raw_t &q, int j)
    {
        if constexpr (sizeof(T) == 4) return __uint_as_float(q[j]);
        else return (T)(q[j / 2] >> 16 * (j & 1));
    }
    // element of lw at which output o's entry for input channel c and tap 0 lies (both of one group); -1 if o is not the block's
    __device__ __forceinline__ int place(int o, int c) const
    {
        const int oi = o - ob, s = oi >> 4, rel = c - cin_first(ob + (s << 4), g);
        if ((unsigned)oi >= (unsigned)(g.NS * 16) || o >= g.CO) return -1;
        return (((s * KK) * g.nk + (rel >> 4)) * (4 * QUAD) + (rel >> 2 & 3) * QUAD + (oi & 15)) * 4 + (rel & 3);
    }
    __device__ __forceinline__ void put(T *lw, int i, const u4raw_t &q, Finite<T> &seen) const
    {
        if (i >= nvec) return;
        const int tstep = g.nk * (4 * QUAD) * 4;
        const int row = fdiv(i, rnvr), v = (i - row * nvr) * VE;
#pragma unroll
        for (int k = 0; k < 4; ++k) seen.add(q[k]);
        if constexpr (NHWC && !BWD) {
            const int tap = fdiv(row, rX), x = row - tap * X, o = ob + v;
            if (!g.packed) {                                                   // one group, all outputs there
                T *at = lw + place(o, fdiv(o, g.rCgo) * g.Cgi + x) + tap * tstep;
#pragma unroll
                for (int j = 0; j < VE; ++j) at[4 * j] = entry(q, j);
            } else {
                const int oi = o - ob, s = oi >> 4, c0 = cin_first(ob + (s << 4), g);
                T *at = lw + (((s * KK + tap) * g.nk) * (4 * QUAD) + (oi & 15)) * 4;
#pragma unroll
                for (int j = 0; j < VE; ++j) {
                    const int rel = fdiv(o + j, g.rCgo) * g.Cgi + x - c0;
                    if (o + j < g.CO) at[(rel >> 4) * (16 * QUAD) + (rel >> 2 & 3) * (QUAD * 4) + 4 * j + (rel & 3)] = entry(q, j);
                }
            }
        } else if constexpr (NHWC) {
            const int tap = fdiv(row, rX), x = row - tap * X, c = (int)first + v;
            T *to = lw + (slots ? slots[tap] : tap) * tstep;
            if (g.Cgi % 4 == 0) {
#pragma unroll
                for (int u = 0; u < VE; u += 4) {
                    const int grp = fdiv(c + u, g.rCgi), at = place(grp * g.Cgo + fc0 + x, c + u);
                    if (at < 0 || grp < g0 || grp > g1) continue;
                    Frag<T> f;
                    if constexpr (sizeof(T) == 4) f.v = make_float4(entry(q, 0), entry(q, 1), entry(q, 2), entry(q, 3));
                    else f.v = make_uint2(q[u / 2], q[u / 2 + 1]);
                    *reinterpret_cast<Frag<T> *>(to + at) = f;
                }
            } else {
#pragma unroll
                for (int j = 0; j < VE; ++j) {
                    const int grp = fdiv(c + j, g.rCgi), at = place(grp * g.Cgo + fc0 + x, c + j);
                    if (at >= 0 && grp >= g0 && grp <= g1) to[at] = entry(q, j);
                }
            }
        } else {
            const int r = fdiv(row, rX), x = row - r * X, tap = min(v, KK - VE);
            int at;
            if (!BWD) at = place(ob + r, fdiv(ob + r, g.rCgo) * g.Cgi + x);
            else at = place((g0 + fdiv(r, g.rCgi)) * g.Cgo + fc0 + x, g0 * g.Cgi + r);
            if (at < 0) return;
#pragma unroll
            for (int j = 0; j < VE; ++j) lw[at + (BWD && slots ? slots[tap + j] : tap + j) * tstep] = entry(q, j);
        }
    }
};

// ---------------------------------------------------------------------------------------------
// Forward and input gradient.  SCATTER: NCHW outputs that are not consecutive (strides of the input gradient).  P: 16-pixel tiles that a wavefront computes at a time against one read of the filter.  E = 2: the
// input gradient at stride 2 in NCHW, both columns of a pair of output classes at a time, so that a lane's four positions are eight
// consecutive outputs (aligned for rows of whole vectors: with an odd padding the pair is class 1 of a position and class 0 of the next).
// ---------------------------------------------------------------------------------------------
template <typename T, bool NHWC, bool BWD, int FAST, int P, int E, bool SCATTER, int QUAD>
__global__ __launch_bounds__(256, 4) void k_gconv_gemm(GemmGeom g, StageGeom sg, const T *__restrict__ in, const T *__restrict__ w, T *__restrict__ out,
                                                    int nparts, unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int chb = (int)(lb % (unsigned)g.nchb), part = (int)(lb / (unsigned)g.nchb);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    constexpr bool OUTER = NHWC || SCATTER;                                // a lane has four outputs of one position, otherwise one output of four
    const int OS = BWD ? g.OS : 1, IS = BWD ? 1 : g.IS;
    const int K = g.K, KK = K * K, ob = chb * g.NS * 16;
    constexpr int VE = 16 / (int)sizeof(T), CHUNK = 4 * QUAD;
    const int ca = cin_first(ob, g) & ~(VE - 1);
    Frag<T> *lw = reinterpret_cast<Frag<T> *>(smem);                       // [sub-block][tap][chunk][lane]
    const int npos = g.TN * g.TA * g.TB, ngrp = (npos + 16 * P - 1) / (16 * P), nent = ngrp * 16 * P;
    // of every position: element of its first input pixel in LDS, element of its output (-1: none; the image's first for OS > 1), and
    // for OS > 1 row and column of that
    int *tabx = reinterpret_cast<int *>(lw + (size_t)g.NS * KK * g.nk * (4 * QUAD)), *tabo = tabx + nent, *tabr = tabo + nent;
    int *slots = OS > 1 ? tabr + 2 * nent : nullptr;       // taps in the order of their classes
    int *flag = OS > 1 ? slots + 64 : tabr;                // an infinity or NaN in the filter or the tile (two, in turn)
    T *lx = reinterpret_cast<T *>(flag + 4);
    if (threadIdx.x < 2) flag[threadIdx.x] = 0;
    const int ntiles = g.tn * g.ta * g.tb;
    const int nfrag = g.NS * KK * g.nk * 64;
    const unsigned imin = (unsigned)(g.CI * g.Hi * g.Wi), imout = (unsigned)(g.CO * g.Ho * g.Wo);

    auto tile_at = [&](int tile, int &n0, int &a0, int &b0) {
        const int row = FAST ? uniform_div(tile, g.rtb) : tile / g.tb, tn = FAST ? uniform_div(row, g.rta) : row / g.ta;
        n0 = tn * g.TN; a0 = g.a0 + (row - tn * g.ta) * g.TA; b0 = g.b0 + (tile - row * g.tb) * g.TB;
    };
    constexpr int BT = NHWC || sizeof(T) == 2 ? 4 : 2;       // items of a lane in flight
    [[maybe_unused]] Stager<T, NHWC, FAST, BT, true> stager(sg);
    auto load_tile = [&](int tile, int it0) {
        if constexpr (FAST) {
            int n0, a0, b0;
            tile_at(tile, n0, a0, b0);
            const int nimg = min(g.TN, g.N - n0), h0 = IS * a0 - g.ip + g.lo, w0 = IS * b0 - g.ip + g.lo;
            stager.load(sg, in, (unsigned)n0 * imin, (unsigned)g.N * imin, nimg, g.CI, g.Hi, g.Wi, h0, w0, ca, it0);
        }
    };

    load_tile(part, 0);
    // zeros: entries that pair different groups, inputs beside the group, outputs beside the tensor; pixels beside the rows
    Finite<T> wseen;
    const FilterLoader<T, NHWC, BWD, FAST, QUAD> fl(g, ob, slots);
    const bool vectors = FAST && FilterLoader<T, NHWC, BWD, FAST, QUAD>::takes(g) && fl.nvec <= (NHWC ? nfrag : nfrag * 3 / 2);       // (see there)
    if (vectors && g.packed)
        for (int i = threadIdx.x; i < g.NS * KK * g.nk * (4 * QUAD) * 4 / VE; i += 256) reinterpret_cast<u4v_t *>(lw)[i] = u4v_t{0u, 0u, 0u, 0u};
    if (!NHWC && FAST == 1)
        for (int i = threadIdx.x; i < (g.TN * g.LH * g.LW * g.pitch + VE - 1) / VE; i += 256) reinterpret_cast<u4v_t *>(lx)[i] = u4v_t{0u, 0u, 0u, 0u};
    if (OS > 1 && (int)threadIdx.x < KK) {
        const int kh = (int)threadIdx.x / K, kw = (int)threadIdx.x - kh * K, f = kh % OS, e = kw % OS;
        auto before = [&](int f) { int n = 0; for (int i = 0; i < f; ++i) n += (K - i + OS - 1) / OS; return n; };
        const int nl = (K - e + OS - 1) / OS;
        slots[threadIdx.x] = before(f) * K + (K - f + OS - 1) / OS * before(e) + kh / OS * nl + kw / OS;
    }
    if (!NHWC || g.packed || OS > 1) __syncthreads();
    if (vectors) {
        constexpr int FB = 2;                                              // vectors of a lane in flight (four: the same)
#pragma unroll 1
        for (int i0 = threadIdx.x; i0 - (int)threadIdx.x < fl.nvec; i0 += FB * 256) {
            u4raw_t q[FB];
#pragma unroll
            for (int b = 0; b < FB; ++b) q[b] = fl.load(w, i0 + b * 256);
#pragma unroll
            for (int b = 0; b < FB; ++b) fl.put(reinterpret_cast<T *>(lw), i0 + b * 256, q[b], wseen);
        }
    } else {
        // four entries of a fragment at a time, in operand order
#pragma unroll 1
        for (int i = threadIdx.x; i < nfrag; i += 256) {
            const int ln = i & 63, f = i >> 6, t = fdiv(f, g.rnk), kc = f - t * g.nk, s = fdiv(t, g.rKK), tap = t - s * KK;
            const int o = ob + s * 16 + (ln & 15), c0 = cin_first(ob + s * 16, g) + kc * 16 + (ln >> 4) * 4, grp = fdiv(o, g.rCgo);
            // the input channels of the output's group
            const int cg0 = grp * g.Cgi, cg1 = o < g.CO ? min(cg0 + g.Cgi, g.CI) : cg0;
            T e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = c0 + k;
                const int fo = BWD ? c : o, fc = BWD ? o - grp * g.Cgo : c - cg0;
                e[k] = T(0);
                if (c >= cg0 && c < cg1) e[k] = w[(unsigned)(NHWC ? (tap * g.FCg + fc) * g.FO + fo : (fo * g.FCg + fc) * KK + tap)];
            }
            Frag<T> q;
            if constexpr (sizeof(T) == 4) {
                q.v = make_float4(e[0], e[1], e[2], e[3]);
#pragma unroll
                for (int k = 0; k < 4; ++k) wseen.add(__float_as_uint(e[k]));
            } else {
                q.v = make_uint2((uint32_t)e[0] | (uint32_t)e[1] << 16, (uint32_t)e[2] | (uint32_t)e[3] << 16);
                wseen.add(q.v.x); wseen.add(q.v.y);
            }
            lw[((s * KK + (slots ? slots[tap] : tap)) * g.nk + kc) * (4 * QUAD) + (ln >> 4) * QUAD + (ln & 15)] = q;
        }
    }
    const bool wbad = wseen.bad();
    int turn = 0;
    __syncthreads();

    for (int tile = part; tile < ntiles; tile += nparts) {
        int n0, a0, b0;
        tile_at(tile, n0, a0, b0);
        const int h0 = IS * a0 - g.ip + g.lo, w0 = IS * b0 - g.ip + g.lo;
        if (tile != part) __syncthreads();                   // the previous tile has been read
        bool bad = false;
        if constexpr (FAST) {
            Finite<T> seen;
#pragma unroll 1
            for (int it0 = 0;;) {
                stager.commit(sg, lx, g.Wi, w0, it0, g.packed != 0, seen);
                it0 += BT;
                if (it0 >= sg.iters) break;
                load_tile(tile, it0);
            }
            bad = seen.bad();
        } else
            bad = stage_pixels<T, NHWC>(in, lx, g.N, g.CI, g.Hi, g.Wi, n0, g.TN, h0, w0, g.LH, g.LW, ca, g.CL, g.pitch, g.packed != 0);
        for (int t = threadIdx.x; t < nent; t += 256) {
            const int q = t < npos ? t : 0, r = fdiv(q, g.rTB), im = fdiv(r, g.rTA), da = r - im * g.TA, db = q - r * g.TB;
            tabx[t] = ((im * g.LH + IS * da - g.lo) * g.LW + IS * db - g.lo) * g.pitch;
            const bool there = t < npos && a0 + da < g.a0 + g.na && b0 + db < g.b0 + g.nb && n0 + im < g.N;
            const int row = OS * (a0 + da) - g.op, col = OS * (b0 + db) - g.op + (E == 2 ? g.shift : 0);
            const int o = NHWC ? ((im * g.Ho + row) * g.Wo + col) * g.CO : im * (int)imout + row * g.Wo + col;
            if (OS == 1) tabo[t] = there && (unsigned)row < (unsigned)g.Ho && (unsigned)col < (unsigned)g.Wo ? o : -1;
            else { tabo[t] = o; tabr[t] = there ? row : 1 << 29; tabr[nent + t] = col; }
        }
        // One barrier behind the staging of every tile, whatever the filter and the tile hold: both paths below read pixels that other
        // wavefronts staged.  (wbad: what this lane laid out of the filter, so it counts for every tile of the block.)
        if (wbad || bad) flag[turn] = 1;
        __syncthreads();
        const bool alone = __builtin_amdgcn_readfirstlane(flag[turn]) != 0;
        turn ^= 1;
        if (threadIdx.x == 0) flag[turn] = 0;                // read by all before the last barrier, set again behind the next one
        if (FAST && tile + nparts < ntiles) load_tile(tile + nparts, 0);       // on its way while this one is computed
        if (__builtin_expect(alone, 0)) {
            own_group_only<T, NHWC, QUAD>(g, lw, slots, lx, out, n0, a0, b0, ob, ca);
            continue;
        }

        T *const on = out + (size_t)n0 * imout;
        for (int item = wv; item < g.NS * ngrp; item += 4) {
            const int s = g.NS == 1 ? 0 : item % g.NS, pg = g.NS == 1 ? item : item / g.NS;
            if (ob + s * 16 >= g.CO) continue;
            const int cl = cin_first(ob + s * 16, g) - ca + lk * 4;
            int base[P];
#pragma unroll
            for (int p = 0; p < P; ++p) base[p] = tabx[(pg * P + p) * 16 + li] + cl;
            // where the outputs of the lane's positions go
            [[maybe_unused]] int out0[P], row0[P], col0[P];
            if constexpr (OUTER) {
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int t = (pg * P + p) * 16 + li;
                    out0[p] = tabo[t];
                    if (OS > 1) { row0[p] = tabr[t]; col0[p] = tabr[nent + t]; }
                }
            }
            const Frag<T> *pw = lw + s * KK * g.nk * (4 * QUAD) + lk * QUAD + li;
            for (int f = 0; f < OS; ++f)
                for (int e0 = 0; e0 < OS; e0 += E) {
                    v4f acc[E][P];
#pragma unroll
                    for (int e = 0; e < E; ++e)
#pragma unroll
                        for (int p = 0; p < P; ++p) acc[e][p] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        // the class's fragments in order: chunks, columns, rows; two to an instruction
                        const int nl = (K - e0 - e + OS - 1) / OS, n = (K - f + OS - 1) / OS * nl * g.nk;
                        const int xs = BWD ? -g.pitch : g.pitch, rs = xs * (g.LW - nl);
                        int kc = 0, l = 0, x = E == 2 && e == 0 ? g.shift * g.pitch : 0, i = 0;
                        auto next = [&]() {
                            const int at = x + kc * 16;
                            if (++kc == g.nk) { kc = 0; x += xs; if (++l == nl) { l = 0; x += rs; } }
                            return at;
                        };
                        // (U pairs at a time: their reads are under way together)
                        constexpr int U = E * P * (int)sizeof(T) <= 8 ? 2 : 1;
                        auto pairs_of = [&](auto count) {
                            constexpr int U = decltype(count)::value;
                            Frag<T> a0[U], a1[U], b0[U][P], b1[U][P];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                a0[u] = pw[u * 2 * (4 * QUAD)]; a1[u] = pw[(u * 2 + 1) * (4 * QUAD)];
                                const int x0 = next(), x1 = next();
#pragma unroll
                                for (int p = 0; p < P; ++p) {
                                    b0[u][p] = *reinterpret_cast<const Frag<T> *>(lx + base[p] + x0);
                                    b1[u][p] = *reinterpret_cast<const Frag<T> *>(lx + base[p] + x1);
                                }
                            }
#pragma unroll
                            for (int u = 0; u < U; ++u)
#pragma unroll
                                for (int p = 0; p < P; ++p)
                                    acc[e][p] = OUTER ? mma32(a0[u], a1[u], b0[u][p], b1[u][p], acc[e][p]) : mma32(b0[u][p], b1[u][p], a0[u], a1[u], acc[e][p]);
                            i += 2 * U; pw += 2 * (4 * QUAD) * U;
                        };
                        if constexpr (U > 1) {
#pragma unroll 1
                            while (i + 2 * U <= n) pairs_of(std::integral_constant<int, U>());
                        }
#pragma unroll 1
                        while (i + 1 < n) pairs_of(std::integral_constant<int, 1>());
                        if (i < n) {
                            const Frag<T> a0 = *pw;
                            Frag<T> b0[P];
#pragma unroll
                            for (int p = 0; p < P; ++p) b0[p] = *reinterpret_cast<const Frag<T> *>(lx + base[p] + x + kc * 16);
#pragma unroll
                            for (int p = 0; p < P; ++p) acc[e][p] = OUTER ? mma16(a0, b0[p], acc[e][p]) : mma16(b0[p], a0, acc[e][p]);
                            pw += CHUNK;
                        }
                    }
                    // the outputs at a position's column and (E = 2) the next one
                    auto lower = [&](int p, int r) { return E == 2 && g.shift ? acc[E - 1][p][r] : acc[0][p][r]; };
                    [[maybe_unused]] auto upper = [&](int p, int r) { return E == 2 && g.shift ? acc[0][p][r] : acc[E - 1][p][r]; };
                    const int o = ob + s * 16 + (OUTER ? lk * 4 : li);
                    if (o >= g.CO) continue;
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        if constexpr (OUTER) {
                            int at = out0[p];
                            bool ok = at >= 0;
                            if (OS > 1) {
                                ok = (unsigned)(row0[p] + f) < (unsigned)g.Ho && (unsigned)(col0[p] + e0) < (unsigned)g.Wo;
                                at += (f * g.Wo + e0) * (NHWC ? g.CO : 1);
                            }
                            if (!ok) continue;
                            if constexpr (!NHWC) {
                                T *po = on + (size_t)((unsigned)o * (unsigned)(g.Ho * g.Wo)) + at;
#pragma unroll
                                for (int k = 0; k < 4; ++k) if (o + k < g.CO) stf(po + (unsigned)(k * g.Ho * g.Wo), acc[0][p][k]);
                                continue;
                            }
                            T *po = on + (unsigned)(at + o);
                            const float r[4] = {acc[0][p][0], acc[0][p][1], acc[0][p][2], acc[0][p][3]};
                            if (FAST == 1 || g.CO % 4 == 0) Vec<T, 4>::store(po, r);
                            else if (o + 3 < g.CO) store_run<T, 4>(po, acc[0][p]);
                            else {
#pragma unroll
                                for (int k = 0; k < 4; ++k) if (o + k < g.CO) stf(po + k, r[k]);
                            }
                        } else {
                            const int t = (pg * P + p) * 16 + lk * 4;
                            const int4 at = *reinterpret_cast<const int4 *>(tabo + t);
                            T *po = on + (size_t)((unsigned)o * (unsigned)(g.Ho * g.Wo)) + (f * g.Wo + e0);
                            const int ats[4] = {at.x, at.y, at.z, at.w};
                            if (OS == 1) {
                                if (at.x >= 0 && at.w == at.x + 3) store_run<T, 4>(po + at.x, acc[0][p]);
                                else {
#pragma unroll
                                    for (int r = 0; r < 4; ++r) if (ats[r] >= 0) stf(po + ats[r], acc[0][p][r]);
                                }
                                continue;
                            }
                            const int4 row = *reinterpret_cast<const int4 *>(tabr + t), col = *reinterpret_cast<const int4 *>(tabr + nent + t);
                            const int rows[4] = {row.x, row.y, row.z, row.w}, cols[4] = {col.x, col.y, col.z, col.w};
                            if constexpr (E == 2) {
                                if (col.x >= 0 && col.w == col.x + 6 && row.w == row.x && col.w + 1 < g.Wo && (unsigned)(row.x + f) < (unsigned)g.Ho) {
                                    typedef float v8f __attribute__((ext_vector_type(8)));
                                    v8f v;
#pragma unroll
                                    for (int r = 0; r < 4; ++r) { v[2 * r] = lower(p, r); v[2 * r + 1] = upper(p, r); }
                                    store_run<T, 8>(po + at.x, v);
                                    continue;
                                }
                            }
#pragma unroll
                            for (int r = 0; r < 4; ++r)
#pragma unroll
                                for (int e = 0; e < E; ++e)
                                    if ((unsigned)(rows[r] + f) < (unsigned)g.Ho && (unsigned)(cols[r] + e0 + e) < (unsigned)g.Wo)
                                        stf(po + ats[r] + e, e == 0 ? lower(p, r) : upper(p, r));
                        }
                    }
                }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Filter gradient, stage 1.  A wavefront owns one pair of 16 output channels and 16 input channels (a "pair") and every WS-th step of
// the tile's positions; a block holds NPAIR pairs and 4 / NPAIR = WS position splits, whose sums it adds up in LDS: one partial a block.
// A step is 32 positions in bf16, the lanes' operands read from [pixel][channel] with the transposing LDS reads (two instructions
// instead of eight 2-byte reads and their packing for every tap), and 16 positions in fp32.
// ---------------------------------------------------------------------------------------------
template <typename T> constexpr int filter_step() { return sizeof(T) == 2 ? 32 : 16; }

typedef __attribute__((address_space(3))) v4s lds_v4s;
// Channel lane%16 of the block's four pixels: in every 16 lanes, lane l hands the address of channels l%4*4 .. +3 of pixel l/4.
__device__ __forceinline__ v4s read_transposed(const bf16_t *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)p);
}

template <typename T, bool NHWC, int FAST, int K>
__global__ __launch_bounds__(256, K > 3 ? 2 : sizeof(T) == 4 ? 3 : 4) void k_gconv_gemm_filter(GemmGeom g, StageGeom sx, StageGeom sy, const T *__restrict__ x,
                                                                            const T *__restrict__ dy, float *__restrict__ ws, int npair, int nparts,
                                                                            int J, unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    constexpr int VE = 16 / (int)sizeof(T), KK = K * K, STEP = filter_step<T>();
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int chb = (int)(lb % (unsigned)g.nchb), part = (int)(lb / (unsigned)g.nchb);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int WS = 4 / npair, mine = wv % npair, pair = chb * npair + mine, split = wv / npair;
    const int s = pair / g.nk, kc = pair - s * g.nk;                       // 16-channel output block, input chunk
    const int s0 = chb * npair / g.nk;
    const int cxa = (cin_first(s0 * 16, g) + (chb * npair - s0 * g.nk) * 16) & ~(VE - 1), cya = s0 * 16;
    const int cx = cin_first(s * 16, g) + kc * 16 - cxa, cy = s * 16 - cya;
    const int npos = g.TN * g.TA * g.TB, steps = (npos + STEP - 1) / STEP, pitchy = sy.pitch;
    int *tab = reinterpret_cast<int *>(smem);                              // position -> LDS element of its input pixel
    T *lx = reinterpret_cast<T *>(tab + steps * STEP);
    T *ly = lx + (size_t)g.TN * g.LH * g.LW * g.pitch;

    const int ntiles = g.tn * g.ta * g.tb;
    const unsigned imx = (unsigned)(g.CI * g.Hi * g.Wi), imy = (unsigned)(g.CO * g.Ho * g.Wo);
    auto tile_at = [&](int tile, int &n0, int &a0, int &b0) {
        const int row = FAST ? uniform_div(tile, g.rtb) : tile / g.tb, tn = FAST ? uniform_div(row, g.rta) : row / g.ta;
        n0 = tn * g.TN; a0 = (row - tn * g.ta) * g.TA; b0 = (tile - row * g.tb) * g.TB;
    };
    constexpr int BT = NHWC ? 4 : sizeof(T) == 2 && K <= 3 ? 2 : 1;        // items of a lane in flight
    [[maybe_unused]] Stager<T, NHWC, FAST, BT, false> stx(sx), sty(sy);
    auto load_x = [&](int n0, int a0, int b0, int it0) {
        const int nimg = min(g.TN, g.N - n0), h0 = g.IS * a0 - g.ip, w0 = g.IS * b0 - g.ip;
        stx.load(sx, x, (unsigned)n0 * imx, (unsigned)g.N * imx, nimg, g.CI, g.Hi, g.Wi, h0, w0, cxa, it0);
    };
    auto load_y = [&](int n0, int a0, int b0, int it0) {
        const int nimg = min(g.TN, g.N - n0);
        sty.load(sy, dy, (unsigned)n0 * imy, (unsigned)g.N * imy, nimg, g.CO, g.Ho, g.Wo, a0, b0, cya, it0);
    };
    if constexpr (FAST) {
        int n0, a0, b0;
        tile_at(part, n0, a0, b0);
        load_x(n0, a0, b0, 0);
        load_y(n0, a0, b0, 0);
    }
    for (int p = threadIdx.x; p < steps * STEP; p += 256) {
        const int q = min(p, npos - 1), r = fdiv(q, g.rTB), im = fdiv(r, g.rTA), da = r - im * g.TA, db = q - r * g.TB;
        tab[p] = ((im * g.LH + g.IS * da) * g.LW + g.IS * db) * g.pitch;
    }
    // beside the rows of x (NCHW) and behind the positions of dy: zeros
    if (!NHWC && FAST == 1)
        for (int i = threadIdx.x; i < g.TN * g.LH * g.LW * g.pitch / 4; i += 256) reinterpret_cast<Frag<T> *>(lx)[i].v = decltype(Frag<T>::v){};
    for (int i = threadIdx.x; i < (steps * STEP - npos) * pitchy; i += 256) ly[npos * pitchy + i] = T(0);
    // fp32: the 16 positions of a step are added up on their own before they join a sum.  A chain of n matrix instructions has a relative error of
    // about 2^-24 * sqrt(n / 6), and a 3x3 sum had up to twice the error of the kernels that these replaced (mean over random layers 1.65e-7
    // against the row walk's 1.12e-7, now 1.03e-7; 1.45e-7 against the generic kernels' 2.15e-7, now 1.02e-7), at 57x57x128 130 -> 141 us.  5x5 is
    // at 1.36e-7 against 2.38e-7 without, and has no registers for it (24 channels a group, 28x28, batch 64: 63 -> 95 us).
    constexpr bool FRESH = sizeof(T) == 4 && K <= 3;
    v4f acc[KK];
#pragma unroll
    for (int t = 0; t < KK; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    const bool live = s * 16 < g.CO;                                       // uniform: the last block may have pairs to spare

    for (int tile = part; tile < ntiles; tile += nparts) {
        int n0, a0, b0;
        tile_at(tile, n0, a0, b0);
        __syncthreads();
        if constexpr (FAST) {
            Finite<T> unused;
            const int w0 = g.IS * b0 - g.ip;
#pragma unroll 1
            for (int it0 = 0;;) {
                stx.commit(sx, lx, g.Wi, w0, it0, false, unused);
                it0 += BT;
                if (it0 >= sx.iters) break;
                load_x(n0, a0, b0, it0);
            }
#pragma unroll 1
            for (int it0 = 0;;) {
                sty.commit(sy, ly, g.Wo, b0, it0, false, unused);
                it0 += BT;
                if (it0 >= sy.iters) break;
                load_y(n0, a0, b0, it0);
            }
        } else {
            stage_pixels<T, NHWC>(x, lx, g.N, g.CI, g.Hi, g.Wi, n0, g.TN, g.IS * a0 - g.ip, g.IS * b0 - g.ip, g.LH, g.LW, cxa, g.CL, g.pitch, false);
            stage_pixels<T, NHWC>(dy, ly, g.N, g.CO, g.Ho, g.Wo, n0, g.TN, a0, b0, g.TA, g.TB, cya, pitchy / 16 * 16, pitchy, false);
        }
        __syncthreads();
        if (FAST && tile + nparts < ntiles) {                              // on its way while this one is computed
            tile_at(tile + nparts, n0, a0, b0);
            load_x(n0, a0, b0, 0);
            load_y(n0, a0, b0, 0);
        }
        if (!live) continue;
#pragma unroll 1
        for (int st = split; st < steps; st += WS) {
            if constexpr (sizeof(T) == 2) {
                const int q = st * 32 + lk * 4 + (li >> 2), c = (li & 3) * 4;
                const T *py = ly + q * pitchy + cy + c, *px0 = lx + tab[q] + cx + c, *px1 = lx + tab[q + 16] + cx + c;
                Frag<T> d0, d1;
                d0.v = __builtin_bit_cast(uint2, read_transposed(py)); d1.v = __builtin_bit_cast(uint2, read_transposed(py + 16 * pitchy));
#pragma unroll
                for (int kh = 0; kh < K; ++kh)
#pragma unroll
                    for (int kw = 0; kw < K; ++kw) {
                        const int toff = (kh * g.LW + kw) * g.pitch;
                        Frag<T> b0, b1;
                        b0.v = __builtin_bit_cast(uint2, read_transposed(px0 + toff)); b1.v = __builtin_bit_cast(uint2, read_transposed(px1 + toff));
                        acc[kh * K + kw] = mma32(b0, b1, d0, d1, acc[kh * K + kw]);
                    }
            } else {
                const int q = st * 16 + lk * 4;                            // the lane's four positions
                const int4 t4 = *reinterpret_cast<const int4 *>(tab + q);
                const T *py = ly + q * pitchy + cy + li, *px[4] = {lx + t4.x + cx + li, lx + t4.y + cx + li, lx + t4.z + cx + li, lx + t4.w + cx + li};
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
    }
    // the splits' sums through LDS, taken up by split 0 in order
    v4f *red = reinterpret_cast<v4f *>(smem) + (size_t)mine * KK * 64 + lane;
    for (int t = 1; t < WS; ++t) {
        __syncthreads();                                                   // the tile, or the split before, has been read
        if (split == t) {
#pragma unroll
            for (int k = 0; k < KK; ++k) red[k * 64] = acc[k];
        }
        __syncthreads();
        if (split == 0) {
#pragma unroll
            for (int k = 0; k < KK; ++k) acc[k] += red[k * 64];
        }
    }
    // lane: output s*16 + li against input channels kc*16 + lk*4 + r, so that 16 lanes write 16 consecutive outputs in NHWC
    // and a lane consecutive entries in NCHW; entries that pair different groups are dropped
    const int o = s * 16 + li, grp = fdiv(o, g.rCgo), c0 = cin_first(s * 16, g) + kc * 16 + lk * 4 - grp * g.Cgi;
    if (!live || split || o >= g.CO) return;
    float *dst = ws + (size_t)part * J;
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

// Output channels after which the blocks of 16 lie in their groups, and the inputs of those in the 16-byte vectors, as at the first one (a layer of 1024 channels in
// groups of 8 is planned in 0.3 us, by all its blocks in 1.5).
int span_period(const GemmGeom &g)
{
    int p = 16;
    while (p < g.CO && (p % g.Cgo || p / g.Cgo * g.Cgi % 8)) p += 16;
    return p;
}

// channel chunks of 16 that the inputs of any 16 consecutive outputs span, and the channels in LDS of `ns` such blocks
void channel_span(GemmGeom &g, int ns, int VE, int period, int *CL)
{
    int nk = 1;
    auto first = [&](int o) { return o / g.Cgo * g.Cgi & ~3; };
    for (int o = 0; o < g.CO && o < period; o += 16) {
        const int end = ((o + 15 < g.CO ? o + 15 : g.CO - 1) / g.Cgo + 1) * g.Cgi;
        if (cdivg(end - first(o), 16) > nk) nk = cdivg(end - first(o), 16);
    }
    g.nk = nk;
    int cl = 0;
    for (int o = 0; o < g.CO && o < ns * period; o += 16 * ns) {
        const int ca = first(o) & ~(VE - 1);
        for (int s = 0; s < ns && o + s * 16 < g.CO; ++s)
            if (first(o + s * 16) + nk * 16 - ca > cl) cl = first(o + s * 16) + nk * 16 - ca;
    }
    *CL = cdivg(cl, 8) * 8;
}

// two blocks on a compute unit; one where the filter leaves no room for two
constexpr size_t LDS_OF_TWO = 80 << 10, LDS_OF_ONE = 160 << 10;
// blocks of four wavefronts that the chip holds at a time where registers allow `most` on a compute unit
int resident_blocks(size_t lds, int most)
{
    const size_t n = (160u << 10) / (lds ? (lds + 1279) / 1280 * 1280 : 1280);
    return 256 * (int)(n < 1 ? 1 : n > (size_t)most ? most : n);
}

// 16-position tiles that a wavefront computes at a time (P of k_gconv_gemm), of a tile of npos positions and NS output blocks.  Four share a read of the
// filter, but only from 256 positions and output blocks on is there work for all four wavefronts of a block that way: at 128 half of them are idle.
// So, the shortest longest wavefront: cycles of its matrix instructions, of the LDS reads of all four, and of the loop.  (us, four at a time from 80
// on -> this: 30x492x19x19 in 41 groups, 7x7, fp32 NCHW input gradient 221 -> 138; 26x832x14x14 in 13 groups, fp32 NCHW forward 137 -> 87; random
// layers 0.94 of the time at the mean in fp32, 0.98 in bf16.  One or four at a time, without two, 0.96 and 1.02.)
int tiles_at_once(int NS, int npos, int dtype, int *longest = nullptr)
{
    const int tiles16 = cdivg(npos, 16), mfma = dtype == DT_F32 ? 128 : 16, read = dtype == DT_F32 ? 32 : 16, loop = 40;
    int best = 1, least = 1 << 30;
    for (int P = 1; P <= 4; P *= 2) {
        const int cycles = cdivg(NS * cdivg(tiles16, P), 4) * (P * mfma + (1 + P) * read + loop);
        if (cycles < least) { least = cycles; best = P; }
    }
    if (longest) *longest = least;
    return best;
}

// The widest tile (of positions from `from` down to `to`) that fits, as tile(positions) sets it up; up to half of it less where that lets `most`
// blocks onto a compute unit and it does not.  Returns the positions, 0 if nothing fits.  (14x14 16 channels a group 10.1 us with 256 positions,
// 13.0 with 128; 28x28 32 channels a group, bf16 NHWC batch 64: 55 us with 256 positions and three blocks, 47 with 128 and four.)
// Of such tiles the one whose `launched` blocks go through the chip in the shortest rounds, each its positions and 32 of fixed work: 51x34x106 in 53 groups,
// fp32 NCHW batch 45, 204 positions (40 us, 49 with 102), 61x59x84 in 42, batch 27, 122 (44 us, 56 with 183).  `positions`: the tile's, or what its time is that of.
template <typename F, typename B, typename P>
int widest_tile(const GemmGeom &g, F tile, B launched, P positions, int from, int to, int most, size_t limit, const size_t *lds)
{
    for (int want = from; want >= to; want /= 2) {
        tile(want);
        if (*lds > limit) continue;
        if (want / 2 >= 64 && resident_blocks(*lds, most) < 256 * most) {
            int best = 0;
            long long least = 0;
            for (int less = want - want / 8; less >= want / 2; less -= want / 8) {
                tile(less);
                const long long time = (launched() + 256 * most - 1) / (256 * most) * (positions() + 32);
                if (resident_blocks(*lds, most) == 256 * most && (!best || time <= least)) { best = less; least = time; }
            }
            tile(best ? best : want);
            if (best) return best;
        }
        return want;
    }
    return 0;
}

// positions of a tile: whole rows where they fit, several images of a small map; a row of a multiple of `quad` positions, so that
// four of them have consecutive outputs
void pick_positions(GemmGeom &g, int want, int maxb, int quad = 1)
{
    g.TB = g.nb < maxb ? g.nb : cdivg(g.nb, cdivg(g.nb, maxb));
    g.TB = cdivg(g.TB, quad) * quad;
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

// copying a tile of TN images of LH x LW pixels and CL channels (NCHW: rows of W columns) with 256 lanes
StageGeom stage_geom(int layout, int VE, int TN, int LH, int LW, int CL, int pitch, int W, bool split)
{
    StageGeom s = {};
    const bool nhwc = layout == LAYOUT_NHWC;
    s.LH = LH; s.LW = LW; s.pitch = pitch;
    s.imrows = TN * LH;
    s.rows = nhwc ? s.imrows : s.imrows * (CL / 4);
    s.nv = nhwc ? CL / VE : 1;
    const int width = nhwc ? LW : cdivg(split ? LW + 3 : W, 4);             // columns, or runs of four
    s.width = width;
    const int most = 256 / s.nv > 0 ? 256 / s.nv : 1, passes = cdivg(width, most);
    s.cols = cdivg(width, passes);
    s.per = s.cols * s.nv;
    s.RPI = s.per <= 256 ? 256 / s.per : 1;                                 // (more items a pixel than lanes: not FAST)
    s.nrit = cdivg(s.rows, s.RPI);
    s.iters = s.nrit * passes;
    s.rper = 1.0f / (float)s.per; s.rnv = 1.0f / (float)s.nv; s.rLH = 1.0f / (float)LH; s.rimrows = 1.0f / (float)s.imrows;
    return s;
}

bool gemm_plan_as(const GGeom &q, int layout, int dtype, int pass, bool pairs, GemmPlan *pl)
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
        if (pairs) { g.pairs = 1; g.shift = q.p & 1; g.nb = (q.W + 1) / 2; }
    }
    const int reach = pass == 1 ? 1 - g.lo : q.K;                           // input rows of one position
    const int blocks16 = cdivg(g.CO, 16), period = span_period(g);
    if (pass < 2) {
        // A launch of few blocks is one short round of them beside idle compute units, each as long as its tile: smaller tiles, down to a
        // 16-position tile for each wavefront, then one output block a block.  (us: 4x64x9x9 in 2 groups, stride 2, fp32 NCHW input gradient 30 -> 13,
        // 8x480x21x11 in 15, stride 3, 37 -> 14.6; random layers 0.94 of the time at the mean forward, 0.86 (fp32) and 0.89 (bf16) in the input
        // gradient, 0.3 % longer by more than 8 %.  Below 128 or 256 blocks 0.5 % longer.)
        constexpr int FEW = 192;
        // output blocks of 16 per block: two where they read the same input channels (us, one -> two: 7x7 32 channels a group, batch 64, 1024
        // channels, bf16 NHWC 16.1 -> 14.1, fp32 NCHW 39.3 -> 38.7; 28x28x512 batch 64 bf16 NHWC 55.5 -> 45.3), otherwise one (two against one: 14x14x512
        // 16 channels a group, batch 32, bf16 NHWC 10.6 and 10.2, fp32 NCHW 26.0 and 22.9; 56x56x240 24 channels a group, bf16 NHWC batch 64 187 and
        // 174; 57x57x128 4 channels a group, fp32 NCHW batch 64 124 and 109)
        int ns = g.Cgo % 32 == 0 ? 2 : 1;
        if (ns > blocks16) ns = blocks16;
        for (;; ns = (ns + 1) / 2) {
            g.NS = ns;
            channel_span(g, ns, VE, period, &g.CL);
            g.packed = !(g.Cgo % 16 == 0 && g.Cgi % 16 == 0);
            // (16-byte or, in NCHW, four-channel LDS stores)
            g.pitch = g.CL + (layout == LAYOUT_NHWC ? VE : 4);
            auto tile = [&](int want) {
                pick_positions(g, want, layout == LAYOUT_NHWC ? 32 : 64, pairs ? 4 : 1);
                g.LH = g.IS * (g.TA - 1) + reach; g.LW = g.IS * (g.TB - 1) + reach + g.shift;
                // (positions in the tables up to a multiple of 64)
                pl->lds = (size_t)ns * q.K * q.K * g.nk * 256 * esz + (size_t)cdivg(g.TN * g.TA * g.TB, 64) * 64 * (g.OS > 1 ? 16 : 8) + (g.OS > 1 ? 256 : 0) + 16 +
                          ((size_t)g.TN * g.LH * g.LW * g.pitch * esz + 15) / 16 * 16;
            };
            auto blocks = [&]() { return (long long)g.tn * g.ta * g.tb * cdivg(blocks16, ns); };
            // (two output blocks: a wavefront's work comes in steps, and 144 to 224 positions take as long as 256.  By the positions alone 28x28x512 in 16
            // groups, bf16 NHWC batch 64, had 196 and took 51 us, with 112 41.5; 44x44x32 in one, batch 356, 50 -> 42, input gradient 58 -> 47)
            auto positions = [&]() {
                const int npos = g.TN * g.TA * g.TB;
                int steps, full;
                if (ns == 1) return npos;
                tiles_at_once(ns, npos, dtype, &steps); tiles_at_once(ns, 256, dtype, &full);
                return 256 * steps / full;
            };
            int want = widest_tile(g, tile, blocks, positions, 256, 16, 4, LDS_OF_TWO, &pl->lds);
            if (!want && ns == 1) want = widest_tile(g, tile, blocks, positions, 256, 16, 4, LDS_OF_ONE, &pl->lds);
            if (!want && ns == 1) return false;
            if (!want) continue;
            auto few = [&]() { return blocks() < FEW; };
            for (; want > 64 && few(); tile(want)) want /= 2;
            if (ns == 1 || !few()) break;
        }
        g.nchb = cdivg(blocks16, g.NS);
        const long long tiles = (long long)g.tn * g.ta * g.tb;
        // the filter is laid out once per block and the next tile is on its way while one is computed: as many blocks as are resident,
        // the tiles of a channel block shared among them
        long long parts = resident_blocks(pl->lds, 4) / g.nchb;
        if (parts < 1) parts = 1;
        if (parts > tiles) parts = tiles;
        parts = (tiles + (tiles + parts - 1) / parts - 1) / ((tiles + parts - 1) / parts);
        pl->nparts = (int)parts;
        pl->nblocks = (unsigned)(parts * g.nchb);
    } else {
        if (q.K > 5) return false;
        int dummy;
        channel_span(g, 1, VE, period, &dummy);
        const int pairs = blocks16 * g.nk;
        // NHWC: two pairs a block read whole 64-byte runs of channels (14x14 16 channels a group, bf16 batch 32: 14.5 us, with one 15.5); NCHW
        // gains nothing by it and a pair alone leaves smaller tiles (56x56 8 channels a group at stride 2, bf16 batch 16: 23.6 against 28)
        const int blocks = q.K > 3 ? 2 : 4;                                 // on a compute unit, by registers
        int npair = q.K == 1 ? 4 : layout == LAYOUT_NHWC || g.nk > 1 ? 2 : 1;
        while (npair > pairs) npair /= 2;
        bool fits = false;
        for (; npair >= 1 && !fits; npair /= 2) {
            pl->npair = npair;
            g.nchb = cdivg(pairs, npair);
            // channels in LDS of any block: its pairs run over (output block, chunk)
            int clx = 0, cly = 0;
            auto first = [&](int o) { return o / g.Cgo * g.Cgi & ~3; };
            const long long pairs_of_period = (long long)(period / 16) * g.nk;
            for (int b = 0; b < g.nchb && (b == 0 || (long long)b * npair % pairs_of_period != 0); ++b) {
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
            g.pitch = g.CL + (layout == LAYOUT_NHWC ? VE : 4); pl->pitchy = cly + (layout == LAYOUT_NHWC ? VE : 4);
            // tiles of fewer than 64 positions only if nothing else fits
            auto tile = [&](int want) {
                pick_positions(g, want, layout == LAYOUT_NHWC ? 32 : 64);
                g.LH = g.IS * (g.TA - 1) + q.K; g.LW = g.IS * (g.TB - 1) + q.K;
                const int npos = g.TN * g.TA * g.TB, step = esz == 2 ? 32 : 16, padded = (npos + step - 1) / step * step;
                pl->lds = (size_t)padded * 4 + ((size_t)g.TN * g.LH * g.LW * g.pitch + (size_t)padded * pl->pitchy) * esz;
                // the sums of a split, where there are several
                const size_t sums = npair < 4 ? (size_t)npair * q.K * q.K * 1024 : 0;
                if (pl->lds < sums) pl->lds = sums;
            };
            // Few blocks: smaller tiles, then fewer pairs a block, as above, but a partial is added up again, so not beyond 128.  (us, stage 2 in
            // it: 1x48x46x46 in 8 groups, 5x5, fp32 NHWC 31 -> 15, 10x192x56x5 in 12, 3x3 at stride 3, bf16 NCHW 29 -> 12; random layers 0.945 of
            // the time at the mean, 0.4 % longer by more than 8 %.  192 blocks: 0.95 and 2.2 %.)
            constexpr int FEW = 128;
            auto launched = [&]() { return (long long)g.tn * g.ta * g.tb * g.nchb; };
            auto positions = [&]() { return g.TN * g.TA * g.TB; };
            int want = widest_tile(g, tile, launched, positions, 256, npair > 1 ? 64 : 16, blocks, LDS_OF_TWO, &pl->lds);
            auto few = [&]() { return launched() < FEW; };
            for (; want > 32 && few(); tile(want)) want /= 2;
            fits = want > 0 && (npair == 1 || !few());
            if (fits) break;
        }
        if (!fits) return false;
        const long long tiles = (long long)g.tn * g.ta * g.tb, J = (long long)q.O * q.Cg * q.K * q.K;
        long long parts = resident_blocks(pl->lds, blocks) / g.nchb;
        if (parts > tiles) parts = tiles;
        const long long most = (16ll << 20) / (J * 4);
        if (parts > most) parts = most;
        if (parts < 1) parts = 1;
        if (J * 4 > (64ll << 20)) return false;
        parts = (tiles + (tiles + parts - 1) / parts - 1) / ((tiles + parts - 1) / parts);
        pl->nparts = (int)parts;
        pl->nblocks = (unsigned)(parts * g.nchb);
    }
    g.rCgi = 1.0f / (float)g.Cgi; g.rCgo = 1.0f / (float)g.Cgo; g.rKK = 1.0f / (float)(q.K * q.K); g.rnk = 1.0f / (float)g.nk;
    g.rTA = 1.0f / (float)g.TA; g.rTB = 1.0f / (float)g.TB;
    g.rta = 1.0f / (float)g.ta; g.rtb = 1.0f / (float)g.tb;
    // whole vectors of channels, or whole rows, or neither; the images of a tile below 2 GiB and 2^24 pixels, for the staging's offsets and products
    const long long inpix = (long long)g.TN * g.Hi * g.Wi, outpix = (long long)g.TN * g.Ho * g.Wo;
    pl->fast = (layout == LAYOUT_NHWC ? q.C % VE == 0 && q.O % VE == 0 : g.tb == 1) ? 1 : 2;
    const bool small = inpix < 1 << 24 && outpix < 1 << 24 &&
               inpix * g.CI * esz < 1ll << 31 && outpix * g.CO * esz < 1ll << 31 && (long long)g.tn * g.ta * g.tb < 1 << 21;
    pl->sg = stage_geom(layout, VE, g.TN, g.LH, g.LW, g.CL, g.pitch, g.Wi, g.tb > 1);
    if (pass == 2) pl->sy = stage_geom(layout, VE, g.TN, g.TA, g.TB, pl->CLy, pl->pitchy, g.Wo, g.tb > 1);
    // as many lanes as a pixel has vectors; a vector's elements for the unaligned loads
    const bool stageable = small && pl->sg.per <= 256 && (pass < 2 || pl->sy.per <= 256) && (long long)g.N * g.CI * g.Hi * g.Wi >= 8 &&
                           (long long)g.N * g.CO * g.Ho * g.Wo >= 8;
    if (!stageable) pl->fast = 0;
    // (filter gradient in fp32: four loads of a lane, each of 64 lanes in a row, are the shorter way; us, 376x127x127 in 188 groups, NCHW, 40 against 46,
    // 94x87x6 in three groups, 5x5, NHWC batch 7, 20 against 24)
    if (pass == 2 && dtype == DT_F32 && pl->fast == 2) pl->fast = 0;
    pl->quad = 16;
    if (pass < 2 && layout == LAYOUT_NCHW && pl->fast) {
        const size_t padded = pl->lds + (size_t)g.NS * q.K * q.K * g.nk * 16 * esz;
        if (padded <= LDS_OF_ONE && resident_blocks(padded, 4) == resident_blocks(pl->lds, 4)) { pl->quad = 17; pl->lds = padded; }
    }
    pl->g = g;
    return true;
}

}  // namespace

bool gconv_gemm_plan(const GGeom &q, int layout, int dtype, int pass, GemmPlan *pl)
{
    if (pass == 2 && q.K != 1 && q.K != 3 && q.K != 5) return false;
    if (pass == 1 && layout == LAYOUT_NCHW && q.s == 2 && gemm_plan_as(q, layout, dtype, pass, true, pl) && pl->fast) return true;
    return gemm_plan_as(q, layout, dtype, pass, false, pl);
}

// The launch, laying out the filter (768 fragments a time), then for every tile of the block a fixed latency, the staging (4 KiB a time) and the products of
// its longest wavefront, each with a part that grows with the blocks on a compute unit, and the classes of output pixels.  Fitted to 64 000
// random layers: four of five between 0.85 and 1.12 (NCHW input gradient 0.81 and 1.15) times the measured time.
double gconv_gemm_us(const GemmPlan &pl, int layout, int dtype)
{
    static const float fit[2][2][2][2][8] = {                               // [pass][layout][dtype][ragged channels or tiles]
        {{{{4.57f, 0.474f, 0, 0.142f, 0.0103f, 0.169f, 0.0784f, 0}, {5.31f, 0.383f, 0, 0.172f, 0.00555f, 0.151f, 0.0768f, 0}},
          {{2.62f, 0.518f, 2.18f, 0.193f, 0.0101f, 0.23f, 0.00959f, 0}, {2.34f, 0.38f, 3.27f, 0.0859f, 0.0117f, 0.253f, 0.0058f, 0}}},
         {{{3.73f, 0.558f, 0, 0.0646f, 0.0402f, 0.232f, 0.0602f, 0}, {3.88f, 0.297f, 0, 0.264f, 0.0102f, 0.167f, 0.0801f, 0}},
          {{3.14f, 0.65f, 0.848f, 0.0247f, 0.0132f, 0.268f, 0.00746f, 0}, {2.72f, 0.454f, 1.44f, 0.217f, 0.016f, 0.234f, 0.00353f, 0}}}},
        {{{{4.58f, 0.777f, 0, 0.0718f, 0.021f, 0.269f, 0.07f, 0.398f}, {4.82f, 0.857f, 0, 0.0165f, 0.0263f, 0.305f, 0.0505f, 0.914f}},
          {{3.72f, 0.817f, 0.955f, 0.0757f, 0.018f, 0.434f, 0.00379f, 0.437f}, {3.31f, 0.46f, 1.73f, 0.109f, 0.0141f, 0.379f, 0.00206f, 0.896f}}},
         {{{3.86f, 0.703f, 0, 0, 0.0416f, 0.349f, 0.0573f, 0.284f}, {4.72f, 0.0744f, 0, 0, 0.0645f, 0.484f, 0.0413f, 0.368f}},
          {{4.01f, 0.823f, 0.132f, 0, 0.0101f, 0.393f, 0.00718f, 0.285f}, {4.16f, 0.417f, 0.9f, 0.21f, 0.0213f, 0.354f, 0, 0.352f}}}}};
    const GemmGeom &g = pl.g;
    const float *c = fit[g.bwd][layout == LAYOUT_NHWC][dtype != DT_F32][pl.fast != 1];
    const int tiles = cdivg(g.tn * g.ta * g.tb, pl.nparts), tiles16 = cdivg(g.TN * g.TA * g.TB, 16), P = tiles_at_once(g.NS, g.TN * g.TA * g.TB, dtype);
    const double resident = resident_blocks(pl.lds, 4), cu = pl.nblocks / 256.0;
    const double rounds = pl.nblocks > resident ? pl.nblocks / resident : 1.0, beside = cu < 1 ? 1 : cu > resident / 256 ? resident / 256 : cu;
    const double staging = (double)g.TN * g.LH * g.LW * g.CL * (dtype == DT_F32 ? 4 : 2) / 4096;
    const double products = (double)cdivg(g.NS * cdivg(tiles16, P), 4) * P * g.K * g.K * g.nk;
    return c[0] + rounds * (c[1] * (g.NS * g.K * g.K * g.nk * 64) / 768 +
                            tiles * (c[2] + c[3] * staging + c[4] * products + beside * (c[5] * staging + c[6] * products) + c[7] * g.OS * g.OS));
}

void gconv_gemm_filter_tiles(const GemmPlan &pl, FilterGradSrc *f)
{
    f->TN = pl.g.TN; f->TA = pl.g.TA; f->TB = pl.g.TB;
    f->tn = pl.g.tn; f->ta = pl.g.ta; f->tb = pl.g.tb;
    f->per = 0; f->nparts = pl.nparts;
}

template <typename T, bool NHWC>
static hipError_t gemm_go(const GemmPlan &pl, const void *in, const void *w, void *out, hipStream_t st)
{
    constexpr bool NCHW = !NHWC;
    auto pick = [&](auto p, auto fast, auto quad) {
        constexpr int P = decltype(p)::value, FAST = decltype(fast)::value, QUAD = decltype(quad)::value;
        return !pl.g.bwd ? k_gconv_gemm<T, NHWC, false, FAST, P, 1, false, QUAD>
               : pl.g.pairs ? k_gconv_gemm<T, NHWC, true, FAST, P, (NCHW && FAST ? 2 : 1), false, QUAD>
               : pl.g.OS > 1 ? k_gconv_gemm<T, NHWC, true, FAST, P, 1, NCHW, QUAD> : k_gconv_gemm<T, NHWC, true, FAST, P, 1, false, QUAD>;
    };
    const int P = tiles_at_once(pl.g.NS, pl.g.TN * pl.g.TA * pl.g.TB, sizeof(T) == 4 ? DT_F32 : DT_BF16);
    auto of = [&](auto fast, auto quad) {
        return P == 4 ? pick(std::integral_constant<int, 4>(), fast, quad)
               : P == 2 ? pick(std::integral_constant<int, 2>(), fast, quad) : pick(std::integral_constant<int, 1>(), fast, quad);
    };
    auto padded = [&](auto fast) {
        if constexpr (NCHW) {
            if (pl.quad == 17) return of(fast, std::integral_constant<int, 17>());
        }
        return of(fast, std::integral_constant<int, 16>());
    };
    auto kernel = pl.fast == 1 ? padded(std::integral_constant<int, 1>()) : pl.fast ? padded(std::integral_constant<int, 2>())
                  : of(std::integral_constant<int, 0>(), std::integral_constant<int, 16>());
    hipLaunchKernelGGL(kernel, dim3(pl.nblocks), dim3(256), pl.lds, st, pl.g, pl.sg, (const T *)in, (const T *)w, (T *)out,
                       pl.nparts, pl.nblocks);
    return hipGetLastError();
}
hipError_t gconv_gemm(const GemmPlan &pl, int layout, int dtype, const void *in, const void *w, void *out, hipStream_t st)
{
    if (dtype == DT_F32) return layout == LAYOUT_NHWC ? gemm_go<float, true>(pl, in, w, out, st) : gemm_go<float, false>(pl, in, w, out, st);
    return layout == LAYOUT_NHWC ? gemm_go<bf16_t, true>(pl, in, w, out, st) : gemm_go<bf16_t, false>(pl, in, w, out, st);
}

template <typename T, bool NHWC>
static hipError_t gemm_filter_go(const GemmPlan &pl, const void *x, const void *dy, float *ws, hipStream_t st)
{
    const int J = pl.g.FO * pl.g.FCg * pl.g.K * pl.g.K;
    auto of = [&](auto fast) {
        constexpr int FAST = decltype(fast)::value;
        return pl.g.K == 1 ? k_gconv_gemm_filter<T, NHWC, FAST, 1> : pl.g.K == 3 ? k_gconv_gemm_filter<T, NHWC, FAST, 3> : k_gconv_gemm_filter<T, NHWC, FAST, 5>;
    };
    auto kernel = pl.fast == 1 ? of(std::integral_constant<int, 1>()) : of(std::integral_constant<int, 0>());
    if constexpr (sizeof(T) == 2) {                                        // (fp32: not planned, see there)
        if (pl.fast == 2) kernel = of(std::integral_constant<int, 2>());
    }
    hipLaunchKernelGGL(kernel, dim3(pl.nblocks), dim3(256), pl.lds, st, pl.g, pl.sg, pl.sy, (const T *)x, (const T *)dy, ws, pl.npair,
                       pl.nparts, J, pl.nblocks);
    return hipGetLastError();
}
hipError_t gconv_gemm_bwd_filter(const GemmPlan &pl, int layout, int dtype, const void *x, const void *dy, float *ws, hipStream_t st)
{
    if (dtype == DT_F32) return layout == LAYOUT_NHWC ? gemm_filter_go<float, true>(pl, x, dy, ws, st) : gemm_filter_go<float, false>(pl, x, dy, ws, st);
    return layout == LAYOUT_NHWC ? gemm_filter_go<bf16_t, true>(pl, x, dy, ws, st) : gemm_filter_go<bf16_t, false>(pl, x, dy, ws, st);
}

}  // namespace dwc

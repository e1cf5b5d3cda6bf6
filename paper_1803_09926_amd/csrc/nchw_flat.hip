// NCHW kernels for rows of any width: 3x3, 5x5 and 7x7 filters, stride 1 and 2, any padding, any multiplier (the input
// gradient: 1 and 2).
//
// Rows of 19, 37 or 74 elements are no whole number of 16-byte vectors, but a run of rows of a plane is one flat range of
// memory, and so is a run of whole planes.  A block takes U planes and a band of TR output rows of each: the input rows go to
// LDS as flat ranges in memory order (16 bytes per lane straight into LDS, `dma_range`: no register, no wait before
// the block's barrier), a lane owns one output column (or two) of one plane and walks down the band, and every output row leaves
// straight from the registers: consecutive lanes consecutive elements, lines completed in L2 by the next row or plane.  (Gathered in
// a second LDS area and stored as 16-byte vectors they left room for half as many blocks: forward at batch 64 28x28x256 7x7 fp32
// 46 -> 34 us, 41x41x240 5x5 bf16 55 -> 44, 19x19x728 fp32 17.7 -> 13.7, 74x74x256 bf16 46.6 -> 44.8, the last two at batch 32.)
// Every lane of the block is in the same row at the same time, so what depends on the row (padding above and below, the first and last steps of the walk) is scalar; padding to the left and
// right is one select per value read.  A step reads K values of one input row (consecutive lanes consecutive words: no bank
// conflict) for K*K multiply-adds.  Every block is short; several blocks per compute unit overlap one's loads with
// another's arithmetic.
#include "bounds.hpp"
#include "point.hpp"
#include <type_traits>

namespace dwc {

namespace {

template <typename T> constexpr int ve_of() { return 16 / (int)sizeof(T); }

// Bands of planes staged in LDS.  Whole planes (`whole`) are one range; otherwise every plane's band is a segment of its own,
// `pitch` elements apart in LDS.  A range starts in LDS at the 16-byte boundary below its first element.
struct Bands {
    int plane0, nplanes;   // planes in the tile
    int HW, W;             // plane size, row width
    int r0, r1;            // rows of the band (inside the plane)
    int pitch;             // LDS elements between segments (0: whole planes, one range)
    __device__ __forceinline__ int first(int j) const { return (plane0 + j) * HW + r0 * W; }       // element index of segment j
    // LDS element of row r0, column 0 of plane j
    template <typename T> __device__ __forceinline__ int at(int j) const
    {
        return pitch ? j * pitch + (first(j) & (ve_of<T>() - 1)) : (first(0) & (ve_of<T>() - 1)) + j * HW;
    }
};

typedef __attribute__((address_space(1))) const void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

// Copies the bands to `lds` (16-byte aligned).  The caller waits (dma_wait) and synchronises before reading.
template <typename T>
__device__ __forceinline__ void dma_bands(const T *__restrict__ src, int total, const Bands &b, T *lds)
{
    constexpr int VE = ve_of<T>();
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int nseg = b.pitch ? b.nplanes : 1, len = b.pitch ? (b.r1 - b.r0) * b.W : b.nplanes * b.HW;
    const int nc = (len + VE - 1 + VE - 1) / VE / 64 + 1;          // 64-vector chunks of a segment, at most
    for (int i = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); i < nseg * nc; i += nw) {
        const int s = i / nc, ch = i - s * nc;
        const int e0 = b.first(s), a0 = e0 & ~(VE - 1), nvec = (e0 + len - a0 + VE - 1) / VE;
        const int idx = ch * 64 + lane;
        T *base = lds + s * b.pitch + ch * 64 * VE;
        if (idx < nvec) {
            const int a = a0 + idx * VE;
            if (vector_inside(a, VE, total))
                __builtin_amdgcn_global_load_lds((gptr_t)(src + a), (lptr_t)base, 16, 0, 0);
            else {                                                   // the last vector of a tensor that is no whole number of vectors
                for (int j = 0; j < VE && a <= total - 1 - j; ++j) base[lane * VE + j] = src[a + j];
            }
        }
    }
}
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One element of a lane, soff the same in every lane.  (Without the readfirstlane of BufView's own members, which keeps a loop from
// being unrolled: the row offset comes from the loop counter and is scalar as it is.)
template <typename T> __device__ __forceinline__ void store_one(const BufView &v, float f, uint32_t voff, uint32_t soff)
{
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f), v.rsrc, (int)voff, (int)soff, 0);
    else {
        T h;
        stf(&h, f);
        __builtin_amdgcn_raw_buffer_store_b16(h, v.rsrc, (int)voff, (int)soff, 0);
    }
}
template <typename T> __device__ __forceinline__ void store_two(const BufView &v, float f, float h, uint32_t voff, uint32_t soff)
{
    if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b64(u2raw_t{__float_as_uint(f), __float_as_uint(h)}, v.rsrc, (int)voff, (int)soff, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(pack2_bf16(f, h), v.rsrc, (int)voff, (int)soff, 0);
}
template <typename T> __device__ __forceinline__ T load_one(const BufView &v, uint32_t voff, uint32_t soff)
{
    if constexpr (sizeof(T) == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(v.rsrc, (int)voff, (int)soff, 0));
    else return __builtin_amdgcn_raw_buffer_load_b16(v.rsrc, (int)voff, (int)soff, 0);
}

// What a launch of these kernels is cut into.
struct FlatTile {
    int U, TR, nbands;     // planes per block, output rows per band (bwd_data_s2: row pairs), bands per plane
    int pin, pout;         // LDS elements from plane to plane (0: whole planes); of dy, if it is in LDS too (0: it is not)
    int nin;               // LDS elements of the input area
    int threads;
};

// A value read beside the row (padding) is cleared by its lane's mask: a select would let the compiler branch around the read.
__device__ __forceinline__ float masked(float f, uint32_t m) { return __uint_as_float(__float_as_uint(f) & m); }

constexpr int GUARD = 16;  // LDS elements in front of and behind the input area that an edge lane may read (and drop)

}  // namespace

// ---------------------------------------------------------------------------------------------
// out[plane][oh][ow] = sum over q < M, kh, kw of w[kh][kw] * in[plane * M / mdiv + q][oh*S - pad + kh][ow*S - pad + kw].
// Forward: M = 1, mdiv = the multiplier.  Input gradient of a stride-1 layer (flip): in = dy, filters rotated by 180
// degrees, pad = K - 1 - p, M = the multiplier.
// ---------------------------------------------------------------------------------------------
template <typename T, int K, int S, int M, bool SAME, int NC>
__global__ __launch_bounds__(512) void k_nchwf_conv(const T *__restrict__ in, const T *__restrict__ w, T *__restrict__ out,
                                                    int nplanes, int OC, int Hi, int Wi, int Ho, int Wo, int pad, int mdiv,
                                                    int total_in, int flip, FlatTile ft, unsigned nblocks, Geom g)
{
    extern __shared__ uint4 smem[];
    constexpr int NA = (K + S - 1) / S;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int band = (int)(lb % (unsigned)ft.nbands), p0 = (int)(lb / (unsigned)ft.nbands) * ft.U;
    const int np = min(ft.U, nplanes - p0);
    const int oh0 = band * ft.TR, oh1 = min(Ho, oh0 + ft.TR);
    const int ip0 = M > 1 ? p0 * M : p0 / mdiv, ip1 = M > 1 ? (p0 + np) * M : (p0 + np - 1) / mdiv + 1;
    const int r0 = min(max(oh0 * S - pad, 0), Hi), r1 = max(min((oh1 - 1) * S - pad + K, Hi), r0);
    const Bands bi = {ip0, ip1 - ip0, Hi * Wi, Wi, r0, r1, ft.pin};
    T *lin = reinterpret_cast<T *>(smem) + GUARD;
    dma_bands<T>(in, total_in, bi, lin);

    constexpr int VW = S * (NC - 1) + K;                   // values of an input row that the lane's NC columns reach
    const int ncol = (Wo + NC - 1) / NC;
    const int u = (int)threadIdx.x / ncol, ow = ((int)threadIdx.x - u * ncol) * NC;
    const bool active = u < np;
    const int pl = p0 + (active ? u : 0), oc = pl % OC;
    uint32_t ok[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i) ok[i] = (unsigned)(ow * S - pad + i) < (unsigned)Wi ? ~0u : 0u;
    const int col0 = min(max(ow * S - pad, -VW), Wi);      // a column further out has every tap dropped anyway
    float wr[M][K][K];
    int src[M];                                            // LDS element of (plane, row r0, column col0)
#pragma unroll
    for (int q = 0; q < M; ++q) {
#pragma unroll
        for (int kh = 0; kh < K; ++kh)
#pragma unroll
            for (int kw = 0; kw < K; ++kw) {
                const int tap = kh * K + kw;
                wr[q][kh][kw] = ldf(w + (oc * M + q) * K * K + (flip ? K * K - 1 - tap : tap));
            }
        src[q] = bi.at<T>((M > 1 ? pl * M + q : pl / mdiv) - ip0) + col0;
    }
    // a column that is none is stored outside the view: no lane mask in the walk
    const BufView vout(out + (size_t)p0 * Ho * Wo, (uint32_t)(np * Ho * Wo) * (uint32_t)sizeof(T));
    uint32_t voff[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) voff[n] = active && ow + n < Wo ? (uint32_t)((u * Ho + oh0) * Wo + ow + n) * (uint32_t)sizeof(T) : BufView::OUTSIDE;
    float acc[NA][NC];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int n = 0; n < NC; ++n) acc[i][n] = 0.f;
    NonFinite bad;
#pragma unroll
    for (int q = 0; q < M; ++q)
#pragma unroll
        for (int e = 0; e < K * K; ++e) bad.add(wr[q][e / K][e % K]);
    const bool redo = bad.any() && active;
    dma_wait();
    __syncthreads();

    // Step t reads the S input rows from row (oh0 + t)*S - pad on; they meet the outputs of rows oh0 + t - i, and the one with
    // i = NA - 1 is complete.  Steps [ta, tb) have all their rows in the band and check nothing.
    // At the ends of the walk only the outputs of the band are added to.
    const int base = oh0 * S - pad - r0, nrows = r1 - r0, TRb = oh1 - oh0;
    auto step = [&](int t, auto checked) {
        constexpr bool CK = decltype(checked)::value;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int row = base + t * S + j;              // everything about the row is uniform
            if (CK && (row < 0 || row >= nrows)) continue; // padding
#pragma unroll
            for (int q = 0; q < M; ++q) {
                const T *p = lin + src[q] + row * Wi;
                float v[VW];
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    const float f = ldf(p + i);
                    v[i] = SAME && NC == 1 && i == K / 2 ? f : masked(f, ok[i]);      // the centre tap is never outside
                }
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    if (j + i * S >= K || (CK && K > 3 && (unsigned)(t - i) >= (unsigned)TRb)) continue;
#pragma unroll
                    for (int kw = 0; kw < K; ++kw)
#pragma unroll
                        for (int n = 0; n < NC; ++n) acc[i][n] = fmaf(wr[q][j + i * S][kw], v[n * S + kw], acc[i][n]);
                }
            }
        }
        if (!CK || t >= NA - 1) {
            const uint32_t so = (uint32_t)((t - (NA - 1)) * Wo) * (uint32_t)sizeof(T);
#pragma unroll
            for (int n = 0; n < NC; ++n) store_one<T>(vout, acc[NA - 1][n], voff[n], so);
        }
#pragma unroll
        for (int i = NA - 1; i > 0; --i)
#pragma unroll
            for (int n = 0; n < NC; ++n) acc[i][n] = acc[i - 1][n];
#pragma unroll
        for (int n = 0; n < NC; ++n) acc[0][n] = 0.f;
    };
    const int steps = TRb + NA - 1;
    const int ta = (S - 1 - base) / S, tb = min((nrows - base) / S, K > 3 ? TRb : steps);
    int t = 0;
    for (; t < min(max(ta, NA - 1), steps); ++t) step(t, std::true_type());
#pragma unroll NA
    for (; t < tb; ++t) step(t, std::false_type());
    for (; t < steps; ++t) step(t, std::true_type());
    if (__builtin_expect(redo, 0)) {          // the lane's columns again, without the padding
        const int n = pl / OC;
#pragma unroll 1
        for (int i = 0; i < TRb * NC; ++i) {
            const int t = i / NC, c = ow + i - t * NC;
            if (c < Wo)
                stf(out + ((size_t)pl * Ho + oh0 + t) * Wo + c, flip ? point_bwd_data<T, LAYOUT_NCHW>(g, in, w, n, oc, oh0 + t, c)
                                                          : point_fwd<T, LAYOUT_NCHW>(g, in, w, n, oc, oh0 + t, c));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The same for 3x3 "same" stride 1 in bf16 on rows of an even width: a lane owns two adjacent columns, which are one aligned word in LDS as in
// the output, and reads the words beside it, half of each masked away.  A row of three taps is two packed dot products an output, nothing is
// widened: 12 dot products, two masks and three LDS reads for two columns of three rows, against 18 multiply-adds, ten other
// instructions and six reads.
// us, one column a lane -> this, batch 32 74x74x256 47.0 -> 43.4, batch 16 146x146x96 32.3 -> 26.1 and 35.0 -> 28.0 (input gradient), batch 16
// 50x50x300 14.8 -> 13.4, batch 64 13x90x64 8.7 -> 7.7.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(512) void k_nchwf_conv_pairs(const bf16_t *__restrict__ in, const bf16_t *__restrict__ w, bf16_t *__restrict__ out,
                                                          int nplanes, int OC, int H, int W, int mdiv, int total_in, int flip, FlatTile ft,
                                                          unsigned nblocks, Geom g)
{
    extern __shared__ uint4 smem[];
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int band = (int)(lb % (unsigned)ft.nbands), p0 = (int)(lb / (unsigned)ft.nbands) * ft.U;
    const int np = min(ft.U, nplanes - p0);
    const int oh0 = band * ft.TR, oh1 = min(H, oh0 + ft.TR);
    const int ip0 = p0 / mdiv, ip1 = (p0 + np - 1) / mdiv + 1;
    const int r0 = max(oh0 - 1, 0), r1 = min(oh1 + 1, H);
    const Bands bi = {ip0, ip1 - ip0, H * W, W, r0, r1, ft.pin};
    bf16_t *lin = reinterpret_cast<bf16_t *>(smem) + GUARD;
    dma_bands<bf16_t>(in, total_in, bi, lin);

    const int ncol = W / 2, u = (int)threadIdx.x / ncol, ow = ((int)threadIdx.x - u * ncol) * 2;
    const bool active = u < np;
    const int pl = p0 + (active ? u : 0), oc = pl % OC;
    // of the word to the left the right half, of the one to the right the left half
    const uint32_t okl = ow > 0 ? 0xffff0000u : 0u, okr = ow + 2 < W ? 0x0000ffffu : 0u;
    uint32_t wl[3], w12[3], w01[3], wrt[3];                 // filter rows against the three words: (0, w0), (w1, w2) and (w0, w1), (w2, 0)
    NonFinite bad;
#pragma unroll
    for (int kh = 0; kh < 3; ++kh) {
        uint32_t e[3];
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
            const int tap = kh * 3 + kw;
            e[kw] = w[oc * 9 + (flip ? 8 - tap : tap)];
            bad.add(bf16_to_f32((bf16_t)e[kw]));
        }
        wl[kh] = e[0] << 16; w12[kh] = e[1] | e[2] << 16;
        w01[kh] = e[0] | e[1] << 16; wrt[kh] = e[2];
    }
    const bool redo = bad.any() && active;
    // (rows of an even width start at even elements: the words are aligned)
    const bf16_t *p = lin + bi.at<bf16_t>(pl / mdiv - ip0) + ow - r0 * W;
    const BufView vout(out + (size_t)p0 * H * W, (uint32_t)(np * H * W) * 2u);
    const uint32_t voff = active ? (uint32_t)((u * H + oh0) * W + ow) * 2u : BufView::OUTSIDE;
    float acc[3][2];
#pragma unroll
    for (int i = 0; i < 6; ++i) acc[i / 2][i % 2] = 0.f;
    dma_wait();
    __syncthreads();

    // step t reads image row oh0 - 1 + t, which meets the outputs of rows oh0 + t - i; the one with i = 2 is complete
    const int rows = oh1 - oh0;
    auto step = [&](int t, auto checked) {
        constexpr bool CK = decltype(checked)::value;
        const int row = oh0 - 1 + t;                       // everything about the row is uniform
        if (!CK || (unsigned)row < (unsigned)H) {
            const uint32_t *q = reinterpret_cast<const uint32_t *>(p + row * W);
            const uint32_t l = q[-1] & okl, m = q[0], r = q[1] & okr;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                acc[i][0] = dot2_bf16(m, w12[i], dot2_bf16(l, wl[i], acc[i][0]));
                acc[i][1] = dot2_bf16(r, wrt[i], dot2_bf16(m, w01[i], acc[i][1]));
            }
        }
        if (!CK || t >= 2) store_two<bf16_t>(vout, acc[2][0], acc[2][1], voff, (uint32_t)((t - 2) * W) * 2u);
#pragma unroll
        for (int i = 2; i > 0; --i) { acc[i][0] = acc[i - 1][0]; acc[i][1] = acc[i - 1][1]; }
        acc[0][0] = acc[0][1] = 0.f;
    };
    const int steps = rows + 2, tb = min(steps, H + 1 - oh0);      // steps [2, tb) have their row inside the image
    int t = 0;
    for (; t < 2; ++t) step(t, std::true_type());
#pragma unroll 3
    for (; t < tb; ++t) step(t, std::false_type());
    for (; t < steps; ++t) step(t, std::true_type());
    if (__builtin_expect(redo, 0)) {          // the lane's columns again, without the padding
        const int n = pl / OC;
#pragma unroll 1
        for (int i = 0; i < 2 * rows; ++i) {
            const int row = oh0 + i / 2, cw = ow + i % 2;
            stf(out + ((size_t)pl * H + row) * W + cw,
                flip ? point_bwd_data<bf16_t, LAYOUT_NCHW>(g, in, w, n, oc, row, cw) : point_fwd<bf16_t, LAYOUT_NCHW>(g, in, w, n, oc, row, cw));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Input gradient of a stride-2 layer.  With h + p = 2a + f and c + p = 2b + e the taps that reach dx[h][c] are kh = 2k + f,
// kw = 2l + e against dy[a - k][b - l]: a lane owns two neighbouring dx columns, walks down the dy rows with the K/2 row
// pairs a row reaches in rotating accumulators, and a dy row costs (K+1)/2 reads and K*K multiply-adds for four outputs.
// SH: the columns are e = 0, 1 of one b for an even padding and e = 1 of b, e = 0 of b + 1 for an odd one, so that either way
// the first is even and rows of an even width take both in one aligned store (74x74x256 3x3 fp32: 71 us with the pairs at odd columns).
// ---------------------------------------------------------------------------------------------
template <typename T, int K, int M, int SH>
__global__ __launch_bounds__(512) void k_nchwf_bwd_data_s2(const T *__restrict__ dy, const T *__restrict__ w, T *__restrict__ dx,
                                                           int nplanes, int C, int H, int W, int Ho, int Wo, int pad, int NB,
                                                           int total_dy, FlatTile ft, unsigned nblocks, Geom g)
{
    extern __shared__ uint4 smem[];
    constexpr int NA = (K + 1) / 2;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int band = (int)(lb % (unsigned)ft.nbands), p0 = (int)(lb / (unsigned)ft.nbands) * ft.U;
    const int np = min(ft.U, nplanes - p0);
    const int a0 = pad / 2 + band * ft.TR, a1 = min((H - 1 + pad) / 2 + 1, a0 + ft.TR);      // row pairs of the band
    const int r0 = min(max(a0 - (NA - 1), 0), Ho), r1 = max(min(a1, Ho), r0);
    const int h0 = max(2 * a0 - pad, 0), h1 = min(2 * a1 - pad, H);
    const Bands bi = {p0 * M, np * M, Ho * Wo, Wo, r0, r1, ft.pin};
    T *lin = reinterpret_cast<T *>(smem) + GUARD;
    dma_bands<T>(dy, total_dy, bi, lin);

    const int u = (int)threadIdx.x / NB, bi0 = (int)threadIdx.x - u * NB, b = (pad - SH) / 2 + bi0;
    const bool active = u < np;
    const int pl = p0 + (active ? u : 0), c = pl % C;
    uint32_t ok[NA];
#pragma unroll
    for (int l = 0; l < NA; ++l) ok[l] = (unsigned)(b + SH - l) < (unsigned)Wo ? ~0u : 0u;
    const int colb = min(b + SH, Wo + NA - 1);                  // a column further out has every tap dropped anyway
    float wr[M][K][K];
    int src[M];
#pragma unroll
    for (int q = 0; q < M; ++q) {
#pragma unroll
        for (int kh = 0; kh < K; ++kh)
#pragma unroll
            for (int kw = 0; kw < K; ++kw) wr[q][kh][kw] = ldf(w + (c * M + q) * K * K + kh * K + kw);
        src[q] = bi.at<T>((active ? u : 0) * M + q) + colb;
    }
    // columns col and col + 1; one that is none is stored outside the view.  Rows of an even width: one aligned store for both.
    const int col = 2 * bi0;
    const bool even = W % 2 == 0;
    const BufView vout(dx + (size_t)p0 * H * W, (uint32_t)(np * H * W) * (uint32_t)sizeof(T));
    const uint32_t v0 = active ? (uint32_t)(u * H * W + col) * (uint32_t)sizeof(T) : BufView::OUTSIDE;
    const uint32_t v1 = active && col + 1 < W ? v0 + (uint32_t)sizeof(T) : BufView::OUTSIDE;
    float acc[NA][2][2];
#pragma unroll
    for (int k = 0; k < NA; ++k) acc[k][0][0] = acc[k][0][1] = acc[k][1][0] = acc[k][1][1] = 0.f;
    NonFinite bad;
#pragma unroll
    for (int q = 0; q < M; ++q)
#pragma unroll
        for (int e = 0; e < K * K; ++e) bad.add(wr[q][e / K][e % K]);
    const bool redo = bad.any() && active;
    dma_wait();
    __syncthreads();

    // dy row r reaches the row pairs r .. r + NA - 1; pair r is complete after it.  Rows [r0, r1) are in the band.
    auto step = [&](int r, auto read, auto checked) {
        constexpr bool CK = decltype(checked)::value;
        if constexpr (decltype(read)::value) {
#pragma unroll
            for (int q = 0; q < M; ++q) {
                const T *p = lin + src[q] + (r - r0) * Wo;
                float v[NA];
#pragma unroll
                for (int l = 0; l < NA; ++l) v[l] = masked(ldf(p - l), ok[l]);
#pragma unroll
                for (int k = 0; k < NA; ++k)
#pragma unroll
                    for (int f = 0; f < 2; ++f)
#pragma unroll
                        for (int l = 0; l < NA; ++l)
#pragma unroll
                            for (int e = 0; e < 2; ++e)
                                if (2 * k + f < K && 2 * l + e < K) acc[k][f][e] = fmaf(wr[q][2 * k + f][2 * l + e], v[e ? l + SH : l], acc[k][f][e]);
            }
        }
        if (!CK || r >= a0) {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int h = 2 * r - pad + f;
                if (!CK || (h >= h0 && h < h1)) {              // uniform
                    const uint32_t so = (uint32_t)(h * W) * (uint32_t)sizeof(T);
                    if (even) store_two<T>(vout, acc[0][f][SH], acc[0][f][1 - SH], v0, so);
                    else {
                        store_one<T>(vout, acc[0][f][SH], v0, so);
                        store_one<T>(vout, acc[0][f][1 - SH], v1, so);
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[k][i >> 1][i & 1] = k + 1 < NA ? acc[k + 1][i >> 1][i & 1] : 0.f;
    };
    // rows above r0 are padding; pairs [ra, rb) lie in the band with both their rows
    const int ra = a0 + (2 * a0 - pad < h0 ? 1 : 0), rb = min(r1, a1 - (2 * a1 - pad > h1 ? 1 : 0));
    int r = max(a0 - (NA - 1), r0);
    for (; r < min(ra, r1); ++r) step(r, std::true_type(), std::true_type());
#pragma unroll NA
    for (; r < rb; ++r) step(r, std::true_type(), std::false_type());
    for (; r < r1; ++r) step(r, std::true_type(), std::true_type());
    for (; r < a1; ++r) step(r, std::false_type(), std::true_type());
    if (__builtin_expect(redo, 0)) {          // the lane's columns again, without the padding
        const int n = pl / C;
#pragma unroll 1
        for (int i = 0; i < 2 * (h1 - h0); ++i) {
            const int h = h0 + i / 2, cw = col + i % 2;
            if ((unsigned)cw < (unsigned)W) stf(dx + ((size_t)pl * H + h) * W + cw, point_bwd_data<T, LAYOUT_NCHW>(g, dy, w, n, c, h, cw));
        }
    }
}

// The sums of a block's lanes, channel by channel (`np` of them from o0 on, `ncol` lanes each), to its partial.
template <int K, int SETS>
__device__ __forceinline__ void add_columns(const float (&acc)[SETS][K][K], float *red, float *__restrict__ dst, int np, int ncol, int o0)
{
    // CH sums at a time (all of them up to 5x5): [CH][threads] in LDS, then Q lanes per (channel, tap) add every Q-th column
    const int Q = ncol < 16 ? 1 : ncol < 64 ? 4 : 8;
    constexpr int CH = K * K <= 25 ? K * K : 25;
    const int nt = blockDim.x;
#pragma unroll
    for (int e0 = 0; e0 < K * K; e0 += CH) {
        const int ne = K * K - e0 < CH ? K * K - e0 : CH;
#pragma unroll
        for (int e = 0; e < CH; ++e)
            if (e0 + e < K * K) {
                const float s = acc[0][(e0 + e) / K][(e0 + e) % K];
                red[e * nt + threadIdx.x] = SETS == 2 ? s + acc[SETS - 1][(e0 + e) / K][(e0 + e) % K] : s;
            }
        __syncthreads();
        const int jobs = np * ne;
        for (int f0 = 0; f0 < jobs * Q; f0 += nt) {        // uniform trip count
            const int f = f0 + (int)threadIdx.x, job = f / Q, q = f & (Q - 1);
            const int uj = job / ne, e = job - uj * ne;
            float s = 0.f;
            if (job < jobs) {                              // four sums side by side: a chain of n adds 2^-24 * sqrt(n / 6) to the error
                const float *col = red + e * nt + uj * ncol;
                float p[4] = {0.f, 0.f, 0.f, 0.f};
                int i = q;
                for (; i + 3 * Q < ncol; i += 4 * Q) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) p[k] += col[i + k * Q];
                }
                for (; i < ncol; i += Q) p[0] += col[i];
                s = (p[0] + p[1]) + (p[2] + p[3]);
            }
            for (int h = Q >> 1; h >= 1; h >>= 1) s += __shfl_xor(s, h, 64);
            if (job < jobs && q == 0) dst[(o0 + uj) * K * K + e0 + e] = s;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Filter gradient, stage 1.  A block owns U output channels and walks (image, band) items: x bands staged as above, dy read by the
// lanes that own its columns a few rows ahead (or from LDS, see DY_LDS); a lane keeps the K*K sums of its column over all of
// them against a window of the last K/S dy rows.  The columns of a channel are added through LDS in a fixed order at the end,
// one partial per block.
// ---------------------------------------------------------------------------------------------
template <typename T, int K, int S, bool SAME, int NC, bool DYLDS, int SETS>
__global__ __launch_bounds__(512) void k_nchwf_bwd_filter(Geom g, const T *__restrict__ x, const T *__restrict__ dy,
                                                          float *__restrict__ ws, int parts, int per_part, FlatTile ft,
                                                          unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    constexpr int NA = (K + S - 1) / S;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int part = (int)(lb % (unsigned)parts), o0 = (int)(lb / (unsigned)parts) * ft.U;
    const int np = min(ft.U, g.O - o0);
    const int c0 = o0 / g.m, c1 = (o0 + np - 1) / g.m + 1;
    constexpr int VW = S * (NC - 1) + K;
    const int ncol = (g.Wo + NC - 1) / NC;
    const int u = (int)threadIdx.x / ncol, ow = ((int)threadIdx.x - u * ncol) * NC;
    const bool active = u < np;
    const int uu = active ? u : 0, ju = (o0 + uu) / g.m - c0;
    uint32_t ok[VW];
#pragma unroll
    for (int i = 0; i < VW; ++i) ok[i] = (unsigned)(ow * S - g.p + i) < (unsigned)g.W ? ~0u : 0u;
    const int col0 = min(max(ow * S - g.p, -VW), g.W);
    T *lx = reinterpret_cast<T *>(smem) + GUARD;
    // the dy columns of the lane; one that is none reads as zero
    uint32_t offd[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) offd[n] = active && ow + n < g.Wo ? (uint32_t)(u * g.Ho * g.Wo + ow + n) * (uint32_t)sizeof(T) : BufView::OUTSIDE;
    // SETS = 2: steps add to either set in turn
    float acc[SETS][K][K];
#pragma unroll
    for (int e = 0; e < SETS * K * K; ++e) acc[e / (K * K)][e / K % K][e % K] = 0.f;

    const int items = g.N * ft.nbands, it1 = part_end(items, per_part, part);
    for (int it = part * per_part; it < it1; ++it) {
        // The last prefetches of dy are in flight and dead; a wait for their registers inside dma_bands' loop would wait for every
        // DMA (44x44x78 5x5 stride 2 fp32 batch 390: 104 -> 82 us)
        __builtin_amdgcn_s_waitcnt(0xf70);                  // vmcnt(0)
        const int n = it / ft.nbands, band = it - n * ft.nbands;
        const int oh0 = band * ft.TR, oh1 = min(g.Ho, oh0 + ft.TR);
        const int r0 = min(max(oh0 * S - g.p, 0), g.H), r1 = max(min((oh1 - 1) * S - g.p + K, g.H), r0);
        const Bands bx = {n * g.C + c0, c1 - c0, g.H * g.W, g.W, r0, r1, ft.pin};
        const BufView vd(dy + (size_t)(n * g.O + o0) * g.Ho * g.Wo, (uint32_t)(np * g.Ho * g.Wo) * (uint32_t)sizeof(T));
        dma_bands<T>(x, g.N * g.C * g.H * g.W, bx, lx);
        const T *px = lx + bx.at<T>(ju) + col0;
        const T *pd = lx;
        if constexpr (DYLDS) {
            const Bands by = {n * g.O + o0, np, g.Ho * g.Wo, g.Wo, oh0, oh1, ft.pout};
            T *ldy = lx + ft.nin + GUARD;
            dma_bands<T>(dy, g.N * g.O * g.Ho * g.Wo, by, ldy);
            pd = ldy + by.at<T>(active ? u : 0) + (active ? ow : 0);
        }
        float d[NA][NC];
#pragma unroll
        for (int i = 0; i < NA; ++i)
#pragma unroll
            for (int n = 0; n < NC; ++n) d[i][n] = 0.f;
        const int rows = oh1 - oh0, steps = rows + NA - 1;
        // dy rows t .. t + PD - 1 are on their way (3x3: three rows ahead 84 us at 74x74x256 fp32, six 74, nine 84; 5x5: five 67 at
        // 41x41x240, ten 70)
        constexpr int PD = K == 3 ? 6 : NA;
        T dq[PD][NC];
        auto fetch = [&](int t, T (&q)[NC]) {
#pragma unroll
            for (int n = 0; n < NC; ++n) q[n] = load_one<T>(vd, offd[n], (uint32_t)((oh0 + min(t, rows - 1)) * g.Wo) * (uint32_t)sizeof(T));
        };
        if constexpr (!DYLDS) {
#pragma unroll
            for (int i = 0; i < PD; ++i) fetch(i, dq[i]);
        }
        dma_wait();
        __syncthreads();
        // step t: the S x rows from row (oh0 + t)*S - p on, against dy rows oh0 + t - i; steps [ta, tb) have all of them in the band
        const int base = oh0 * S - g.p - r0, nrows = r1 - r0;
        auto step = [&](int t, auto checked, int set) {
            constexpr bool CK = decltype(checked)::value;
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                if constexpr (DYLDS) d[0][n] = !CK || t < rows ? ldf(pd + t * g.Wo) : 0.f;
                else {
                    const float f = ldf(&dq[0][n]);
                    d[0][n] = !CK || t < rows ? f : 0.f;
                }
            }
            if constexpr (!DYLDS) {
#pragma unroll
                for (int i = 0; i + 1 < PD; ++i)
#pragma unroll
                    for (int n = 0; n < NC; ++n) dq[i][n] = dq[i + 1][n];
                fetch(t + PD, dq[PD - 1]);
            }
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const int row = base + t * S + j;
                if (CK && (row < 0 || row >= nrows)) continue;
                const T *p = px + row * g.W;
                float v[VW];
#pragma unroll
                for (int i = 0; i < VW; ++i) {
                    const float e = ldf(p + i);
                    v[i] = SAME && NC == 1 && i == K / 2 ? e : masked(e, ok[i]);
                }
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    if (j + i * S >= K || (CK && K > 3 && (unsigned)(t - i) >= (unsigned)rows)) continue;
#pragma unroll
                    for (int kw = 0; kw < K; ++kw)
#pragma unroll
                        for (int n = 0; n < NC; ++n) acc[set][j + i * S][kw] = fmaf(d[i][n], v[n * S + kw], acc[set][j + i * S][kw]);
                }
            }
#pragma unroll
            for (int i = NA - 1; i > 0; --i)
#pragma unroll
                for (int n = 0; n < NC; ++n) d[i][n] = d[i - 1][n];
        };
        const int ta = (S - 1 - base) / S, tb = min((nrows - base) / S, rows);
        int t = 0;
        constexpr int UN = DYLDS ? NA : PD;                 // steps after which the windows are in the same registers
        for (; t < min(K > 3 ? max(ta, NA - 1) : ta, steps); ++t) step(t, std::true_type(), 0);
        if constexpr (SETS == 2) {
#pragma unroll 1
            for (; t + UN <= tb; t += UN) {
#pragma unroll
                for (int i = 0; i < UN; ++i) step(t + i, std::false_type(), i % 2);
            }
        }
#pragma unroll SETS == 2 ? 1 : UN
        for (; t < tb; ++t) step(t, std::false_type(), 0);
        for (; t < steps; ++t) step(t, std::true_type(), 0);
        __syncthreads();
    }

    add_columns<K, SETS>(acc, reinterpret_cast<float *>(smem), ws + (size_t)part * g.O * K * K, np, ncol, o0);
}

// ---------------------------------------------------------------------------------------------
// The same on column pairs (see k_nchwf_conv_pairs): the two products of a tap and a pair are one packed dot product, of the dy word with the
// x word of the same columns or with one put together from two of them.
// us with stage 2, one column a lane -> this: 74x74x256 batch 32 54.7 -> 52.5, 146x146x96 batch 16 44.4 -> 35.4, 13x90x64 batch 64 12.8 -> 11.1.
// ---------------------------------------------------------------------------------------------
template <bool DYLDS>
__global__ __launch_bounds__(512) void k_nchwf_bwd_filter_pairs(Geom g, const bf16_t *__restrict__ x, const bf16_t *__restrict__ dy, float *__restrict__ ws,
                                                                int parts, int per_part, FlatTile ft, unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    constexpr int PD = 6;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int part = (int)(lb % (unsigned)parts), o0 = (int)(lb / (unsigned)parts) * ft.U;
    const int np = min(ft.U, g.O - o0), W = g.W, HW = g.H * g.W;
    const int c0 = o0 / g.m, c1 = (o0 + np - 1) / g.m + 1;
    const int ncol = W / 2, u = (int)threadIdx.x / ncol, ow = ((int)threadIdx.x - u * ncol) * 2;
    const bool active = u < np;
    const int uu = active ? u : 0, ju = (o0 + uu) / g.m - c0;
    const uint32_t okl = ow > 0 ? ~0u : 0u, okr = ow + 2 < W ? ~0u : 0u, here = active ? ~0u : 0u;
    bf16_t *lx = reinterpret_cast<bf16_t *>(smem) + GUARD;
    const uint32_t offd = active ? (uint32_t)(u * HW + ow) * 2u : BufView::OUTSIDE;
    float acc[2][3][3];
#pragma unroll
    for (int e = 0; e < 18; ++e) acc[e / 9][e / 3 % 3][e % 3] = 0.f;

    const int items = g.N * ft.nbands, it1 = part_end(items, per_part, part);
    for (int it = part * per_part; it < it1; ++it) {
        __builtin_amdgcn_s_waitcnt(0xf70);                  // vmcnt(0): the last prefetches (see above)
        const int n = it / ft.nbands, band = it - n * ft.nbands;
        const int oh0 = band * ft.TR, oh1 = min(g.H, oh0 + ft.TR), rows = oh1 - oh0;
        const int r0 = max(oh0 - 1, 0), r1 = min(oh1 + 1, g.H);
        const Bands bx = {n * g.C + c0, c1 - c0, HW, W, r0, r1, ft.pin};
        const BufView vd(dy + (size_t)(n * g.O + o0) * HW, (uint32_t)(np * HW) * 2u);
        dma_bands<bf16_t>(x, g.N * g.C * HW, bx, lx);
        const bf16_t *px = lx + bx.at<bf16_t>(ju) + ow - r0 * W;           // row r of the image at px + r * W
        const bf16_t *pd = lx;
        if constexpr (DYLDS) {
            const Bands by = {n * g.O + o0, np, HW, W, oh0, oh1, ft.pout};
            bf16_t *ldy = lx + ft.nin + GUARD;
            dma_bands<bf16_t>(dy, g.N * g.O * HW, by, ldy);
            pd = ldy + by.at<bf16_t>(uu) + ow;
        }
        uint32_t dq[PD];
        auto fetch = [&](int t) { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(vd.rsrc, (int)offd, (int)((uint32_t)((oh0 + min(t, rows - 1)) * W) * 2u), 0); };
        if constexpr (!DYLDS) {
#pragma unroll
            for (int i = 0; i < PD; ++i) dq[i] = fetch(i);
        }
        dma_wait();
        __syncthreads();
        // x row oh0 - 1 + t meets dy rows oh0 + t - kh, tap row kh; d[kh]: that dy row, zero where the band has none
        uint32_t d[3] = {0u, 0u, 0u};
        auto step = [&](int t, auto checked, int set) {
            constexpr bool CK = decltype(checked)::value;
            if constexpr (DYLDS) d[0] = !CK || t < rows ? *reinterpret_cast<const uint32_t *>(pd + t * W) & here : 0u;
            else {
                d[0] = !CK || t < rows ? dq[0] : 0u;
#pragma unroll
                for (int i = 0; i + 1 < PD; ++i) dq[i] = dq[i + 1];
                dq[PD - 1] = fetch(t + PD);
            }
            const int row = oh0 - 1 + t;
            if (!CK || (unsigned)row < (unsigned)g.H) {
                const uint32_t *q = reinterpret_cast<const uint32_t *>(px + row * W);
                const uint32_t m = q[0];
                // columns (c - 1, c), (c, c + 1), (c + 1, c + 2)
                const uint32_t e[3] = {__builtin_amdgcn_perm(m, q[-1] & okl, 0x05040302u), m, __builtin_amdgcn_perm(q[1] & okr, m, 0x05040302u)};
#pragma unroll
                for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw) acc[set][kh][kw] = dot2_bf16(d[kh], e[kw], acc[set][kh][kw]);
            }
            d[2] = d[1]; d[1] = d[0];
        };
        const int steps = rows + 2, tb = min(rows, g.H + 1 - oh0);         // steps [1, tb) have both their rows
        int t = 0;
        step(t++, std::true_type(), 0);
#pragma unroll 1
        for (; t + PD <= tb; t += PD) {
#pragma unroll
            for (int i = 0; i < PD; ++i) step(t + i, std::false_type(), i % 2);
        }
#pragma unroll 1
        for (; t < tb; ++t) step(t, std::false_type(), 0);
        for (; t < steps; ++t) step(t, std::true_type(), 0);
        __syncthreads();
    }
    add_columns<3, 2>(acc, reinterpret_cast<float *>(smem), ws + (size_t)part * g.O * 9, np, ncol, o0);
}

// ---------------------------------------------------------------------------------------------
// Whole backward pass, 3x3 "same" stride 1, multiplier 1: the input gradient and stage 1 of the filter gradient from one walk over x and
// dy.  Blocks and items of the filter gradient; the dy bands with their halo rows go to LDS, a lane reads x only in its own column, a few
// rows ahead.  The 3x3 window of dy around (row t, column c) gives dx[t][c] and, its middle row against x rows t - 1, t and t + 1 of
// column c, the filter gradient summed per x column: 18 multiply-adds for three LDS reads, one load and one store.
// The two passes and this one, stage 2 in both, us on one MI355X: 19x19x728 batch 32 fp32 33.5 -> 25.3, bf16 28.3 -> 21.4; 74x74x256 batch 32 162 -> 129 and
// 96 -> 83 (one column a lane in both; on pairs 89); 147x147x96 batch 16 134 -> 104; 10x10x240 batch 128 22.2 -> 16.8; 21x21x32 batch 8 11.3 -> 8.4.  On
// rows that neither pass takes in pairs it is 0.76 of the two at the mean of 40 000 random layers, and none was longer by 8 % and a microsecond;
// for the others see two_passes_shorter.
// ---------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(512) void k_nchwf_bwd_fused(Geom g, const T *__restrict__ x, const T *__restrict__ dy, const T *__restrict__ w,
                                                         T *__restrict__ dx, float *__restrict__ ws, int parts, int per_part, FlatTile ft,
                                                         unsigned nblocks)
{
    extern __shared__ uint4 smem[];
    constexpr int PD = 6;                                  // x rows on their way; a multiple of the window, so that it returns to its registers
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int part = (int)(lb % (unsigned)parts), o0 = (int)(lb / (unsigned)parts) * ft.U;
    const int np = min(ft.U, g.O - o0), W = g.W, HW = g.H * g.W;
    const int u = (int)threadIdx.x / W, c = (int)threadIdx.x - u * W;
    const bool active = u < np;
    const int uu = active ? u : 0;
    const uint32_t okl = c > 0 ? ~0u : 0u, okr = c < W - 1 ? ~0u : 0u;
    T *ld = reinterpret_cast<T *>(smem) + GUARD;
    const uint32_t off = active ? (uint32_t)(u * HW + c) * (uint32_t)sizeof(T) : BufView::OUTSIDE;      // a column that is none reads zero and is not stored
    float wr[3][3];
    NonFinite bad;
#pragma unroll
    for (int e = 0; e < 9; ++e) { wr[e / 3][e % 3] = ldf(w + (o0 + uu) * 9 + e); bad.add(wr[e / 3][e % 3]); }
    const bool redo = bad.any() && active;
    float acc[2][3][3];
#pragma unroll
    for (int e = 0; e < 18; ++e) acc[e / 9][e / 3 % 3][e % 3] = 0.f;

    const int items = g.N * ft.nbands, it1 = part_end(items, per_part, part);
    for (int it = part * per_part; it < it1; ++it) {
        __builtin_amdgcn_s_waitcnt(0xf70);                  // vmcnt(0): the last prefetches (see the filter gradient)
        const int n = it / ft.nbands, band = it - n * ft.nbands;
        const int oh0 = band * ft.TR, oh1 = min(g.H, oh0 + ft.TR), rows = oh1 - oh0;
        const int r0 = max(oh0 - 1, 0), r1 = min(oh1 + 1, g.H);
        const size_t image = (size_t)(n * g.O + o0) * HW;
        const uint32_t bytes = (uint32_t)(np * HW) * (uint32_t)sizeof(T);
        const BufView vx(x + image, bytes), vout(dx + image, bytes);
        const Bands b = {n * g.O + o0, np, HW, W, r0, r1, ft.pin};
        dma_bands<T>(dy, g.N * g.O * HW, b, ld);
        T xq[PD];
        auto fetch = [&](int t) { return load_one<T>(vx, off, (uint32_t)(min(max(oh0 + t, 0), g.H - 1) * W) * (uint32_t)sizeof(T)); };
        const T xa = fetch(-1), xb = fetch(0);
#pragma unroll
        for (int i = 0; i < PD; ++i) xq[i] = fetch(min(i + 1, rows));
        dma_wait();
        __syncthreads();
        const T *p = ld + b.at<T>(uu) + c - 1 - r0 * W;      // row r of the image at p + r * W
        auto read = [&](int r, float (&v)[3]) {
            const T *q = p + r * W;
            v[0] = masked(ldf(q), okl); v[1] = ldf(q + 1); v[2] = masked(ldf(q + 2), okr);
        };
        float d[3][3], xw[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) d[0][i] = 0.f;
        if (oh0 > 0) read(oh0 - 1, d[0]);
        read(oh0, d[1]);
        xw[0] = oh0 > 0 ? ldf(&xa) : 0.f; xw[1] = ldf(&xb);
        // step t: row oh0 + t of dx and of dy; the rows below it are read here
        auto step = [&](int t, auto last, int set) {
            constexpr bool LAST = decltype(last)::value;     // the plane's last row
            if constexpr (LAST) {
#pragma unroll
                for (int i = 0; i < 3; ++i) d[2][i] = 0.f;
                xw[2] = 0.f;
            } else {
                read(oh0 + t + 1, d[2]);
                xw[2] = ldf(&xq[0]);
            }
#pragma unroll
            for (int i = 0; i + 1 < PD; ++i) xq[i] = xq[i + 1];
            if constexpr (!LAST) xq[PD - 1] = fetch(min(t + 1 + PD, rows));
            float s = 0.f;
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int kw = 0; kw < 3; ++kw) {
                    s = fmaf(wr[2 - kh][2 - kw], d[kh][kw], s);       // in the order of the separate pass (one column a lane)
                    acc[set][kh][kw] = fmaf(d[1][2 - kw], xw[kh], acc[set][kh][kw]);
                }
            store_one<T>(vout, s, off, (uint32_t)((oh0 + t) * W) * (uint32_t)sizeof(T));
#pragma unroll
            for (int i = 0; i < 3; ++i) { d[0][i] = d[1][i]; d[1][i] = d[2][i]; }
            xw[0] = xw[1]; xw[1] = xw[2];
        };
        const int tb = oh1 < g.H ? rows : rows - 1;
        int t = 0;
#pragma unroll 1
        for (; t + PD <= tb; t += PD) {
#pragma unroll
            for (int i = 0; i < PD; ++i) step(t + i, std::false_type(), i % 2);
        }
#pragma unroll 1
        for (; t < tb; ++t) step(t, std::false_type(), 0);
        if (t < rows) step(t, std::true_type(), 0);
        if (__builtin_expect(redo, 0)) {          // the lane's column again, without the padding
#pragma unroll 1
            for (int h = oh0; h < oh1; ++h) stf(dx + image + (size_t)u * HW + h * W + c, point_bwd_data<T, LAYOUT_NCHW>(g, dy, w, n, o0 + u, h, c));
        }
        __syncthreads();
    }
    add_columns<3, 2>(acc, reinterpret_cast<float *>(smem), ws + (size_t)part * g.O * 9, np, W, o0);
}

// ---- host side --------------------------------------------------------------------------------

namespace {

// U planes of `cols` lanes each and the block size that leave the fewest lanes idle, at up to 256 threads (blocks of 448 filled
// better on rows of 74 and 147 and still measured 5-20 % slower: fewer of them overlap), 512 for wider rows.
void pick_lanes(int cols, int planes, int maxu, int *U, int *threads)
{
    double best = -1.0;
    *U = 0;
    const int tmax = cols > 256 ? 512 : 256;
    for (int t = 192; t <= tmax; t += 64) {
        int u = t / cols;
        if (u > maxu) u = maxu;
        if (u > planes) u = planes;
        if (u < 1) continue;
        int tt = (u * cols + 63) / 64 * 64;
        const double eff = (double)(u * cols) / tt;
        if (eff > best + 1e-9) { best = eff; *U = u; *threads = tt; }
    }
}

// LDS of a block.  Bands of about 32 KiB, 40 for the longer halos of 5x5 and 7x7, whole planes, which have no halo, up to 40 KiB: less
// reads too many halo rows, more leaves too few blocks to overlap, with little between 24 and 40 (56x56x128 5x5 stride 2 fp32 forward at
// batch 64 16 KiB 35 us, 24 31, 32 29, 40 30, filter gradient 46, 51, 48, 44; 56x56 5x5 multiplier 2 input gradient 16 KiB 99, 20 96,
// 24 84, 32 83, 40 81).
inline int lds_target(int K) { return K == 3 ? 32 << 10 : 40 << 10; }
constexpr int LDS_WHOLE = 40 << 10;
constexpr int LDS_MOST = 64 << 10;
constexpr int MIN_LANES = 65536, LEAST_BAND = 256, LEAST_FILTER_BAND = 1024;

inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

int second_area(const FlatTile &ft) { return GUARD + ft.U * ft.pout; }       // LDS elements of the dy bands of a tile

// Tile of a launch: `cols` lanes per plane; a band of t units (rows, or row pairs) needs in_rows(t) input rows; Mi input planes per
// output plane, or mdiv output planes per input plane; copies: launches of the planes side by side (images of the filter gradient);
// second: bands of the output rows are in LDS too; least: see the end.
template <typename FI>
bool pick_tile(int esz, int cols, int units, int nplanes, int maxu, int Hi, int Wi, int Ho, int Wo, FI in_rows, int Mi, int mdiv,
               int target, FlatTile *ft, int copies, int least, bool second = false)
{
    const int VE = 16 / esz;
    // a block's planes are one buffer view (2 GiB at most)
    const long long fit = ((1LL << 31) - 1) / ((long long)Ho * Wo * esz);
    pick_lanes(cols, nplanes, fit < maxu ? (int)fit : maxu, &ft->U, &ft->threads);
    if (ft->U < 1) return false;
    for (;;) {
        const int nin_planes = Mi > 1 ? ft->U * Mi : (mdiv > 1 ? (ft->U - 1) / mdiv + 2 : ft->U);
        auto lds = [&](int t, FlatTile *o) {
            const bool whole = t >= units;
            const int ir = in_rows(t) < Hi ? in_rows(t) : Hi;
            o->TR = t; o->nbands = whole ? 1 : (units + t - 1) / t;
            o->pin = whole ? 0 : round_up(ir * Wi + VE, VE);
            o->nin = whole ? round_up(nin_planes * Hi * Wi + VE, VE) : nin_planes * o->pin;
            o->pout = second ? round_up(t * Wo + VE, VE) : 0;
            return (long long)(o->nin + 2 * GUARD + (second ? second_area(*o) : 0)) * esz;
        };
        int t = units;
        if (lds(t, ft) > LDS_WHOLE) {                        // the tallest band within the target, by bisection
            int lo = 1, hi = units - 1 > 1 ? units - 1 : 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) / 2;
                if (lds(mid, ft) <= target) lo = mid; else hi = mid - 1;
            }
            t = lo;
        }
        // balanced bands
        const int nb = (units + t - 1) / t;
        t = (units + nb - 1) / nb;
        if (lds(t, ft) <= LDS_MOST && (t >= 4 || t >= units || ft->U == 1)) {
            // A launch of fewer than MIN_LANES lanes is one short round of blocks, each as long as its band: bands of half the height,
            // and half again down to four rows, while a plane's band is `least` bytes and more.  Each is a DMA of its own, of up to 1024
            // bytes, where whole planes of a block are one stream.  Of random layers with rows of up to 60, with every band halved / none below
            // 256 bytes: 10 / 0.4 % of the 3x3 and 17 / 1.0 % of the 5x5 forward passes on rows under 13 were slower by more than a tenth than with
            // the tall bands (15x50x23x3 3x3 stride 2: 7.4 and 4.9 us); the filter gradient, whose bands are partials too, below 1024: 20 / 0.1 %.
            const long long groups = (long long)((nplanes - 1) / ft->U + 1) * copies;
            while (ft->TR > 4 && groups * ft->nbands * ft->threads < MIN_LANES) {
                const int h = (ft->TR + 1) / 2, n = (units + h - 1) / h, t2 = (units + n - 1) / n;
                if ((long long)in_rows(t2) * Wi * esz < least) break;
                lds(t2, ft);
            }
            return true;
        }
        if (ft->U == 1) return false;
        ft->U = (ft->U + 1) / 2;
        ft->threads = (ft->U * cols + 63) / 64 * 64;
    }
}

size_t tile_lds(const FlatTile &ft, int esz) { return (size_t)(ft.nin + 2 * GUARD) * esz; }

// Planes per block, at most: about two blocks per compute unit in the launch (planes of more than 24 rows are several bands),
// but a wavefront's worth of columns.
int most_planes(long long planes, int rows, int cols)
{
    const long long want = planes * (rows > 24 ? rows / 24 : 1) / 512, wave = (63 + cols) / cols, u = want > wave ? want : wave;
    return (int)(u < 64 ? u : 64);
}

bool flat_k(const Geom &g) { return (g.K == 3 || g.K == 5 || g.K == 7) && (g.s == 1 || g.s == 2); }

// Output columns per lane of the forward kernel and the filter gradient: two for 5x5 and 7x7 in bf16, whose K values a row and
// column are 16-bit LDS reads that have to be widened (28x28x256 7x7 batch 64: forward 35 -> 32 us, filter gradient 47 -> 42;
// 56x56x128 5x5 stride 2: 35 -> 30 and 42 -> 32).  In fp32 half the lanes per LDS byte cost more than the shared reads give
// (40 -> 52 us), and so they do for 3x3 in bf16 (74x74x256 forward 45 -> 58 us, filter gradient 56 -> 67).
int flat_cols(const Geom &g, int dtype) { return g.K > 3 && dtype == DT_BF16 ? 2 : 1; }

// Whether k_nchwf_conv_pairs takes the pass: rows of 36 and more in launches of some size.  Half the lanes mean bands of half the height where
// the launch is short, and narrow rows gain nothing (us, one column a lane -> pairs: 150x150x32 batch 4 7.6 -> 8.6, 18x18x728 batch 2 5.0 -> 5.5, 30x30x128
// batch 32 8.3 -> 8.6, 20x20x512 batch 256 62.0 -> 61.2; 36x36x256 batch 64 18.9 -> 18.6, 42x42x240 batch 8 8.2 -> 7.4).
bool conv_pairs(const Geom &g, int dtype, bool bwd)
{
    return dtype == DT_BF16 && g.K == 3 && g.s == 1 && g.p == 1 && g.W % 2 == 0 && !(bwd && g.m > 1) && g.W >= 36 &&
           (long long)g.N * g.O * (g.W / 2) >= 32768;
}

// Whether k_nchwf_bwd_filter_pairs does: wider rows, whose planes are bands with dy in LDS beside them or few rows (38x38x256 batch 64, whole planes
// and dy read by the lanes: 27.5 -> 32.6; 50x50x300 batch 16 20.6 -> 20.7).
bool filter_pairs(const Geom &g, int dtype) { return conv_pairs(g, dtype, false) && g.W >= 64; }

bool conv_tile(const Geom &g, int dtype, bool bwd, FlatTile *ft)
{
    const int esz = dtype == DT_F32 ? 4 : 2, nc = conv_pairs(g, dtype, bwd) ? 2 : flat_cols(g, dtype), cols = ((bwd ? g.W : g.Wo) + nc - 1) / nc;
    auto in_rows = [&](int t) { return (t - 1) * g.s + g.K; };
    if (!bwd)
        return pick_tile(esz, cols, g.Ho, g.N * g.O, most_planes((long long)g.N * g.O, g.Ho, cols), g.H, g.W, g.Ho, g.Wo, in_rows, 1, g.m, lds_target(g.K), ft, 1, LEAST_BAND);
    return pick_tile(esz, cols, g.H, g.N * g.C, most_planes((long long)g.N * g.C, g.H, cols), g.Ho, g.Wo, g.H, g.W, in_rows, g.m, 1, lds_target(g.K), ft, 1, LEAST_BAND);
}

int s2_cols(const Geom &g) { return (g.W + 1) / 2; }
int s2_pairs(const Geom &g) { return (g.H - 1 + g.p) / 2 - g.p / 2 + 1; }
bool s2_tile(const Geom &g, int dtype, FlatTile *ft)
{
    const int esz = dtype == DT_F32 ? 4 : 2, NA = (g.K + 1) / 2;
    auto in_rows = [&](int t) { return t + NA - 1; };
    return pick_tile(esz, s2_cols(g), s2_pairs(g), g.N * g.C, most_planes((long long)g.N * g.C, g.H, s2_cols(g)), g.Ho, g.Wo, g.H, g.W, in_rows, g.m, 1,
                     lds_target(g.K), ft, 1, LEAST_BAND);
}
// Whether the filter gradient reads dy from LDS too.  Every dy value is read once, by one lane, so that it needs no LDS, and without it
// more blocks fit a compute unit: 28x28x256 7x7 fp32 batch 64 54 -> 42 us, 37x37x256 multiplier 2 41 -> 32, 19x19x728 bf16 17 -> 15,
// 74x74x256 3x3 fp32 78 -> 74.  But a lane's own loads are short, and a band starts with a wait for them: planes that are
// too large for LDS together with their dy keep bands of both there for 3x3 in bf16 (74x74x256 49 us against 56) and at stride 2 (fp32 55 against 63), and for 5x5 in fp32 (41x41x240 63 against 67;
// at stride 2 56x56x128 47 against 45).
// Sets of sums per lane.  A lane's chain of n products has a relative error of about 2^-24 * sqrt(n / 6); two sets halve n.  Mean over
// random layers against 64 bits, with this rule (the kernels these replaced): 3x3 fp32 1.05e-7 (1.01e-7; one set 1.16e-7), 3x3 bf16 7.78e-8
// (7.75e-8; 7.95e-8), 5x5 fp32 1.03e-7 (0.96e-7; 1.06e-7), 5x5 bf16 7.59e-8 (7.41e-8), 7x7 fp32 1.09e-7 (1.07e-7), 7x7 bf16 8.02e-8 (7.84e-8).
// They take the time of one where LDS bounds the waves: 74x74x256 3x3 72.0 -> 72.8 us, 41x41x240 5x5 with dy in LDS 62.1 -> 62.6.  Where
// registers do, 25 more cost 21x21x240 5x5 batch 238 51 -> 62 us and 49 more 28x28x256 7x7 40 -> 52.
constexpr int filter_sets(int K, bool dylds) { return K == 3 || (K == 5 && dylds) ? 2 : 1; }
template <typename T, int K, int S> constexpr bool DY_LDS = K == 3 ? sizeof(T) == 2 || S == 2 : K == 5 && S == 1 && sizeof(T) == 4;
bool filter_tile(const Geom &g, int dtype, FlatTile *ft)
{
    const int esz = dtype == DT_F32 ? 4 : 2, nc = filter_pairs(g, dtype) ? 2 : flat_cols(g, dtype), cols = (g.Wo + nc - 1) / nc;
    auto in_rows = [&](int t) { return (t - 1) * g.s + g.K; };
    auto pick = [&](bool second) {
        return pick_tile(esz, cols, g.Ho, g.O, most_planes((long long)g.N * g.O, g.Ho, cols), g.H, g.W, g.Ho, g.Wo, in_rows, 1, g.m, lds_target(g.K), ft, g.N, LEAST_FILTER_BAND, second);
    };
    const bool lds = g.K == 3 ? dtype == DT_BF16 || g.s == 2 : g.K == 5 && g.s == 1 && dtype == DT_F32;      // DY_LDS
    return (lds && pick(true) && ft->nbands > 1) || pick(false);
}

bool fused_tile(const Geom &g, int dtype, FlatTile *ft)
{
    auto in_rows = [&](int t) { return t + 2; };
    return pick_tile(dtype == DT_F32 ? 4 : 2, g.W, g.H, g.O, most_planes((long long)g.N * g.O, g.H, g.W), g.H, g.W, g.H, g.W, in_rows, 1, 1, lds_target(3), ft,
                     g.N, LEAST_FILTER_BAND);
}
// Parts of the filter gradient: about eight blocks per compute unit in the launch, two items per block and more where the launch has more
// than four blocks per compute unit that way, and at most 8 MiB of partials.
int filter_parts(const Geom &g, const FlatTile &ft)
{
    const long long groups = (g.O + ft.U - 1) / ft.U, items = (long long)g.N * ft.nbands;
    long long parts = (2048 + groups - 1) / groups;
    if (groups * items > 1024 && parts > (items + 1) / 2) parts = (items + 1) / 2;
    if (parts > items) parts = items;
    const long long J = (long long)g.O * g.K * g.K;
    if (parts * J * 4 > (8 << 20)) parts = (8 << 20) / (J * 4);
    if (parts < 1) parts = 1;
    const long long per = (items + parts - 1) / parts;
    return (int)((items + per - 1) / per);
}

}  // namespace

bool nchwf_fwd_supported(const Geom &g, int dtype)
{
    FlatTile ft;
    return flat_k(g) && conv_tile(g, dtype, false, &ft) && launchable((long long)cdiv(g.N * g.O, ft.U) * ft.nbands, ft.threads);
}
bool nchwf_bwd_data_supported(const Geom &g, int dtype)
{
    FlatTile ft;
    if (!flat_k(g) || g.m > 2) return false;
    return (g.s == 1 ? conv_tile(g, dtype, true, &ft) : s2_tile(g, dtype, &ft)) && launchable((long long)cdiv(g.N * g.C, ft.U) * ft.nbands, ft.threads);
}

int nchwf_bwd_filter_parts(const Geom &g, int dtype)
{
    FlatTile ft;
    if (!flat_k(g) || !filter_tile(g, dtype, &ft)) return 0;
    return filter_parts(g, ft);
}

// Where both passes run on column pairs (bf16, an even width from 64 on) and the fused walk, which widens every value, is the longer way: large layers of
// few rows, whose halo rows it reads twice, unless a row about fills its block of 256 lanes (193 to 256); and rows of just under half a
// block, whose tall planes leave room for few of those blocks.  Fused / two passes, buffers in turn, 59 000 random layers: 4 million outputs and more, rows
// of 128 to 192: 1.05 to 1.26 at 4 to 8 rows, 0.88 to 1.17 at 8 to 24, 0.83 to 1.02 beyond; of 258 to 512: 1.06 to 1.33, 0.97 to 1.32, 0.77 to
// 1.04; of 193 to 256: 0.77 to 1.01; of 64 to 94: 0.79 to 1.07; of 98 to 126: 0.85 to 1.09, from 110 rows on 0.95 to 1.44.  Fewer outputs: 0.70 to
// 1.0.  By this rule 4.7 % of the layers on pairs stay fused and are longer by more than a twentieth (always fused 15.7 %, up to 1.7 times), 2.0 % run in two
// passes and are.
static bool two_passes_shorter(const Geom &g, int dtype)
{
    if (!filter_pairs(g, dtype) || !conv_pairs(g, dtype, true) || (long long)g.N * g.O * g.H * g.W < 1 << 22) return false;
    return (g.H < 24 && g.W >= 128 && (g.W <= 192 || g.W > 256)) || (g.H >= 110 && g.W > 96 && g.W < 128);
}

int nchwf_bwd_fused_parts(const Geom &g, int dtype)
{
    FlatTile ft;
    if (!(g.K == 3 && g.s == 1 && g.p == 1 && g.m == 1) || two_passes_shorter(g, dtype) || !fused_tile(g, dtype, &ft)) return 0;
    return filter_parts(g, ft);
}
void nchwf_bwd_fused_tiles(const Geom &g, int dtype, int parts, FilterGradSrc *f)
{
    FlatTile ft;
    fused_tile(g, dtype, &ft);
    f->TN = 1; f->TA = ft.TR; f->TB = g.Wo;
    f->tn = g.N; f->ta = ft.nbands; f->tb = 1;
    f->per = cdiv(g.N * ft.nbands, parts); f->nparts = parts;
}

void nchwf_bwd_filter_tiles(const Geom &g, int dtype, int parts, FilterGradSrc *f)
{
    FlatTile ft;
    filter_tile(g, dtype, &ft);
    f->TN = 1; f->TA = ft.TR; f->TB = g.Wo;
    f->tn = g.N; f->ta = ft.nbands; f->tb = 1;
    f->per = cdiv(g.N * ft.nbands, parts); f->nparts = parts;
}

template <typename T, int K, int S, int M>
static hipError_t conv_go(const Geom &g, int dtype, const void *in, const void *w, void *out, bool bwd, hipStream_t st)
{
    FlatTile ft;
    if (!conv_tile(g, dtype, bwd, &ft)) return hipErrorInvalidValue;
    const int Hi = bwd ? g.Ho : g.H, Wi = bwd ? g.Wo : g.W, Ho = bwd ? g.H : g.Ho, Wo = bwd ? g.W : g.Wo;
    const int OC = bwd ? g.C : g.O, nplanes = g.N * OC;
    const unsigned nblocks = (unsigned)cdiv(nplanes, ft.U) * ft.nbands;
    const int total_in = g.N * (bwd ? g.O : g.C) * Hi * Wi;
    if constexpr (sizeof(T) == 2 && K == 3 && S == 1 && M == 1) {
        if (conv_pairs(g, dtype, bwd)) {
            hipLaunchKernelGGL(k_nchwf_conv_pairs, dim3(nblocks), dim3(ft.threads), tile_lds(ft, sizeof(T)), st, (const T *)in, (const T *)w, (T *)out, nplanes,
                               OC, g.H, g.W, bwd ? 1 : g.m, total_in, bwd ? 1 : 0, ft, nblocks, g);
            return hipGetLastError();
        }
    }
    const bool same = (bwd ? K - 1 - g.p : g.p) == K / 2;
    constexpr int NC = K > 3 && sizeof(T) == 2 ? 2 : 1;
    auto kernel = same ? k_nchwf_conv<T, K, S, M, true, NC> : k_nchwf_conv<T, K, S, M, false, NC>;
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(ft.threads), tile_lds(ft, sizeof(T)), st, (const T *)in, (const T *)w,
                        (T *)out, nplanes, OC, Hi, Wi, Ho, Wo, bwd ? K - 1 - g.p : g.p, bwd ? 1 : g.m, total_in,
                       bwd ? 1 : 0, ft, nblocks, g);
    return hipGetLastError();
}
template <typename T, int K, int M>
static hipError_t s2_go(const Geom &g, int dtype, const void *dy, const void *w, void *dx, hipStream_t st)
{
    FlatTile ft;
    if (!s2_tile(g, dtype, &ft)) return hipErrorInvalidValue;
    const int nplanes = g.N * g.C;
    const unsigned nblocks = (unsigned)cdiv(nplanes, ft.U) * ft.nbands;
    auto kernel = g.p % 2 ? k_nchwf_bwd_data_s2<T, K, M, 1> : k_nchwf_bwd_data_s2<T, K, M, 0>;
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(ft.threads), tile_lds(ft, sizeof(T)), st, (const T *)dy,
                       (const T *)w, (T *)dx, nplanes, g.C, g.H, g.W, g.Ho, g.Wo, g.p, s2_cols(g), g.N * g.O * g.Ho * g.Wo, ft,
                       nblocks, g);
    return hipGetLastError();
}
template <typename T, int K, int S>
static hipError_t filter_go(const Geom &g, int dtype, const void *x, const void *dy, float *ws, int parts, hipStream_t st)
{
    FlatTile ft;
    if (!filter_tile(g, dtype, &ft)) return hipErrorInvalidValue;
    const int items = g.N * ft.nbands, per = cdiv(items, parts);
    const unsigned nblocks = (unsigned)cdiv(g.O, ft.U) * parts;
    size_t lds = tile_lds(ft, sizeof(T)) + (ft.pout ? (size_t)second_area(ft) * sizeof(T) : 0);
    const size_t red = (size_t)(K * K <= 25 ? K * K : 25) * ft.threads * 4;
    if (red > lds) lds = red;
    if constexpr (sizeof(T) == 2 && K == 3 && S == 1) {
        if (filter_pairs(g, dtype)) {
            auto pairs = ft.pout ? k_nchwf_bwd_filter_pairs<true> : k_nchwf_bwd_filter_pairs<false>;
            hipLaunchKernelGGL(pairs, dim3(nblocks), dim3(ft.threads), lds, st, g, (const T *)x, (const T *)dy, ws, parts, per, ft, nblocks);
            return hipGetLastError();
        }
    }
    constexpr int NC = K > 3 && sizeof(T) == 2 ? 2 : 1;
    constexpr int SETS = filter_sets(K, false), SETS_LDS = filter_sets(K, true);
    auto kernel = g.p == K / 2 ? k_nchwf_bwd_filter<T, K, S, true, NC, false, SETS> : k_nchwf_bwd_filter<T, K, S, false, NC, false, SETS>;
    if constexpr (DY_LDS<T, K, S>) {
        if (ft.pout) kernel = g.p == K / 2 ? k_nchwf_bwd_filter<T, K, S, true, NC, true, SETS_LDS> : k_nchwf_bwd_filter<T, K, S, false, NC, true, SETS_LDS>;
    }
    hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(ft.threads), lds, st, g, (const T *)x, (const T *)dy, ws, parts,
                       per, ft, nblocks);
    return hipGetLastError();
}

template <typename T>
static hipError_t fused_go(const Geom &g, int dtype, const void *x, const void *dy, const void *w, void *dx, float *ws, int parts, hipStream_t st)
{
    FlatTile ft;
    if (!fused_tile(g, dtype, &ft)) return hipErrorInvalidValue;
    const int items = g.N * ft.nbands, per = cdiv(items, parts);
    const unsigned nblocks = (unsigned)cdiv(g.O, ft.U) * parts;
    size_t lds = tile_lds(ft, sizeof(T));
    const size_t red = (size_t)9 * ft.threads * 4;
    if (red > lds) lds = red;
    hipLaunchKernelGGL(k_nchwf_bwd_fused<T>, dim3(nblocks), dim3(ft.threads), lds, st, g, (const T *)x, (const T *)dy, (const T *)w, (T *)dx, ws, parts,
                       per, ft, nblocks);
    return hipGetLastError();
}
hipError_t nchwf_bwd_fused(const Geom &g, int dtype, const void *x, const void *dy, const void *w, void *dx, float *ws, int parts, hipStream_t st)
{
    return dtype == DT_F32 ? fused_go<float>(g, dtype, x, dy, w, dx, ws, parts, st) : fused_go<bf16_t>(g, dtype, x, dy, w, dx, ws, parts, st);
}

#define BY_K(F, ...) (g.K == 3 ? F<T, 3, __VA_ARGS__> : g.K == 5 ? F<T, 5, __VA_ARGS__> : F<T, 7, __VA_ARGS__>)
template <typename T>
static hipError_t fwd_t(const Geom &g, int dtype, const void *x, const void *w, void *y, hipStream_t st)
{
    return (g.s == 1 ? BY_K(conv_go, 1, 1) : BY_K(conv_go, 2, 1))(g, dtype, x, w, y, false, st);
}
template <typename T>
static hipError_t bwd_data_t(const Geom &g, int dtype, const void *dy, const void *w, void *dx, hipStream_t st)
{
    if (g.s == 1) return (g.m == 1 ? BY_K(conv_go, 1, 1) : BY_K(conv_go, 1, 2))(g, dtype, dy, w, dx, true, st);
    return (g.m == 1 ? BY_K(s2_go, 1) : BY_K(s2_go, 2))(g, dtype, dy, w, dx, st);
}
template <typename T>
static hipError_t bwd_filter_t(const Geom &g, int dtype, const void *x, const void *dy, float *ws, int parts, hipStream_t st)
{
    return (g.s == 1 ? BY_K(filter_go, 1) : BY_K(filter_go, 2))(g, dtype, x, dy, ws, parts, st);
}
#undef BY_K

hipError_t nchwf_fwd(const Geom &g, int dtype, const void *x, const void *w, void *y, hipStream_t st)
{
    return dtype == DT_F32 ? fwd_t<float>(g, dtype, x, w, y, st) : fwd_t<bf16_t>(g, dtype, x, w, y, st);
}
hipError_t nchwf_bwd_data(const Geom &g, int dtype, const void *dy, const void *w, void *dx, hipStream_t st)
{
    return dtype == DT_F32 ? bwd_data_t<float>(g, dtype, dy, w, dx, st) : bwd_data_t<bf16_t>(g, dtype, dy, w, dx, st);
}
hipError_t nchwf_bwd_filter(const Geom &g, int dtype, const void *x, const void *dy, float *ws, int parts, hipStream_t st)
{
    return dtype == DT_F32 ? bwd_filter_t<float>(g, dtype, x, dy, ws, parts, st) : bwd_filter_t<bf16_t>(g, dtype, x, dy, ws, parts, st);
}

}  // namespace dwc

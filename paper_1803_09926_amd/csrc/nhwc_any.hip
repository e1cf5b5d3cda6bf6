// NHWC row walks for what nhwc.hip does not take: 5x5 at stride 2, 7x7, channel counts that are no multiple of four, other
// paddings and other multipliers (3x3, 5x5 and 7x7; stride 1 and 2).
//
// The mapping is that of nhwc.hip: a lane owns V consecutive channels of one column and walks down the rows of a strip, lanes
// flat over the channels x columns of a row.  Every row of the input is read once per strip and tap column through a buffer view
// of the image (a column outside reads as the zero of the padding; the row offset is scalar), one step ahead of its use, and
// meets ceil(K/S) rotating accumulators; what depends on the row is uniform.  V = 2 for 5x5 and 7x7: K*K*V filter registers (or
// sums) are what limits the wavefronts in flight; V = 4 for 3x3; 1 where the channel count is odd, the multiplier is not 1 or the lanes are few.
//
// One output per thread -> these kernels, us on one MI355X at batch 64, forward / input gradient / filter gradient: 56x56x128 5x5
// stride 2 fp32 142 / 347 / 900 -> 36 / 37 / 41 (bound by its K vector loads per row and column, 8 bytes a lane); 28x28x256 7x7 fp32
// 660 / 890 / 2430 -> 58 / 58 / 65; 56x56x30 3x3 fp32 49 / 67 / 954 -> 12.5 / 12.5 / 18.
#include "bounds.hpp"
#include "point.hpp"
#include <type_traits>

namespace dwc {

namespace {

struct AnyGeom {
    int N, Ci, Co, Hi, Wi, Ho, Wo;   // of the tensor read and the tensor written
    int pad, mdiv;                   // input row oh*S - pad + kh; input channel = output channel / mdiv (forward, V = 1)
    int TH, nstrips, nchunks;        // rows per strip (bwd_data_s2: row pairs)
    int TW, ncols;                   // filter gradient: columns of an item, items across a row
};

template <typename T, int V> __device__ __forceinline__ void load_filter_vec(const T *w, float (&r)[V])
{
    if constexpr (V == 1) r[0] = ldf(w);
    else Vec<T, V>::load(w, r);
}

// ---------------------------------------------------------------------------------------------
// out[oh][ow][c] = sum over kh, kw, q < M of w[kh][kw][c*M + q] * in[oh*S - pad + kh][ow*S - pad + kw][c*M + q] (M = 1: of channel
// c / mdiv).  Forward: M = 1; input gradient of a stride-1 layer: filters rotated, pad = K - 1 - p, M = the multiplier.
// ---------------------------------------------------------------------------------------------
template <typename T, int V, int K, int S, int M>
__global__ __launch_bounds__(256) void k_nhwca_conv(AnyGeom g, const T *__restrict__ in, const T *__restrict__ w, T *__restrict__ out, int OW,
                                                    int flip, unsigned nblocks, int nt, Geom q)
{
    constexpr int NA = (K + S - 1) / S, VI = V * M;
    unsigned b = xcd_remap(blockIdx.x, nblocks);
    const int chunk = b % g.nchunks; b /= g.nchunks;
    const int strip = b % g.nstrips, n = b / g.nstrips;
    const int Q = g.Co / V, l = chunk * (int)blockDim.x + (int)threadIdx.x;
    if (l >= g.Wo * Q) return;                               // the kernel has no barrier
    const int ow = l / Q, c = (l - ow * Q) * V;
    const uint32_t esz = sizeof(T);
    const BufView view(in + (size_t)n * g.Hi * g.Wi * g.Ci, (uint32_t)g.Hi * g.Wi * g.Ci * esz);
    const uint32_t rowbytes = (uint32_t)g.Wi * g.Ci * esz;
    const int ci = M > 1 ? c * M : c / g.mdiv;
    uint32_t off[K];
#pragma unroll
    for (int kw = 0; kw < K; ++kw) {
        const int iw = ow * S - g.pad + kw;
        off[kw] = (unsigned)iw < (unsigned)g.Wi ? (uint32_t)(iw * g.Ci + ci) * esz : BufView::OUTSIDE;
    }
    float wr[K][K][VI];                                      // OW: filter entries of a tap (the layer's output channels)
#pragma unroll
    for (int kh = 0; kh < K; ++kh)
#pragma unroll
        for (int kw = 0; kw < K; ++kw) {
            const int tap = kh * K + kw;
            load_filter_vec<T, VI>(w + (size_t)(flip ? K * K - 1 - tap : tap) * OW + c * M, wr[kh][kw]);
        }
    const int oh0 = strip * g.TH, oh1 = min(g.Ho, oh0 + g.TH), TRb = oh1 - oh0, steps = TRb + NA - 1;
    T *po = out + (((size_t)n * g.Ho + oh0) * g.Wo + ow) * g.Co + c;
    const size_t ostep = (size_t)g.Wo * g.Co;
    float acc[NA][V];
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) acc[i][v] = 0.f;

    // step t reads input rows (oh0 + t)*S - pad + j; they meet the outputs of rows oh0 + t - i, the one with i = NA - 1 is complete
    auto fetch = [&](int t, RawVec<T, VI> (&r)[S][K]) {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int row = min(max((oh0 + t) * S - g.pad + j, 0), g.Hi - 1);
#pragma unroll
            for (int kw = 0; kw < K; ++kw) r[j][kw].load_buf(view, off[kw], (uint32_t)row * rowbytes);
        }
    };
    auto step = [&](int t, const RawVec<T, VI> (&r)[S][K]) {
        const bool inner = K == 3 || (t >= NA - 1 && t < TRb);
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int row = (oh0 + t) * S - g.pad + j;
            if ((unsigned)row >= (unsigned)g.Hi) continue;   // padding; uniform
            float v[K][VI];
#pragma unroll
            for (int kw = 0; kw < K; ++kw) r[j][kw].get(v[kw]);
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                if (j + i * S >= K || !(inner || (unsigned)(t - i) < (unsigned)TRb)) continue;      // a row of the next strip
#pragma unroll
                for (int kw = 0; kw < K; ++kw)
#pragma unroll
                    for (int u = 0; u < VI; ++u) acc[i][u / M] = fmaf(wr[j + i * S][kw][u], v[kw][u], acc[i][u / M]);
            }
        }
        if (t >= NA - 1) { store_vec<T, V>(po, acc[NA - 1], nt != 0); po += ostep; }
#pragma unroll
        for (int i = NA - 1; i > 0; --i)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[i][v] = acc[i - 1][v];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[0][v] = 0.f;
    };
    NonFinite bad;
#pragma unroll
    for (int e = 0; e < K * K * VI; ++e) bad.add(wr[e / VI / K][e / VI % K][e % VI]);
    const bool redo = bad.any();
    RawVec<T, VI> ra[S][K], rb[S][K];
    fetch(0, ra);
    int t = 0;
#pragma unroll 1
    for (; t + 2 <= steps; t += 2) {
        fetch(t + 1, rb);
        step(t, ra);
        fetch(t + 2, ra);
        step(t + 1, rb);
    }
    if (t < steps) step(t, ra);

    if (__builtin_expect(redo, 0)) {                    // the lane's outputs again, without the padding
#pragma unroll 1
        for (int i = 0; i < TRb * V; ++i) {
            const int row = oh0 + i / V, ch = c + i % V;
            stf(out + (((size_t)n * g.Ho + row) * g.Wo + ow) * g.Co + ch,
                flip ? point_bwd_data<T, LAYOUT_NHWC>(q, in, w, n, ch, row, ow) : point_fwd<T, LAYOUT_NHWC>(q, in, w, n, ch, row, ow));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Input gradient of a stride-2 layer: with h + p = 2a + f and w + p = 2b + e the taps kh = 2k + f, kw = 2l + e read
// dy[a - k][b - l]; a lane owns the two dx columns of one b and walks down the dy rows.
// ---------------------------------------------------------------------------------------------
template <typename T, int V, int K, int M>
__global__ __launch_bounds__(256) void k_nhwca_bwd_data_s2(AnyGeom g, const T *__restrict__ dy, const T *__restrict__ w, T *__restrict__ dx, int NB,
                                                           unsigned nblocks, int nt, Geom q)
{
    constexpr int NA = (K + 1) / 2, VI = V * M;
    unsigned bid = xcd_remap(blockIdx.x, nblocks);
    const int chunk = bid % g.nchunks; bid /= g.nchunks;
    const int strip = bid % g.nstrips, n = bid / g.nstrips;
    const int Q = g.Co / V, l0 = chunk * (int)blockDim.x + (int)threadIdx.x;
    if (l0 >= NB * Q) return;
    const int bi = l0 / Q, c = (l0 - bi * Q) * V, b = g.pad / 2 + bi;
    const uint32_t esz = sizeof(T);
    const BufView view(dy + (size_t)n * g.Hi * g.Wi * g.Ci, (uint32_t)g.Hi * g.Wi * g.Ci * esz);
    const uint32_t rowbytes = (uint32_t)g.Wi * g.Ci * esz;
    uint32_t off[NA];
#pragma unroll
    for (int l = 0; l < NA; ++l) off[l] = (unsigned)(b - l) < (unsigned)g.Wi ? (uint32_t)((b - l) * g.Ci + c * M) * esz : BufView::OUTSIDE;
    float wr[K][K][VI];
#pragma unroll
    for (int kh = 0; kh < K; ++kh)
#pragma unroll
        for (int kw = 0; kw < K; ++kw) load_filter_vec<T, VI>(w + (size_t)(kh * K + kw) * g.Ci + c * M, wr[kh][kw]);
    const int a0 = g.pad / 2 + strip * g.TH, a1 = min((g.Ho - 1 + g.pad) / 2 + 1, a0 + g.TH);
    const int col = 2 * b - g.pad;
    const bool st0 = col >= 0 && col < g.Wo, st1 = col + 1 < g.Wo;
    float acc[NA][2][2][V];
#pragma unroll
    for (int k = 0; k < NA; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[k][i >> 1][i & 1][v] = 0.f;
    auto fetch = [&](int r, RawVec<T, VI> (&q)[NA]) {
        const int row = min(max(r, 0), g.Hi - 1);
#pragma unroll
        for (int l = 0; l < NA; ++l) q[l].load_buf(view, off[l], (uint32_t)row * rowbytes);
    };
    // dy row r reaches the row pairs r .. r + NA - 1; pair r is complete after it
    auto step = [&](int r, const RawVec<T, VI> (&q)[NA]) {
        if ((unsigned)r < (unsigned)g.Hi) {                  // uniform
            float x[NA][VI];
#pragma unroll
            for (int l = 0; l < NA; ++l) q[l].get(x[l]);
#pragma unroll
            for (int k = 0; k < NA; ++k)
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int l = 0; l < NA; ++l)
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            if (2 * k + f >= K || 2 * l + e >= K) continue;
#pragma unroll
                            for (int u = 0; u < VI; ++u)
                                acc[k][f][e][u / M] = fmaf(wr[2 * k + f][2 * l + e][u], x[l][u], acc[k][f][e][u / M]);
                        }
        }
        if (r >= a0) {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int h = 2 * r - g.pad + f;
                if ((unsigned)h < (unsigned)g.Ho) {          // uniform
                    T *p = dx + (((size_t)n * g.Ho + h) * g.Wo + col) * g.Co + c;
                    if (st0) store_vec<T, V>(p, acc[0][f][0], nt != 0);
                    if (st1) store_vec<T, V>(p + g.Co, acc[0][f][1], nt != 0);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < V; ++v) acc[k][i >> 1][i & 1][v] = k + 1 < NA ? acc[k + 1][i >> 1][i & 1][v] : 0.f;
    };
    NonFinite bad;
#pragma unroll
    for (int e = 0; e < K * K * VI; ++e) bad.add(wr[e / VI / K][e / VI % K][e % VI]);
    const bool redo = bad.any();
    RawVec<T, VI> ra[NA], rb[NA];
    int r = a0 - (NA - 1);
    fetch(r, ra);
#pragma unroll 1
    for (; r + 2 <= a1; r += 2) {
        fetch(r + 1, rb);
        step(r, ra);
        fetch(r + 2, ra);
        step(r + 1, rb);
    }
    if (r < a1) step(r, ra);

    if (__builtin_expect(redo, 0)) {                    // the lane's outputs again, without the padding
#pragma unroll 1
        for (int i = 0; i < (a1 - a0) * 4 * V; ++i) {
            const int h = 2 * a0 - g.pad + i / (2 * V), cw = col + i / V % 2, ch = c + i % V;
            if ((unsigned)h < (unsigned)g.Ho && (unsigned)cw < (unsigned)g.Wo)
                stf(dx + (((size_t)n * g.Ho + h) * g.Wo + cw) * g.Co + ch, point_bwd_data<T, LAYOUT_NHWC>(q, dy, w, n, ch, h, cw));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Filter gradient, stage 1.  A block: CT channel vectors x 256/CT columns; it takes (image, strip, part of a row) items and, in each, every
// column tile, so that it writes one partial for all of them.  A lane keeps K*K*V sums against a window of the last
// ceil(K/S) dy rows.
// ---------------------------------------------------------------------------------------------
template <typename T, int V, int K, int S>
__global__ __launch_bounds__(256) void k_nhwca_bwd_filter(AnyGeom g, const T *__restrict__ x, const T *__restrict__ dy, float *__restrict__ ws,
                                                          int CT, int parts, int per_part, unsigned nblocks)
{
    __shared__ float red[ReduceLds<K, V>::FLOATS];
    constexpr int NA = (K + S - 1) / S;
    const unsigned lb = xcd_remap(blockIdx.x, nblocks);
    const int part = (int)(lb % (unsigned)parts), ct = (int)(lb / (unsigned)parts);
    const int tx = (int)threadIdx.x % CT, ty = (int)threadIdx.x / CT, nty = 256 / CT;
    const int Q = g.Co / V, cq = ct * CT + tx, c = min(cq, Q - 1) * V, ci = c / g.mdiv;
    const uint32_t esz = sizeof(T), xrow = (uint32_t)g.Wi * g.Ci * esz, drow = (uint32_t)g.Wo * g.Co * esz;
    float acc[K][K][V];
#pragma unroll
    for (int kh = 0; kh < K; ++kh)
#pragma unroll
        for (int kw = 0; kw < K; ++kw)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[kh][kw][v] = 0.f;

    const int it1 = part_end(g.N * g.nstrips * g.ncols, per_part, part);
    for (int it = part * per_part; it < it1; ++it) {
        const int row = it / g.ncols, col0 = (it - row * g.ncols) * g.TW, col1 = min(g.Wo, col0 + g.TW);
        const int n = row / g.nstrips, strip = row - n * g.nstrips;
        const int oh0 = strip * g.TH, oh1 = min(g.Ho, oh0 + g.TH), rows = oh1 - oh0, steps = rows + NA - 1;
        const BufView vx(x + (size_t)n * g.Hi * g.Wi * g.Ci, (uint32_t)g.Hi * g.Wi * g.Ci * esz);
        const BufView vd(dy + (size_t)n * g.Ho * g.Wo * g.Co, (uint32_t)g.Ho * g.Wo * g.Co * esz);
        for (int ow0 = col0; ow0 < col1; ow0 += nty) {
            const int ow = ow0 + ty;
            const bool live = ow < col1 && cq < Q;           // the other lanes read zeros
            const uint32_t offd = live ? (uint32_t)(ow * g.Co + c) * esz : BufView::OUTSIDE;
            uint32_t off[K];
#pragma unroll
            for (int kw = 0; kw < K; ++kw) {
                const int iw = ow * S - g.pad + kw;
                off[kw] = live && (unsigned)iw < (unsigned)g.Wi ? (uint32_t)(iw * g.Ci + ci) * esz : BufView::OUTSIDE;
            }
            float d[NA][V];
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int v = 0; v < V; ++v) d[i][v] = 0.f;
            auto fetch = [&](int t, RawVec<T, V> (&r)[S][K], RawVec<T, V> &e) {
                e.load_buf(vd, offd, (uint32_t)(oh0 + min(t, rows - 1)) * drow);
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    const int row = min(max((oh0 + t) * S - g.pad + j, 0), g.Hi - 1);
#pragma unroll
                    for (int kw = 0; kw < K; ++kw) r[j][kw].load_buf(vx, off[kw], (uint32_t)row * xrow);
                }
            };
            // step t: x rows (oh0 + t)*S - pad + j against dy rows oh0 + t - i
            auto step = [&](int t, const RawVec<T, V> (&r)[S][K], const RawVec<T, V> &e) {
                e.get(d[0]);
                if (t >= rows) {
#pragma unroll
                    for (int v = 0; v < V; ++v) d[0][v] = 0.f;
                }
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    const int row = (oh0 + t) * S - g.pad + j;
                    if ((unsigned)row >= (unsigned)g.Hi) continue;
#pragma unroll
                    for (int kw = 0; kw < K; ++kw) {
                        float xv[V];
                        r[j][kw].get(xv);
#pragma unroll
                        for (int i = 0; i < NA; ++i) {
                            if (j + i * S >= K) continue;
#pragma unroll
                            for (int v = 0; v < V; ++v) acc[j + i * S][kw][v] = fmaf(d[i][v], xv[v], acc[j + i * S][kw][v]);
                        }
                    }
                }
#pragma unroll
                for (int i = NA - 1; i > 0; --i)
#pragma unroll
                    for (int v = 0; v < V; ++v) d[i][v] = d[i - 1][v];
            };
            RawVec<T, V> ra[S][K], rb[S][K], da, db;
            fetch(0, ra, da);
            int t = 0;
#pragma unroll 1
            for (; t + 2 <= steps; t += 2) {
                fetch(t + 1, rb, db);
                step(t, ra, da);
                fetch(t + 2, ra, da);
                step(t + 1, rb, db);
            }
            if (t < steps) step(t, ra, da);
        }
    }
    float *wsp = ws + (size_t)part * (K * K * g.Co);
    block_reduce_taps<K, V>(acc, CT, red, [&](int kh, int kw, int v, float total) {
        if (cq < Q) wsp[(kh * K + kw) * g.Co + cq * V + v] = total;
    });
}

// ---- host side --------------------------------------------------------------------------------

int cdiva(int a, int b) { return (a + b - 1) / b; }

bool any_k(const Geom &g)
{
    return (g.K == 3 || g.K == 5 || g.K == 7) && (g.s == 1 || g.s == 2) && (long long)g.H * g.W * g.C * 4 <= (1LL << 31) &&
           (long long)g.Ho * g.Wo * g.O * 4 <= (1LL << 31);
}

// Channels per lane.  5x5 and 7x7 in launches of few lanes take one channel: the walk is then as long as its loads take, and twice the wavefronts with half the
// registers hide more of them (50 000 random layers, share of the time with two: fp32 5x5 0.80 to 0.97, filter gradient 0.80 to 0.90 below 1.2 M outputs and up to 1.7 above
// (119x119x84 at stride 2, 1.5 M), 7x7 0.75 to 0.92 up to 1.4 M, from there on 0.92 with one in seven longer by more than 8 %, but for the filter gradient, 0.83 up to
// 1.6 M; bf16, whose lanes then read two bytes, filter gradient below 0.4 M 0.75 to 0.93, the other passes below 0.16 M 0.84 to 0.98, above up to 1.25).
int any_vec(const Geom &g, int dtype, int pass)
{
    if (g.m != 1) return 1;
    if (g.C % 4 == 0 && g.K == 3) return 4;
    if (g.C % 2) return 1;
    if (g.K == 3) return 2;
    if (const char *e = tune_env("DWCONV_TUNE_ANY_V")) return atoi(e) == 1 ? 1 : 2;
    const long long outputs = (long long)g.N * g.O * g.Ho * g.Wo;
    const long long few = dtype == DT_F32 ? (pass < 2 ? 1400000 : g.K == 5 ? 1200000 : 1600000) : pass == 2 ? 400000 : 160000;
    return outputs < few ? 1 : 2;
}

// balanced strips of about `target` rows, shorter while the launch has fewer than 1024 wavefronts, down to four rows; to two below 256 (0.87 to 0.9 of
// the time; above, the rows that strips share make it longer: 5x5 of 0.2 M outputs 1.2 to 1.4)
int any_strips(int rows, int target, long long lanes)
{
    while (target > 4 && lanes * cdiva(rows, target) < 65536) target = (target + 1) / 2;
    while (target > 2 && lanes * cdiva(rows, target) < 16384) target = (target + 1) / 2;
    const int n = cdiva(rows, target);
    return cdiva(rows, n);
}

// Block size of the walks without a reduction: the one that leaves the fewest lanes of a row's last block idle (a row of 7 columns x 2
// channels is 14 lanes), the largest of equals.
int any_block(long long lanes)
{
    int best = 256;
    for (int b = 192; b >= 64; b -= 64)
        if ((lanes + b - 1) / b * b < (lanes + best - 1) / best * best) best = b;
    return best;
}

int s2a_cols(const Geom &g) { return (g.W - 1 + g.p) / 2 - g.p / 2 + 1; }
int s2a_pairs(const Geom &g) { return (g.H - 1 + g.p) / 2 - g.p / 2 + 1; }

// Launch of a walk without a reduction over `rows` rows of `lanes` lanes of N images.
struct WalkTile { int TH, nstrips, bs, nchunks; long long blocks; };
WalkTile walk_tile(int N, int rows, long long lanes, int target)
{
    WalkTile t;
    t.TH = any_strips(rows, target, lanes * N);
    t.nstrips = cdiva(rows, t.TH);
    t.bs = any_block(lanes);
    t.nchunks = (int)((lanes + t.bs - 1) / t.bs);
    t.blocks = (long long)N * t.nstrips * t.nchunks;
    return t;
}
WalkTile walk_tile(const Geom &g, int dtype, int pass)
{
    const int V = any_vec(g, dtype, pass), target = g.K == 3 ? 14 : 28;
    if (pass == 0) return walk_tile(g.N, g.Ho, (long long)g.Wo * (g.O / V), target);
    if (g.s == 1) return walk_tile(g.N, g.H, (long long)g.W * (g.C / V), target);
    return walk_tile(g.N, s2a_pairs(g), (long long)s2a_cols(g) * (g.C / V), 14);
}

struct FilterTile { int V, CT, nct, TH, nstrips, TW, ncols, parts, per; };
bool filter_tile_any(const Geom &g, int dtype, FilterTile *f)
{
    f->V = any_vec(g, dtype, 2);
    const int Q = g.O / f->V;
    // channel vectors across a block: the widest power of two that leaves few lanes idle, across the channels and across the columns that
    // the other lanes take (181x3x3x572 7x7 fp32: two across, as the channels alone would have it, 265 us with 3 of 128 columns there)
    int best = 0;
    double beste = 0.0;
    for (int ct = 64; ct >= 1; ct /= 2) {
        const int nty = 256 / ct;
        const double e = (double)Q / (cdiva(Q, ct) * ct) * ((double)g.Wo / ((double)cdiva(g.Wo, nty) * nty));
        if (e > beste * 1.1) { beste = e; best = ct; }
    }
    f->CT = best; f->nct = cdiva(Q, best);
    // about 768 blocks; strips only where there are not enough images, parts of a row only where the strips are fewer than the compute units:
    // each part is a partial more (56x56x128 5x5 stride 2 batch 64, 256 strips: fp32 32 us with 256 partials, 36 with 512)
    const int want = 768, nty = 256 / best;
    int TH = g.Ho;
    while (TH > 7 && (long long)g.N * cdiva(g.Ho, TH) * f->nct < want) TH = (TH + 1) / 2;
    f->TH = cdiva(g.Ho, cdiva(g.Ho, TH));
    f->nstrips = cdiva(g.Ho, f->TH);
    const long long rows = (long long)g.N * f->nstrips;
    int tiles = cdiva(g.Wo, nty);
    while (tiles > 1 && rows * cdiva(cdiva(g.Wo, nty), tiles) * f->nct < 256) tiles = (tiles + 1) / 2;
    f->TW = tiles * nty;
    f->ncols = cdiva(g.Wo, f->TW);
    const long long items = rows * f->ncols, J = (long long)g.O * g.K * g.K;
    long long parts = cdiva(want, f->nct);
    if (parts > items) parts = items;
    if (parts * J * 4 > (8 << 20)) parts = (8 << 20) / (J * 4);
    if (parts < 1) parts = 1;
    f->per = (int)((items + parts - 1) / parts);
    f->parts = (int)((items + f->per - 1) / f->per);
    return true;
}

}  // namespace

bool nhwca_supported(const Geom &g, int dtype, int pass)
{
    if (!any_k(g)) return false;
    if (pass == 2) return true;
    const WalkTile t = walk_tile(g, dtype, pass);
    return launchable(t.blocks, t.bs) && (pass != 1 || g.m <= 2);
}

int nhwca_row_lanes(const Geom &g, int dtype) { return g.Wo * (g.O / any_vec(g, dtype, 0)); }

int nhwca_bwd_filter_parts(const Geom &g, int dtype)
{
    FilterTile f;
    return any_k(g) && filter_tile_any(g, dtype, &f) ? f.parts : 0;
}

void nhwca_bwd_filter_tiles(const Geom &g, int dtype, FilterGradSrc *f)
{
    FilterTile t;
    filter_tile_any(g, dtype, &t);
    f->TN = 1; f->TA = t.TH; f->TB = t.TW;
    f->tn = g.N; f->ta = t.nstrips; f->tb = t.ncols;
    f->per = t.per; f->nparts = t.parts;
}

template <typename T, int V, int K, int S, int M>
static hipError_t conv_any(const Geom &q, const void *in, const void *w, void *out, bool bwd, hipStream_t st)
{
    AnyGeom g = bwd ? AnyGeom{q.N, q.O, q.C, q.Ho, q.Wo, q.H, q.W, K - 1 - q.p, 1, 0, 0, 0, 0, 0}
                    : AnyGeom{q.N, q.C, q.O, q.H, q.W, q.Ho, q.Wo, q.p, q.m, 0, 0, 0, 0, 0};
    const WalkTile t = walk_tile(q, sizeof(T) == 4 ? DT_F32 : DT_BF16, bwd ? 1 : 0);
    g.TH = t.TH; g.nstrips = t.nstrips; g.nchunks = t.nchunks;
    const unsigned nblocks = (unsigned)t.blocks;
    hipLaunchKernelGGL((k_nhwca_conv<T, V, K, S, M>), dim3(nblocks), dim3(t.bs), 0, st, g, (const T *)in, (const T *)w, (T *)out, q.O, bwd ? 1 : 0,
                       nblocks, stream_stores("NHWCA", 0, 0), q);
    return hipGetLastError();
}
template <typename T, int V, int K, int M>
static hipError_t s2_any(const Geom &q, const void *dy, const void *w, void *dx, hipStream_t st)
{
    AnyGeom g = {q.N, q.O, q.C, q.Ho, q.Wo, q.H, q.W, q.p, 1, 0, 0, 0, 0, 0};
    const WalkTile t = walk_tile(q, sizeof(T) == 4 ? DT_F32 : DT_BF16, 1);
    g.TH = t.TH; g.nstrips = t.nstrips; g.nchunks = t.nchunks;
    const unsigned nblocks = (unsigned)t.blocks;
    hipLaunchKernelGGL((k_nhwca_bwd_data_s2<T, V, K, M>), dim3(nblocks), dim3(t.bs), 0, st, g, (const T *)dy, (const T *)w, (T *)dx, s2a_cols(q), nblocks,
                       stream_stores("NHWCA", 0, 0), q);
    return hipGetLastError();
}
template <typename T, int V, int K, int S>
static hipError_t filter_any(const Geom &q, const void *x, const void *dy, float *ws, hipStream_t st)
{
    FilterTile f;
    filter_tile_any(q, sizeof(T) == 4 ? DT_F32 : DT_BF16, &f);
    const AnyGeom g = {q.N, q.C, q.O, q.H, q.W, q.Ho, q.Wo, q.p, q.m, f.TH, f.nstrips, 0, f.TW, f.ncols};
    const unsigned nblocks = (unsigned)f.parts * f.nct;
    hipLaunchKernelGGL((k_nhwca_bwd_filter<T, V, K, S>), dim3(nblocks), dim3(256), 0, st, g, (const T *)x, (const T *)dy, ws, f.CT, f.parts, f.per,
                       nblocks);
    return hipGetLastError();
}

#define BY_KS(F, V, ...) (g.K == 3 ? (g.s == 1 ? F<T, V, 3, 1 __VA_ARGS__> : F<T, V, 3, 2 __VA_ARGS__>) \
                        : g.K == 5 ? (g.s == 1 ? F<T, V, 5, 1 __VA_ARGS__> : F<T, V, 5, 2 __VA_ARGS__>) \
                                   : (g.s == 1 ? F<T, V, 7, 1 __VA_ARGS__> : F<T, V, 7, 2 __VA_ARGS__>))
#define COMMA_ONE , 1
template <typename T>
static hipError_t fwd_any(const Geom &g, const void *x, const void *w, void *y, hipStream_t st)
{
    const int V = any_vec(g, sizeof(T) == 4 ? DT_F32 : DT_BF16, 0);
    if (V == 4) return (g.s == 1 ? conv_any<T, 4, 3, 1, 1> : conv_any<T, 4, 3, 2, 1>)(g, x, w, y, false, st);
    if (V == 2) return BY_KS(conv_any, 2, COMMA_ONE)(g, x, w, y, false, st);
    return BY_KS(conv_any, 1, COMMA_ONE)(g, x, w, y, false, st);
}
#define BY_K(F, V, M) (g.K == 3 ? F<T, V, 3, M> : g.K == 5 ? F<T, V, 5, M> : F<T, V, 7, M>)
#define BY_K1(F, V, M) (g.K == 3 ? F<T, V, 3, 1, M> : g.K == 5 ? F<T, V, 5, 1, M> : F<T, V, 7, 1, M>)
template <typename T>
static hipError_t bwd_data_any(const Geom &g, const void *dy, const void *w, void *dx, hipStream_t st)
{
    const int V = any_vec(g, sizeof(T) == 4 ? DT_F32 : DT_BF16, 1);
    if (g.s == 2) {
        if (g.m == 2) return BY_K(s2_any, 1, 2)(g, dy, w, dx, st);
        if (V == 4) return s2_any<T, 4, 3, 1>(g, dy, w, dx, st);
        if (V == 2) return BY_K(s2_any, 2, 1)(g, dy, w, dx, st);
        return BY_K(s2_any, 1, 1)(g, dy, w, dx, st);
    }
    if (g.m == 2) return BY_K1(conv_any, 1, 2)(g, dy, w, dx, true, st);
    if (V == 4) return conv_any<T, 4, 3, 1, 1>(g, dy, w, dx, true, st);
    if (V == 2) return BY_K1(conv_any, 2, 1)(g, dy, w, dx, true, st);
    return BY_K1(conv_any, 1, 1)(g, dy, w, dx, true, st);
}
template <typename T>
static hipError_t bwd_filter_any(const Geom &g, const void *x, const void *dy, float *ws, hipStream_t st)
{
    const int V = any_vec(g, sizeof(T) == 4 ? DT_F32 : DT_BF16, 2);
    if (V == 4) return (g.s == 1 ? filter_any<T, 4, 3, 1> : filter_any<T, 4, 3, 2>)(g, x, dy, ws, st);
    if (V == 2) return BY_KS(filter_any, 2, )(g, x, dy, ws, st);
    return BY_KS(filter_any, 1, )(g, x, dy, ws, st);
}
#undef BY_K
#undef BY_K1
#undef BY_KS
#undef COMMA_ONE

hipError_t nhwca_fwd(const Geom &g, int dtype, const void *x, const void *w, void *y, hipStream_t st)
{
    return dtype == DT_F32 ? fwd_any<float>(g, x, w, y, st) : fwd_any<bf16_t>(g, x, w, y, st);
}
hipError_t nhwca_bwd_data(const Geom &g, int dtype, const void *dy, const void *w, void *dx, hipStream_t st)
{
    return dtype == DT_F32 ? bwd_data_any<float>(g, dy, w, dx, st) : bwd_data_any<bf16_t>(g, dy, w, dx, st);
}
hipError_t nhwca_bwd_filter(const Geom &g, int dtype, const void *x, const void *dy, float *ws, hipStream_t st)
{
    return dtype == DT_F32 ? bwd_filter_any<float>(g, x, dy, ws, st) : bwd_filter_any<bf16_t>(g, x, dy, ws, st);
}

}  // namespace dwc

// Variant selection and launch dispatch.
#include "plan.hpp"
#include "short_filter.hpp"
#include <stdlib.h>

namespace dwc {

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Optional overrides for tuning runs, from the snapshot of tune.hpp (empty in normal use).
static int tune(const char *name, int dflt)
{
    const char *e = tune_env(name);
    if (!e) return dflt;
    int v = atoi(e);
    return v > 0 ? v : dflt;
}

static bool same_pad_s1(const Geom &g) { return g.s == 1 && (g.K == 3 || g.K == 5) && g.p == (g.K - 1) / 2; }
static bool k3s2p1(const Geom &g) { return g.s == 2 && g.K == 3 && g.p == 1; }

// channels per lane for the NHWC kernels, 0 if the fast path does not apply
static int nhwc_vec(const Geom &g, int dtype)
{
    // multiplier 2 has a fast path for 3x3 stride 1 only; the vector counts OUTPUT channels
    if (g.m == 2) { if (!(g.K == 3 && g.s == 1 && g.p == 1)) return 0; }
    else if (g.m != 1) return 0;
    if (dtype == DT_F32) return g.O % 4 == 0 ? 4 : 0;
    // 5x5: 25 taps x 8 channels would not fit in registers; 2 channels per lane take 110 registers
    // instead of the 208 of 4 channels and measured 1.25x faster.  These kernels address one image through a
    // buffer view of at most 2 GiB.
    if (g.K == 5) return (g.O % 2 == 0 && (long long)g.H * g.W * g.C * 2 <= (1LL << 31)) ? 2 : 0;
    return g.O % 8 == 0 ? 8 : (g.O % 4 == 0 ? 4 : 0);
}

// Rows loaded ahead in the NHWC stride-1 kernel.  fp32 3x3: four (inside the step the nine forward launches of the
// MobileNet stack take 522 us with four rows in flight against 531 with two; the small layers, whose wavefronts are
// all resident at once, gain most); bf16 3x3: three (input gradient 886 -> 870 us over the bf16 stack).  5x5 keeps
// 25 taps x V in registers: two rows.
static int nhwc_pf(const Geom &g, int dtype)
{
    int pf = tune("DWCONV_TUNE_PF", (g.K == 3 && g.m == 1) ? (dtype == DT_F32 ? 4 : 3) : 2);
    if (g.K == 5 && pf > 2) pf = 2;
    if (g.m != 1 && pf > 2) pf = 2;
    if (pf > 3 && !(dtype == DT_F32 && g.K == 3)) pf = 3;
    if (pf > 4) pf = 4;
    return pf;
}

// Rows per strip of the forward / backward-data row walks.  Measured on the benchmark layers:
// short strips win (14 input rows at stride 1, 7 output rows at stride 2) even though each strip
// re-reads K-1 halo rows (those come from L2): more, shorter walks keep the launch's accesses
// closer together in memory.
// A launch with fewer than MIN_LANES lanes (`lanes` per strip) takes strips of half the height, and half again down to four
// rows: it is one short round of wavefronts, each as long as its walk.  us with tall strips -> short ones, forward: bf16 NCHW
// 4x240x40x40 5x5 20.9 -> 5.7, 3x3 15.3 -> 4.7; bf16 NHWC 8x32x112x112 9.4 -> 4.7, 16x128x56x56 10.1 -> 6.4, 64x256x28x28 12.5 ->
// 10.1; fp32 NHWC 1x512x14x14 4.5 -> 3.0.  Half the limit leaves the NHWC 5x5 at 16.1 where this gives 6.6.
constexpr int MIN_LANES = 65536;
// (NCHW fp32 keeps tall strips from 2^20 outputs on where rows are under 64 and for 5x5: 44x32x65x20 3x3 5.9 us, with short ones 7.1;
// 16x64x32x32 5x5 8.6 against 10.  3x3 on wider rows, 400 layers of 2^20 to 2^22 outputs: short ones 14 % faster up to 1.75 million, as long on
// average from 2 million on, between 8 % slower and as fast.)
static long long nchw_lanes(const Geom &g, int dtype, int V)
{
    const long long rows = (long long)g.N * g.O;
    return dtype == DT_F32 && (g.W < 64 || g.K == 5) && rows * g.H * g.W >= 1 << 20 ? MIN_LANES : rows * (g.W / V);
}
static int pick_th(int rows, long long lanes, int stride, int dflt1 = 14, int dflt2 = 0)
{
    // stride 2: 7 output rows, 4 on tall maps (56 output rows and more: 1-4 % on the 112x112 and 56x56 layers);
    // the input gradient takes 4 dy rows on every map (28 dy rows: NHWC 45.2 -> 42.2 us, NCHW 44.0 -> 42.5 us; 14 dy
    // rows: NHWC 21.1 -> 19.5 us) and in NCHW 2 on tall maps (its 112x112 layer: 118 -> 110 us inside the step; NHWC
    // lost 1 % with it)
    if (dflt2 == 0) dflt2 = rows >= 56 ? 4 : 7;
    int target = stride == 1 ? tune("DWCONV_TUNE_TH1", dflt1) : tune("DWCONV_TUNE_TH2", dflt2);
    while (target > 4 && lanes * ceil_div(rows, target) < MIN_LANES) target = (target + 1) / 2;
    // balanced strips: the number of strips that brings their height closest to the target, then equal
    // heights (19 rows are one strip of 19, not 14 + 5; 37 rows are 13 + 13 + 11)
    int nstrips = (rows + target / 2) / target;
    if (nstrips < 1) nstrips = 1;
    const int th = ceil_div(rows, nstrips);
    return tune("DWCONV_TUNE_TH", th);
}

// Lanes that a strip of the NHWC row walks launches, idle ones at the end of a row among them: an image of 12 lanes a row is a block of 128
// whatever the strip (338x111x4x12 5x5 fp32: 19 us in strips of 14 rows, 26 in strips of 4, which counting 12 lanes asked for).
static long long nhwc_lanes(int N, int WQ) { const int b = nhwc_flat_block(WQ); return (long long)N * ((WQ + b - 1) / b * b); }

// Strip height of the NHWC stride-1 row walk: 14 rows for fp32; 28 for bf16, whose walks are bound by their
// vector-ALU work and pay for every halo row a strip computes again (5x5: 46.5 -> 44.2 us and 44.5 -> 41.9 us per
// launch over the bf16 stack; 3x3: 1 %).
static int nhwc_th1(int dtype) { return dtype == DT_BF16 ? 28 : 14; }

// Strip height of the NCHW stride-1 row walk.  The bf16 kernels are bound by their vector-ALU work (twice the
// elements per byte), so the K-1 halo rows a strip computes again cost them more than they cost the fp32 kernels:
// strips of 28 rows measured 2-9 % faster than 14 on the bf16 layers.
// fp32: 14 rows on rows of 112 elements; on rows of 56 and fewer (whole-line write-out in groups of four rows) 8 rows
// measured 3-4 % faster than 14 inside the step, on the forward pass and on the input gradient.
static int nchwd_th1(int dtype, int W) { return dtype == DT_BF16 ? 28 : (W <= 56 ? 8 : 14); }

// Small-plane NCHW kernels: rows of up to 14 always, and whenever the row walk cannot take the shape (bf16 rows that
// are not whole 16-byte vectors).  Rows of 28, where both families apply, go to whichever measured faster inside the
// benchmark step: the filter gradient always to the small-plane kernel (37 against 46 us on the 28x28x256 layer at
// batch 128, 23 against 29 us on its stride-2 sibling), the fp32 forward and the fp32 input gradient at stride 2
// too (stride-1 forward 42 against 47 us, stride-2 forward 28 against 31 us, stride-2 input gradient 21 against
// 22 us); the fp32 stride-1 input gradient stays with the row walk; bf16 see below.
static bool use_small(const Geom &g, int dtype, int pass)
{
    if (!nchws_supported(g, pass)) return false;
    if (g.W <= 14 || nchwd_vec(g, dtype, pass) == 0) return true;
    if (const char *e = tune_env("DWCONV_TUNE_S28")) return atoi(e) == 1;
    if (pass == 2) return true;
    if (dtype == DT_F32) return pass == 0 || (pass == 1 && g.s == 2);
    // bf16 at stride 1 (the 28x28 layer at batch 256, outputs staged in place): 3x3 forward 46 against 73 us, 3x3
    // input gradient 39 against 59 us, 5x5 forward 56 against 74 us, 5x5 input gradient 50 against 63 us
    return g.s == 1;
}

// The any-width NCHW kernels (nchw_flat.hip) take what neither the small planes nor the row walk takes, and of the
// row walk's shapes
// - the fp32 5x5 layers at stride 1 whose arithmetic the row walk does not hide.  Forward and input gradient (batch 64, us, row walk -> any
//   width: 16x16x480 27 -> 17, 20x20x480 34 -> 26, 40x40x240 63 -> 48, 48x48x240 91 -> 69, 56x56x128 at batch 128 125 -> 102; the input
//   gradient of 28x28x240 at batch 128 71 -> 51); small launches 7.5 -> 4.8, 9 -> 5.  The row walk keeps 1.5 to 2 million outputs, up to 4
//   million on rows of 28 and more, where its blocks make whole rounds and these do not (35x15x128x120 17 against 25, 350x22x72x72 11.9 against
//   14), and rows of 96 and more from 1.5 million on (as long or up to 20 % longer up to 2^24).  Filter gradient: rows of 12 to 24 on planes of
//   up to 35 rows (16x16 33 -> 23, 24x24 58 -> 45; 32x32 38 -> 49, 56x56 104 -> 114, 158x16x150x16 25 -> 38, 32x793x39x8 27 -> 34 stay).
// - of the bf16 3x3 layers at stride 1 the forward and input gradient of rows that are no whole number of 16-byte vectors, which the row walk
//   reads 8 bytes a lane (batch 64: 20x20x256 12.1 -> 9.5, 36x36x256 25.6 -> 18.9 and 31 -> 22, 52x52x128 31 -> 24, 60x60x128 38 -> 32,
//   76x76x64 30 -> 25, 100x100x64 49 -> 47; 140x140x32 45 -> 47 stays): rows of up to 24 from 2^22 outputs on (at batch 8 20x20x256 3.1
//   against 4.4), up to 44 from 1.5 times that, wider ones from 2^24 (2^22.5 outputs on rows of 60 9.8 -> 12.4, of 92 9.8 -> 13.2).
// bf16 5x5 stays with the packed-pair row walk (40x40x240 35 against 42).
static bool flat_over_rowwalk(const Geom &g, int dtype, int pass)
{
    if (g.s != 1 || g.W > 512) return false;                 // (the any-width kernels take rows of up to 512)
    const long long outputs = (long long)g.N * g.O * g.Ho * g.Wo;
    if (dtype == DT_F32) {
        if (g.K != 5 || !nchwf_fwd_supported(g, dtype) || !nchwf_bwd_data_supported(g, dtype)) return false;
        if (pass == 2) return g.W >= 12 && g.W <= 24 && g.H <= 35;
        return outputs < 3 << 19 || (g.W < 96 && outputs >= (g.W < 28 ? 1 << 21 : 1 << 22));
    }
    return g.K == 3 && g.W % 8 != 0 && g.W <= 128 && pass < 2 && outputs >= (g.W <= 24 ? 1 << 22 : g.W <= 44 ? 3 << 21 : 1 << 24);
}

static const char *flat_name(int K, int s, int pass)
{
    static const char *const names[3][3][2] = {
        {{"nchw_flat_k3s1", "nchw_flat_k3s2"}, {"nchw_flat_k5s1", "nchw_flat_k5s2"}, {"nchw_flat_k7s1", "nchw_flat_k7s2"}},
        {{"nchw_flat_k3s1_flip", "nchw_flat_bwd_data_k3s2"}, {"nchw_flat_k5s1_flip", "nchw_flat_bwd_data_k5s2"},
         {"nchw_flat_k7s1_flip", "nchw_flat_bwd_data_k7s2"}},
        {{"nchw_flat_bwd_filter_k3s1", "nchw_flat_bwd_filter_k3s2"}, {"nchw_flat_bwd_filter_k5s1", "nchw_flat_bwd_filter_k5s2"},
         {"nchw_flat_bwd_filter_k7s1", "nchw_flat_bwd_filter_k7s2"}}};
    return names[pass][(K - 3) / 2][s - 1];
}
static bool plan_flat(const Geom &g, int dtype, int pass, Plan &pl)
{
    // 7x7 filter gradients of a few thousand outputs stay with the generic kernels: the two reductions here cost more than the sums
    // (generic against these, 2x8x9x9 4.6 us and 9.9, 4x32x14x14 7.8 and 10.0, 8x64x28x28 44 and 14).  The forward pass is shorter here at
    // any size (2x8x9x9 fp32 8.1 us and 5.7, bf16 8.5 and 7.3, 1x256x7x7 unpadded 13.4 and 6.2).
    if (g.K == 7 && pass == 2 && (long long)g.N * g.O * g.Ho * g.Wo < 32768) return false;
    if (pass == 0 ? !nchwf_fwd_supported(g, dtype) : pass == 1 ? !nchwf_bwd_data_supported(g, dtype) : false) return false;
    if (pass == 2) {
        const int parts = nchwf_bwd_filter_parts(g, dtype);
        if (parts < 1) return false;
        pl.parts = parts;
    }
    pl.variant = pass == 0 ? V_NCHWF_FWD : pass == 1 ? V_NCHWF_BWD_DATA : V_NCHWF_BWD_FILTER;
    pl.name = flat_name(g.K, g.s, pass);
    return true;
}

// The NHWC walks of nhwc_any.hip for what nhwc.hip does not take.
static bool plan_any(const Geom &g, int dtype, int pass, Plan &pl)
{
    static const char *const names[3][3][2] = {
        {{"nhwc_any_k3s1", "nhwc_any_k3s2"}, {"nhwc_any_k5s1", "nhwc_any_k5s2"}, {"nhwc_any_k7s1", "nhwc_any_k7s2"}},
        {{"nhwc_any_k3s1_flip", "nhwc_any_bwd_data_k3s2"}, {"nhwc_any_k5s1_flip", "nhwc_any_bwd_data_k5s2"},
         {"nhwc_any_k7s1_flip", "nhwc_any_bwd_data_k7s2"}},
        {{"nhwc_any_bwd_filter_k3s1", "nhwc_any_bwd_filter_k3s2"}, {"nhwc_any_bwd_filter_k5s1", "nhwc_any_bwd_filter_k5s2"},
         {"nhwc_any_bwd_filter_k7s1", "nhwc_any_bwd_filter_k7s2"}}};
    if (!nhwca_supported(g, dtype, pass)) return false;
    const long long pixels = (long long)g.N * g.Ho * g.Wo;
    if (pass == 0) {
        // a forward pass of a few thousand outputs is as fast one output per thread (2x9x9x6 3.0 us against 2.5), and so is one whose rows
        // have so few lanes that most of a wavefront is idle (422x101x4x1 pad 0, multiplier 2 4.7 against 7.7, 506x90x3x2 5x5 stride 2 5.3 against 20)
        if (pixels * g.O < 2048) return false;
        if (nhwca_row_lanes(g, dtype) <= 4 && (long long)g.N * g.Ho >= 4096) return false;
    }
    // The filter gradient of a few pixels: the reduction over the block is longer than the sums (us, generic against this kernel, 3x3 up to
    // 16 pixels 5.7 / 6.3, 32 6.7 / 6.2; 5x5 16 5.6 / 7.6, 64 8.8 / 7.5; 7x7 16 5.7 / 10.5, 64 8.4 / 10.9, 128 15.2 / 11.1).
    if (pass == 2 && pixels < 2 * g.K * g.K) return false;
    if (pass == 2) pl.parts = nhwca_bwd_filter_parts(g, dtype);
    pl.variant = pass == 0 ? V_NHWCA_FWD : pass == 1 ? V_NHWCA_BWD_DATA : V_NHWCA_BWD_FILTER;
    pl.name = names[pass][(g.K - 3) / 2][g.s - 1];
    return true;
}

Plan plan_fwd(const Geom &g, int layout, int dtype)
{
    Plan pl = {V_GENERIC, 0, 0, 0, 0, "generic"};
    if (layout == LAYOUT_NCHW) {
        if (use_small(g, dtype, 0)) { pl.variant = V_NCHWS_FWD; pl.name = g.K == 5 ? "nchw_smallplane_k5s1" : (g.s == 1 ? "nchw_smallplane_k3s1" : "nchw_smallplane_fwd_k3s2"); return pl; }
        const int V = flat_over_rowwalk(g, dtype, 0) ? 0 : nchwd_vec(g, dtype, 0);
        if (V) {
            pl.a = V;
            if (g.s == 1) { pl.variant = V_NCHWD_S1; pl.b = pick_th(g.H, nchw_lanes(g, dtype, V), 1, nchwd_th1(dtype, g.W)); pl.name = g.K == 3 ? "nchw_rowwalk_k3s1" : "nchw_rowwalk_k5s1"; }
            else { pl.variant = V_NCHWD_K3S2; pl.b = pick_th(g.Ho, (long long)g.N * g.O * (g.Wo / V), 2); pl.name = "nchw_rowwalk_fwd_k3s2"; }
            return pl;
        }
        plan_flat(g, dtype, 0, pl);
        return pl;
    }
    if (layout == LAYOUT_NHWC) {
        const int V = nhwc_vec(g, dtype);
        if (V && same_pad_s1(g)) {
            pl.variant = V_NHWC_S1; pl.a = V; pl.b = pick_th(g.H, nhwc_lanes(g.N, g.W * (g.O / V)), 1, nhwc_th1(dtype));
            pl.name = g.m == 2 ? "nhwc_rowwalk_k3s1_m2" : (g.K == 3 ? "nhwc_rowwalk_k3s1" : "nhwc_rowwalk_k5s1");
        } else if (V && k3s2p1(g)) {
            pl.variant = V_NHWC_K3S2; pl.a = V; pl.b = pick_th(g.Ho, nhwc_lanes(g.N, g.Wo * (g.O / V)), 2);
            pl.name = "nhwc_rowwalk_fwd_k3s2";
        } else plan_any(g, dtype, 0, pl);
    }
    return pl;
}

Plan plan_bwd_data(const Geom &g, int layout, int dtype)
{
    Plan pl = {V_GENERIC, 0, 0, 0, 0, "generic"};
    if (layout == LAYOUT_NCHW) {
        if (use_small(g, dtype, 1)) {
            if (g.s == 1) { pl.variant = V_NCHWS_FWD; pl.name = g.K == 5 ? "nchw_smallplane_k5s1_flip" : "nchw_smallplane_k3s1_flip"; }
            else { pl.variant = V_NCHWS_BWD_DATA_S2; pl.name = "nchw_smallplane_bwd_data_k3s2"; }
            return pl;
        }
        const int V = flat_over_rowwalk(g, dtype, 1) ? 0 : nchwd_vec(g, dtype, 1);
        if (V) {
            pl.a = V;
            if (g.s == 1) { pl.variant = V_NCHWD_S1; pl.b = pick_th(g.H, nchw_lanes(g, dtype, V), 1, nchwd_th1(dtype, g.W)); pl.name = g.K == 3 ? "nchw_rowwalk_k3s1_flip" : "nchw_rowwalk_k5s1_flip"; }
            else { pl.variant = V_NCHWD_K3S2; pl.b = pick_th(g.Ho, (long long)g.N * g.O * (g.Wo / V), 2, 14, g.Ho >= 56 ? 2 : 4); pl.name = "nchw_rowwalk_bwd_data_k3s2"; }
            return pl;
        }
        plan_flat(g, dtype, 1, pl);
        return pl;
    }
    if (layout == LAYOUT_NHWC) {
        const int V = nhwc_vec(g, dtype);
        if (V && same_pad_s1(g)) {
            pl.variant = V_NHWC_S1; pl.a = V; pl.b = pick_th(g.H, nhwc_lanes(g.N, g.W * (g.O / V)), 1, nhwc_th1(dtype));
            pl.name = g.m == 2 ? "nhwc_rowwalk_k3s1_flip_m2" : (g.K == 3 ? "nhwc_rowwalk_k3s1_flip" : "nhwc_rowwalk_k5s1_flip");
        } else if (V && k3s2p1(g)) {
            pl.variant = V_NHWC_K3S2; pl.a = V; pl.b = pick_th(g.Ho, nhwc_lanes(g.N, g.Wo * (g.O / V)), 2, 14, 4);
            pl.name = "nhwc_rowwalk_bwd_data_k3s2";
        } else plan_any(g, dtype, 1, pl);
    }
    return pl;
}

// NCHW filter gradient on the small-plane kernels / on the row walk; false if the family does not take the shape.
static bool plan_bwd_filter_nchws(const Geom &g, int dtype, Plan &pl)
{
    int U, NI, parts;
    nchws_bwd_filter_tiling(g, dtype, &U, &NI, &parts);
    NI = tune("DWCONV_TUNE_NI", NI);
    if (NI > g.N) NI = g.N;
    parts = ceil_div(g.N, NI);
    if ((long long)parts * g.O * g.K * g.K * 4 > (64ll << 20)) return false;
    pl.variant = V_NCHWS_BWD_FILTER; pl.a = U; pl.b = 0; pl.c = NI; pl.parts = parts;
    pl.name = g.K == 5 ? "nchw_smallplane_bwd_filter_k5s1"
                       : (g.s == 1 ? "nchw_smallplane_bwd_filter_k3s1" : "nchw_smallplane_bwd_filter_k3s2");
    return true;
}

static bool plan_bwd_filter_nchwd(const Geom &g, int dtype, Plan &pl)
{
    const int V = nchwd_vec(g, dtype, 2);
    if (!V) return false;
    // strip height (measured on the benchmark layers): stride 2 wants short strips of 7 output rows,
    // fp32 stride 1 on large planes 14 rows, everything else whole planes up to 56 rows
    int TH = g.s == 2 && g.Ho >= 28 ? 7
             : (g.s == 1 && dtype == DT_F32 && g.Ho >= 56 ? 14 : (g.Ho > 56 ? (g.Ho + 1) / 2 : g.Ho));
    TH = tune("DWCONV_TUNE_THW", tune("DWCONV_TUNE_TH", TH));
    int lg, nst, rounds, parts;
    nchwd_bwd_filter_tiling(g, V, TH, &lg, &nst, &rounds, &parts);
    // small batches: shorter strips until the launch has about two blocks per CU (one block = one
    // channel x a group of (image, strip) items)
    while (TH > 7 && parts >= 1 && (long long)parts * g.O < 512 && !tune_env("DWCONV_TUNE_THW") && !tune_env("DWCONV_TUNE_TH")) {
        TH = (TH + 1) / 2;
        nchwd_bwd_filter_tiling(g, V, TH, &lg, &nst, &rounds, &parts);
    }
    if (!(lg >= 1 && parts >= 1 && (long long)parts * g.O * g.K * g.K * 4 <= (64ll << 20))) return false;
    pl.variant = V_NCHWD_BWD_FILTER; pl.a = V; pl.b = TH; pl.c = 0; pl.parts = parts;
    pl.name = g.K == 5 ? "nchw_rowwalk_bwd_filter_k5s1"
                       : (g.s == 1 ? "nchw_rowwalk_bwd_filter_k3s1" : "nchw_rowwalk_bwd_filter_k3s2");
    return true;
}

// the depthwise layer as a group convolution of one channel a group
static GGeom as_group(const Geom &g)
{
    GGeom q;
    q.N = g.N; q.C = g.C; q.H = g.H; q.W = g.W; q.K = g.K; q.s = g.s; q.p = g.p; q.G = g.C; q.O = g.O; q.Cg = 1; q.Og = g.m; q.Ho = g.Ho; q.Wo = g.Wo;
    return q;
}

// force_v > 0: channels per lane of the NHWC kernel (the fused backward kernel has four in either type)
static Plan plan_bwd_filter_v(const Geom &g, int layout, int dtype, int force_v)
{
    Plan pl = {V_GENERIC, generic_bwd_filter_parts(g), 0, 0, 0, "generic"};
    if (layout == LAYOUT_NCHW) {
        if (use_small(g, dtype, 2) && plan_bwd_filter_nchws(g, dtype, pl)) return pl;
        if (!flat_over_rowwalk(g, dtype, 2) && plan_bwd_filter_nchwd(g, dtype, pl)) return pl;
        plan_flat(g, dtype, 2, pl);
        return pl;
    }
    if (layout == LAYOUT_NHWC) {
        int V = nhwc_vec(g, dtype);
        // bf16 on small planes: four channels per lane (124 registers, four wavefronts per SIMD) measured faster
        // than eight (182 registers, two wavefronts)
        if (V == 8 && tune("DWCONV_TUNE_WV", g.W <= 14 ? 4 : 8) == 4) V = 4;
        if (force_v > 0 && V >= force_v) V = force_v;
        if (V && (same_pad_s1(g) || k3s2p1(g))) {
            // One block = 256 lanes over (columns x channel-vectors) x one strip x NI images.  Long
            // walks win (fewer partials, less stage-2 work): start from whole columns and one image
            // per block, and only split rows when the launch would have too few blocks to keep the
            // memory system busy.
            int CT, nct, nowt, nst, ngr;
            nhwc_bwd_filter_tiling(g, V, g.Ho, 1, &CT, &nct, &nowt, &nst, &ngr);
            const long long per_strip = (long long)nct * nowt * g.N;   // blocks with NI = 1 and one strip
            // Measured on all benchmark layers: about two blocks per CU (512) is the sweet spot, and a
            // block that walks two images beats two blocks with one image each; stride 2 tolerates
            // half as many blocks again.
            // 5x5 is bound by its multiply-adds and wants four wavefronts per SIMD (1024 blocks), not two
            const long long want = tune("DWCONV_TUNE_WBLOCKS", g.K == 5 ? 1024 : 512), floor_blocks = g.s == 1 ? want * 3 / 4 : want / 2;
            int TH = g.Ho, NI = 1;
            while (TH > 7 && per_strip * ceil_div(g.Ho, TH) * 4 < want * 3) TH = (TH + 1) / 2;
            while (NI < g.N && per_strip * ceil_div(g.Ho, TH) / (NI * 2) >= floor_blocks) NI *= 2;
            TH = tune("DWCONV_TUNE_THW", tune("DWCONV_TUNE_TH", TH)); NI = tune("DWCONV_TUNE_NI", NI);
            if (TH > g.Ho) TH = g.Ho;
            if (NI > g.N) NI = g.N;
            nhwc_bwd_filter_tiling(g, V, TH, NI, &CT, &nct, &nowt, &nst, &ngr);
            // keep the partials within 64 MiB: more images per block, then taller strips; a shape that is
            // still above it with whole columns of the whole batch per block (very many channels times very
            // wide rows) goes to the any-channel kernels, whose partials are at most 8 MiB or a single O*K*K array
            while ((long long)nowt * nst * ngr * g.O * g.K * g.K * 4 > (64ll << 20) && (NI < g.N || TH < g.Ho)) {
                if (NI < g.N) NI = NI * 2 < g.N ? NI * 2 : g.N; else TH = TH * 2 < g.Ho ? TH * 2 : g.Ho;
                nhwc_bwd_filter_tiling(g, V, TH, NI, &CT, &nct, &nowt, &nst, &ngr);
            }
            if ((long long)nowt * nst * ngr * g.O * g.K * g.K * 4 > (64ll << 20)) { plan_any(g, dtype, 2, pl); return pl; }
            pl.variant = V_NHWC_BWD_FILTER; pl.a = V; pl.b = TH; pl.c = NI;
            pl.parts = nowt * nst * ngr;
            pl.name = g.m == 2 ? "nhwc_bwd_filter_k3s1_m2"
                               : (g.s == 2 ? "nhwc_bwd_filter_k3s2" : (g.K == 3 ? "nhwc_bwd_filter_k3s1" : "nhwc_bwd_filter_k5s1"));
        } else plan_any(g, dtype, 2, pl);
    }
    return pl;
}

Plan plan_bwd_filter(const Geom &g, int layout, int dtype)
{
    Plan pl = plan_bwd_filter_v(g, layout, dtype, 0);
    const FilterWay way = pl.variant == V_GENERIC && pl.parts == 1 ? FILTER_GENERIC_ONE : pl.variant == V_NCHWS_BWD_FILTER ? FILTER_SMALL_PLANES : FILTER_TWO;
    if (short_bwd_filter_shorter(as_group(g), layout, dtype, way)) {
        pl.variant = V_SHORT_BWD_FILTER; pl.parts = 1;
        pl.name = layout == LAYOUT_NCHW ? "nchw_short_bwd_filter" : "nhwc_short_bwd_filter";
    }
    return pl;
}

Plan plan_bwd(const Geom &g, int layout, int dtype)
{
    Plan pl = {V_GENERIC, 0, 0, 0, 0, "separate"};
    if (layout == LAYOUT_NHWC && !tune_env("DWCONV_TUNE_NOFUSE")) {
        // the fused kernel takes four channels per lane in either type (bf16 with eight would need more than 256 registers)
        int V = nhwc_vec(g, dtype);
        if (V == 8 && g.W <= tune("DWCONV_TUNE_FUSE_BF16W", 65536)) V = 4;
        if (V && nhwc_bwd_fused_supported(g, dtype, V)) {
            // tiling of the filter gradient: its block count and partial sums decide
            const Plan pf = plan_bwd_filter_v(g, layout, dtype, V);
            if (pf.variant == V_NHWC_BWD_FILTER && pf.a == V) {
                pl = pf;
                pl.variant = V_NHWC_BWD_FUSED;
                pl.name = g.m == 2 ? "nhwc_bwd_fused_k3s1_m2" : (g.s == 1 ? "nhwc_bwd_fused_k3s1" : "nhwc_bwd_fused_k3s2");
            }
        }
    }
    if (layout == LAYOUT_NCHW && !tune_env("DWCONV_TUNE_NOFUSE")) {
        // a fused kernel of either family, whichever the separate filter gradient would run on
        Plan pf = pl;
        // (28-wide fp32 rows at stride 1 are whole 16-byte vectors: they stay with the row-walk fused kernel below)
        const bool rowwalk28 = g.s == 1 && g.W == 28 && dtype == DT_F32;
        if (use_small(g, dtype, 2) && !rowwalk28 && nchws_bwd_fused_supported(g) && plan_bwd_filter_nchws(g, dtype, pf)) {
            int U, NI, parts;
            nchws_bwd_fused_tiling(g, dtype, &U, &NI, &parts);
            if ((long long)parts * g.O * g.K * g.K * 4 <= (64ll << 20)) {
                pl = pf;
                pl.variant = V_NCHWS_BWD_FUSED; pl.a = U; pl.c = NI; pl.parts = parts;
                pl.name = g.s == 1 ? "nchw_smallplane_bwd_fused_k3s1" : "nchw_smallplane_bwd_fused_k3s2";
                return pl;
            }
        }
        pf = pl;
        if (g.s == 2 && !use_small(g, dtype, 2) && !tune_env("DWCONV_TUNE_NOFUSE_NCHW_S2") && plan_bwd_filter_nchwd(g, dtype, pf)) {
            // stride 2 on row-walk shapes: two dy columns per lane, strips of the filter gradient's height made even
            // where a write-out group is four dx rows
            const int V2 = dtype == DT_F32 ? 2 : 4, rs = nchwd_bwd_fused_rs(g, dtype, V2);
            if (rs) {
                const int TH = (2 * pf.b) % rs == 0 ? pf.b : pf.b + 1;
                int lg, nst, rounds, parts;
                nchwd_bwd_filter_tiling(g, V2, TH, &lg, &nst, &rounds, &parts);
                if (lg >= 1 && parts >= 1 && (long long)parts * g.O * g.K * g.K * 4 <= (64ll << 20)) {
                    pl = pf;
                    pl.variant = V_NCHWD_BWD_FUSED; pl.a = V2; pl.b = TH; pl.parts = parts;
                    pl.name = "nchw_bwd_fused_k3s2";
                    return pl;
                }
            }
        }
        pf = pl;
        if (g.s == 1 && plan_bwd_filter_nchwd(g, dtype, pf)) {
            const int rs = nchwd_bwd_fused_rs(g, dtype, pf.a);
            if (rs) {
                // the filter gradient's tiling with the strip height rounded up to whole row groups
                const int TH = (pf.b + rs - 1) / rs * rs;
                int lg, nst, rounds, parts;
                nchwd_bwd_filter_tiling(g, pf.a, TH, &lg, &nst, &rounds, &parts);
                if (lg >= 1 && parts >= 1 && (long long)parts * g.O * g.K * g.K * 4 <= (64ll << 20)) {
                    pl = pf;
                    pl.variant = V_NCHWD_BWD_FUSED; pl.b = TH; pl.parts = parts;
                    pl.name = "nchw_bwd_fused_k3s1";
                    return pl;
                }
            }
        }
        // where both passes would run on the any-width kernels
        if (g.s == 1 && g.K == 3 && plan_bwd_data(g, layout, dtype).variant == V_NCHWF_BWD_DATA && plan_bwd_filter_v(g, layout, dtype, 0).variant == V_NCHWF_BWD_FILTER) {
            const int parts = nchwf_bwd_fused_parts(g, dtype);
            if (parts > 0) { pl = {V_NCHWF_BWD_FUSED, parts, 0, 0, 0, "nchw_flat_bwd_fused_k3s1"}; }
        }
    }
    return pl;
}

hipError_t launch_fwd(const Plan &pl, const Geom &g, int layout, int dtype, const void *x, const void *w, void *y,
                      hipStream_t st)
{
    switch (pl.variant) {
    case V_NHWC_S1: return nhwc_s1(g, dtype, pl.a, x, w, y, false, pl.b, nhwc_pf(g, dtype), st);
    case V_NHWC_K3S2: return nhwc_k3s2(g, dtype, pl.a, x, w, y, false, pl.b, st);
    case V_NHWCA_FWD: return nhwca_fwd(g, dtype, x, w, y, st);
    case V_NCHWF_FWD: return nchwf_fwd(g, dtype, x, w, y, st);
    case V_NCHWD_S1: return nchwd_s1(g, dtype, pl.a, x, w, y, false, pl.b, st);
    case V_NCHWS_FWD: return nchws_fwd(g, dtype, x, w, y, false, st);
    case V_NCHWD_K3S2: return nchwd_k3s2(g, dtype, pl.a, x, w, y, false, pl.b, st);
    default: return generic_fwd(g, layout, dtype, x, w, y, st);
    }
}

hipError_t launch_bwd_data(const Plan &pl, const Geom &g, int layout, int dtype, const void *dy, const void *w,
                           void *dx, hipStream_t st)
{
    switch (pl.variant) {
    case V_NHWC_S1: return nhwc_s1(g, dtype, pl.a, dy, w, dx, true, pl.b, nhwc_pf(g, dtype), st);
    case V_NHWC_K3S2: return nhwc_k3s2(g, dtype, pl.a, dy, w, dx, true, pl.b, st);
    case V_NHWCA_BWD_DATA: return nhwca_bwd_data(g, dtype, dy, w, dx, st);
    case V_NCHWF_BWD_DATA: return nchwf_bwd_data(g, dtype, dy, w, dx, st);
    case V_NCHWD_S1: return nchwd_s1(g, dtype, pl.a, dy, w, dx, true, pl.b, st);
    case V_NCHWS_FWD: return nchws_fwd(g, dtype, dy, w, dx, true, st);
    case V_NCHWS_BWD_DATA_S2: return nchws_bwd_data_s2(g, dtype, dy, w, dx, st);
    case V_NCHWD_K3S2: return nchwd_k3s2(g, dtype, pl.a, dy, w, dx, true, pl.b, st);
    default: return generic_bwd_data(g, layout, dtype, dy, w, dx, st);
    }
}

hipError_t launch_bwd_filter(const Plan &pl, const Geom &g, int layout, int dtype, const void *x, const void *dy,
                             float *ws, hipStream_t st)
{
    switch (pl.variant) {
    case V_NHWC_BWD_FILTER: return nhwc_bwd_filter(g, dtype, pl.a, x, dy, ws, pl.b, pl.c, st);
    case V_NHWCA_BWD_FILTER: return nhwca_bwd_filter(g, dtype, x, dy, ws, st);
    case V_NCHWF_BWD_FILTER: return nchwf_bwd_filter(g, dtype, x, dy, ws, pl.parts, st);
    case V_NCHWD_BWD_FILTER: return nchwd_bwd_filter(g, dtype, pl.a, x, dy, ws, pl.b, st);
    case V_NCHWS_BWD_FILTER: return nchws_bwd_filter(g, dtype, x, dy, ws, pl.a, pl.c, st);
    case V_SHORT_BWD_FILTER: return short_bwd_filter(as_group(g), layout, dtype, x, dy, ws, st);
    default: return generic_bwd_filter(g, layout, dtype, x, dy, ws, pl.parts, st);
    }
}

bool sums_are_final(const Plan &pl)
{
    return pl.parts == 1 && pl.variant != V_NCHWF_BWD_FILTER && pl.variant != V_NHWCA_BWD_FILTER && pl.variant != V_NCHWF_BWD_FUSED;
}

hipError_t launch_reduce(const Plan &pl, const Geom &g, int layout, int dtype, const void *x, const void *dy, const float *ws, float *dw,
                         hipStream_t st)
{
    const int J = g.O * g.K * g.K;
    if (pl.variant != V_NCHWF_BWD_FILTER && pl.variant != V_NHWCA_BWD_FILTER && pl.variant != V_NCHWF_BWD_FUSED) return reduce_partials(ws, pl.parts, J, dw, st);
    FilterGradSrc src = {x, dy, dtype, layout, g.N, g.C, g.H, g.W, g.K, g.s, g.p, g.O, 1, g.m, g.Ho, g.Wo};
    if (pl.variant == V_NCHWF_BWD_FILTER) nchwf_bwd_filter_tiles(g, dtype, pl.parts, &src);
    else if (pl.variant == V_NCHWF_BWD_FUSED) nchwf_bwd_fused_tiles(g, dtype, pl.parts, &src);
    else nhwca_bwd_filter_tiles(g, dtype, &src);
    // (the any-channel walks: one channel a lane leaves fewer lanes across the columns, each with more of them, in fp32 1.014 to 1.018 times the
    // error against 64 bits of two channels a lane; with the partials in 64 bits 0.86 to 0.89, bf16 0.73 to 0.74, in the same time)
    return reduce_partials(ws, pl.parts, J, dw, src, pl.variant == V_NHWCA_BWD_FILTER, st);
}

hipError_t launch_bwd_fused(const Plan &pl, const Geom &g, int layout, int dtype, const void *x, const void *dy,
                            const void *w, void *dx, float *ws, hipStream_t st)
{
    (void)layout;
    if (pl.variant == V_NCHWD_BWD_FUSED) return nchwd_bwd_fused(g, dtype, pl.a, x, dy, w, dx, ws, pl.b, st);
    if (pl.variant == V_NCHWS_BWD_FUSED) return nchws_bwd_fused(g, dtype, x, dy, w, dx, ws, pl.a, pl.c, st);
    if (pl.variant == V_NCHWF_BWD_FUSED) return nchwf_bwd_fused(g, dtype, x, dy, w, dx, ws, pl.parts, st);
    if (pl.variant != V_NHWC_BWD_FUSED) return hipErrorInvalidValue;
    return nhwc_bwd_fused(g, dtype, pl.a, x, dy, w, dx, ws, pl.b, pl.c, st);
}

}  // namespace dwc

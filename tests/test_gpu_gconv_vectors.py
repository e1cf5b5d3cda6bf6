"""GPU parity of the 16x16 group kernels at the edges of how they copy and lay out: the filter in whole vectors (groups that straddle a
vector, filters smaller than one, a last block with half its outputs), tiles of several rounds of loads, pairs of output columns of the
stride-2 input gradient (odd and even padding and width), filters that take more than 64 KiB of LDS, tiles of few positions, and position
splits added up in the block.  Against the CPU group oracle, element by element; a sum has up to 64 * 25 products (fp32: about
sqrt(1600) * 2^-24 = 2.4e-6 of the rms term sum, inside 1e-5)."""
import pytest

import paper_1803_09926_amd as dw
from oracle import gconv as og
from paper_1803_09926_amd import workloads as wl

import gpu_util as gu
from test_gpu_gconv import run_gpu
from test_gpu_gconv_gemm import matrix_instructions        # noqa: F401  (these kernels wherever they take the shape)

pytestmark = pytest.mark.gpu

# name, N, C, O, groups, H, W, K, stride, pad
CASES = [
    ("pairs_even_pad", 2, 32, 32, 2, 20, 24, 3, 2, 0),             # no shift, whole rows of quads
    ("pairs_odd_pad", 2, 32, 32, 2, 21, 32, 3, 2, 1),              # shift, aligned rows
    ("pairs_odd_width", 2, 24, 24, 3, 13, 31, 5, 2, 2),            # the last pair has one column
    ("pairs_pad3", 2, 16, 16, 1, 18, 22, 5, 2, 3),
    ("half_block", 3, 24, 24, 1, 16, 15, 3, 1, 1),                 # 24 outputs: the second block has eight
    ("straddle", 2, 48, 48, 8, 16, 13, 3, 1, 1),                   # groups of 6: vectors and blocks span groups
    ("og4_cg12", 2, 36, 12, 3, 14, 17, 3, 1, 1),
    ("og12_cg4", 2, 16, 48, 4, 14, 17, 3, 1, 1),
    ("cg20", 1, 40, 40, 2, 12, 13, 3, 1, 1),                       # an output block of 4 and one of 16 in a group
    ("k2", 2, 32, 32, 2, 12, 13, 2, 1, 0),                         # four taps: fewer than a bf16 vector has entries
    ("lds_over_64k", 2, 64, 64, 1, 11, 13, 5, 1, 2),
    ("lds_over_64k_s2", 2, 64, 64, 1, 19, 22, 5, 2, 2),
    ("few_positions", 2, 512, 512, 32, 3, 4, 3, 1, 1),             # fewer 16-position tiles than wavefronts
    ("one_pair", 5, 16, 16, 1, 29, 27, 3, 1, 1),                   # filter gradient: four position splits of one pair
    ("wide", 1, 16, 16, 1, 9, 300, 3, 1, 1),                       # more columns than lanes of a row
    ("lds_over_140k", 1, 32, 32, 1, 28, 28, 7, 1, 3),              # fp32: one block on a compute unit
    ("one_input", 1, 2, 2, 1, 1, 1, 3, 1, 20),                     # two input elements: no four to load at once
    ("one_input_301", 301, 2, 1024, 1, 1, 1, 5, 1, 4),             # images of two elements: a tile of one image behind the others
    ("one_pixel", 65537, 2, 64, 1, 1, 1, 1, 1, 0),                 # the same with many images a tile, all passes
    ("odd_groups", 2, 24, 40, 8, 13, 15, 3, 1, 1),                 # a group's filter is no whole number of vectors
    ("tail", 1, 20, 20, 5, 37, 35, 3, 1, 1),                       # a run of four passes the tensor's end
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_vectors_pairs_and_large_filters(case, layout, dtype):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    names = [dw.gconv_variant_name(d, i) for i in range(3)]
    print("case", name, layout, dtype, names, flush=True)
    if "rowwalk" not in names[0]:
        assert names[0] == "group_mfma16" and (names[1] == "group_mfma16_bwd_data" or N * C * H * W < 2048)      # (few outputs: one per thread)
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=91)
    y, dx, dwt = run_gpu(case, layout, dtype, x, w, dy)
    kw = dict(K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    tol = gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16
    gu.assert_close(gu.to_host(y), og.fwd(x, w, **kw), tol, "fwd " + name)
    gu.assert_close(gu.to_host(dx), og.bwd_data(dy, w, x_shape=x.shape, **kw), tol, "bwd_data " + name)
    gu.assert_close(gu.to_host(dwt), og.bwd_filter(x, dy, **kw), gu.TOL_F32_FILTER, "bwd_filter " + name)


# the input gradient alone: images of two and three elements of dy, odd batches; x must come to 2048 elements, y need not.  Then blocks whose
# outputs lie in two groups or are no whole vectors, which lay out the filter entry by entry beside others that take vectors.
DY_CASES = [
    ("dy_of_two", 7, 64, 2, 1, 7, 7, 7, 1, 0),                     # input gradient: two elements of dy an image, an odd batch
    ("dy_of_two_padded", 9, 64, 2, 1, 5, 5, 7, 1, 1),
    ("dy_of_three", 9, 64, 3, 1, 7, 7, 7, 1, 0),
    ("cg100", 3, 200, 200, 2, 9, 11, 3, 1, 1),
    ("cg100_s2", 2, 200, 96, 2, 14, 13, 3, 2, 1),
    ("cg131", 2, 131, 24, 1, 9, 8, 5, 1, 2),                       # NCHW: the last block has three outputs
    ("cg36", 2, 144, 144, 4, 8, 9, 3, 1, 1),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", DY_CASES, ids=[c[0] for c in DY_CASES])
def test_input_gradient_alone(case, layout, dtype):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    print("case", name, layout, dtype, dw.gconv_variant_name(d, 1), flush=True)
    assert dw.gconv_variant_name(d, 1) == "group_mfma16_bwd_data"
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=93)
    _, dx, _ = run_gpu(case, layout, dtype, x, w, dy)
    ref = og.bwd_data(dy, w, x_shape=x.shape, K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    gu.assert_close(gu.to_host(dx), ref, gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16, "bwd_data " + name)


def test_input_gradient_whose_filter_has_27_million_entries():
    """12001 channels are 750 blocks of 16 outputs and one of one output, whose 256 x 9 entries are no run of the filter."""
    N, C, O, H = 2, 12001, 256, 7
    case = ("large_filter", N, C, O, 1, H, H, 3, 1, 1)
    d = dw.group_desc(N, C, H, H, 3, 1, 1, 1, O, wl.NCHW, wl.BF16)
    print("case large_filter", dw.gconv_variant_name(d, 1), flush=True)
    assert dw.gconv_variant_name(d, 1) == "group_mfma16_bwd_data"
    x, w, dy = wl.make_group_inputs(N, C, O, 1, H, H, 3, 1, 1, wl.NCHW, wl.BF16, seed=94)
    _, dx, _ = run_gpu(case, wl.NCHW, wl.BF16, x, w, dy)
    ref = og.bwd_data(dy, w, x_shape=x.shape, K=3, stride=1, pad=1, groups=1, O=O, layout=wl.NCHW, nthreads=8)
    gu.assert_close(gu.to_host(dx), ref, gu.TOL_BF16, "bwd_data")


# launches of about 200 blocks and more whose tiles have 65 to 128 positions and output blocks: a wavefront takes two 16-position tiles at a time
TWO_AT_ONCE = [
    ("g12_16x23", 12, 96, 96, 12, 16, 23, 3, 1, 1),
    ("g12_13x5", 12, 384, 384, 12, 13, 5, 3, 1, 1),                # two output blocks
    ("g8_10x13", 8, 256, 256, 8, 10, 13, 3, 1, 1),
    ("g11_23x11", 12, 88, 88, 11, 23, 11, 3, 1, 1),                # 16 outputs span groups of 8
    ("g6_s2", 11, 192, 192, 6, 20, 21, 3, 2, 1),
    ("g5_s2", 12, 160, 160, 5, 23, 22, 3, 2, 1),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", TWO_AT_ONCE, ids=[c[0] for c in TWO_AT_ONCE])
def test_two_tiles_at_once(case, layout, dtype):
    test_vectors_pairs_and_large_filters(case, layout, dtype)


# the same with tiles of about 200 positions and output blocks and more: four at a time, in all passes' full tiles
FOUR_AT_ONCE = [
    ("g3_25x23", 22, 36, 36, 3, 25, 23, 3, 1, 1),                  # 16 outputs span groups of 12, the last block has four outputs
    ("g7_10x29", 14, 112, 112, 7, 10, 29, 3, 1, 1),
    ("g4_26x11", 23, 80, 80, 4, 26, 11, 3, 1, 1),                  # groups of 20
    ("g7_s2", 15, 224, 224, 7, 25, 26, 3, 2, 1),                   # two output blocks; pairs of columns of the input gradient
    ("g11_s2", 10, 352, 352, 11, 24, 27, 3, 2, 1),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", FOUR_AT_ONCE, ids=[c[0] for c in FOUR_AT_ONCE])
def test_four_tiles_at_once(case, layout, dtype):
    test_vectors_pairs_and_large_filters(case, layout, dtype)

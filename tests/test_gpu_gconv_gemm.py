"""GPU parity of the group-convolution kernels on the 16x16 matrix instructions (any group size, filter, stride, padding,
layout) against the CPU group oracle, element by element, at the edges of their tiling.  fp32 sums have up to 25 * 32 products
(~ sqrt(800) * 2^-24 = 2e-6 of the rms term sum: inside 1e-5); other tolerances as in gpu_util."""
import numpy as np
import pytest
import torch

import paper_1803_09926_amd as dw
from oracle import gconv as og
from paper_1803_09926_amd import workloads as wl

import gpu_util as gu
from test_gpu_gconv import run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def matrix_instructions():
    """These kernels wherever they take the shape: the small ones below are shorter one output per thread and would go there."""
    with dw.tuning_overrides({"DWCONV_TUNE_GROUP_GEMM": 1}):
        yield


# name, N, C, O, groups, H, W, K, stride, pad
CASES = [
    ("cg16", 3, 32, 32, 2, 14, 14, 3, 1, 1),                       # several images a tile
    ("cg32_k5", 2, 64, 64, 2, 13, 11, 5, 1, 2),
    ("cg8_s2_odd", 2, 64, 64, 8, 37, 41, 3, 2, 1),
    ("cg4_s2_even", 2, 24, 24, 6, 40, 56, 3, 2, 1),
    ("cg2_k5_s2", 3, 20, 20, 10, 17, 23, 5, 2, 2),
    ("cg4_odd_width", 2, 12, 12, 3, 31, 57, 3, 1, 1),
    ("wide_rows", 1, 8, 8, 2, 7, 150, 5, 1, 2),                    # more than one tile across
    ("cg24", 2, 48, 48, 2, 20, 22, 3, 2, 1),                       # 16 outputs span two groups, inputs no multiple of 16
    ("cg3_og5", 3, 9, 15, 3, 20, 19, 3, 1, 1),
    ("cg20_og4", 2, 40, 8, 2, 19, 33, 3, 1, 1),
    ("cg2_og6_s2", 2, 8, 24, 4, 30, 21, 3, 2, 1),
    ("one_group_dense", 2, 33, 17, 1, 15, 17, 3, 1, 1),
    ("k1_s2", 4, 32, 32, 2, 15, 16, 1, 2, 0),                      # classes without a tap: zeros
    ("k1", 3, 32, 64, 2, 13, 12, 1, 1, 0),
    ("k3_s3", 2, 16, 16, 2, 40, 37, 3, 3, 1),
    ("pad3_k3", 2, 16, 16, 1, 20, 19, 3, 1, 3),                    # columns of pure padding
    ("k7_fwd", 2, 16, 16, 2, 20, 24, 7, 1, 3),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_mfma16_group_conv_matches_oracle(case, layout, dtype):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    print("case", name, layout, dtype, [dw.gconv_variant_name(d, i) for i in range(3)], flush=True)
    # (NHWC has a row walk for groups of 4 at any width, and 49 taps in fp32 leave no room for a tile)
    if not (layout == wl.NHWC and name == "cg4_odd_width") and not (dtype == wl.F32 and name == "k7_fwd"):
        assert "group_mfma16" in dw.gconv_variant_name(d, 0) + dw.gconv_variant_name(d, 1)
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=77)
    y, dx, dwt = run_gpu(case, layout, dtype, x, w, dy)
    kw = dict(K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    tol = gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16
    gu.assert_close(gu.to_host(y), og.fwd(x, w, **kw), tol, "fwd " + name)
    gu.assert_close(gu.to_host(dx), og.bwd_data(dy, w, x_shape=x.shape, **kw), tol, "bwd_data " + name)
    gu.assert_close(gu.to_host(dwt), og.bwd_filter(x, dy, **kw), gu.TOL_F32_FILTER, "bwd_filter " + name)


# NCHW layers whose filter has no room for a padding of its own: a block less would fit a compute unit, or none at all
TIGHT = [
    ("tight_cg160", 1, 160, 160, 1, 19, 19, 3, 1, 1),
    ("tight_k5", 1, 16, 16, 1, 12, 20, 5, 1, 2),
    ("tight_k5_bf16", 3, 32, 32, 1, 7, 33, 5, 1, 2),
    ("tight_pairs", 1, 96, 96, 2, 7, 12, 3, 2, 1),                 # input gradient, two classes at a time
    ("tight_s3", 1, 10, 41, 1, 7, 6, 5, 3, 0),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", TIGHT, ids=[c[0] for c in TIGHT])
def test_filters_without_padding_match_oracle(case, dtype):
    test_mfma16_group_conv_matches_oracle(case, wl.NCHW, dtype)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
def test_infinity_stays_inside_its_group(layout, dtype):
    """Four channels a group: 16 outputs of an instruction span four groups.  An infinity and a NaN in one channel must leave
    every other group's outputs as they are."""
    case = ("cg4_s2", 2, 32, 32, 8, 21, 23, 3, 2, 1)
    name, N, C, O, G, H, W, K, s, p = case
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=78)
    clean = [gu.to_host(t) for t in run_gpu(case, layout, dtype, x, w, dy)]
    x2, dy2 = x.copy(), dy.copy()
    at = (lambda a, n, c, h, v: a[n, c, h].__setitem__(4, v)) if layout == wl.NCHW else (lambda a, n, c, h, v: a[n, h, 4].__setitem__(c, v))
    at(x2, 1, 9, 7, np.inf); at(x2, 1, 10, 7, np.nan); at(dy2, 0, 17, 5, np.inf)
    got = [gu.to_host(t) for t in run_gpu(case, layout, dtype, x2, w, dy2)]
    for k, group in ((0, 2), (1, 4)):
        ch = 1 if layout == wl.NCHW else 3
        a, b = np.moveaxis(got[k], ch, 0), np.moveaxis(clean[k], ch, 0)
        others = [c for c in range(32) if c // 4 != group]
        assert np.isfinite(a[others]).all()
        gu.assert_close(a[others], b[others], 1e-6 if dtype == wl.F32 else gu.TOL_BF16, "other groups")
        assert not np.isfinite(a[4 * group:4 * group + 4]).all()


# A block of the forward and input-gradient kernels takes at most 256 positions x 16 outputs a tile and a launch has at most 2048
# blocks, so above 2^23 outputs a block has several tiles: the filter stays, the pixels are staged over the last tile's.
SEVERAL = [
    ("tiles_cg8", 12, 256, 256, 32, 53, 53, 3, 1, 2),
    ("tiles_cg16", 12, 256, 256, 16, 53, 53, 3, 1, 2),             # whole 16-channel blocks: no zeros between groups
    ("tiles_cg4_s2", 16, 500, 500, 125, 66, 66, 3, 2, 1),
]


def check_several(case, layout, dtype, plant):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    names = [dw.gconv_variant_name(d, i) for i in range(3)]
    print("case", name, layout, dtype, plant, names, flush=True)
    assert names[:2] == ["group_mfma16", "group_mfma16_bwd_data"]
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=80)
    assert min(x.size, dy.size) > 1 << 23
    w = w.copy()
    for o, ci, kh, kw, v in plant:
        w[(o, ci, kh, kw) if layout == wl.NCHW else (kh, kw, ci, o)] = v
    y, dx, _ = run_gpu(case, layout, dtype, x, w, dy)
    kw = dict(K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    tol = gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16
    for what, got, ref in (("fwd ", gu.to_host(y), og.fwd(x, w, **kw)), ("bwd_data ", gu.to_host(dx), og.bwd_data(dy, w, x_shape=x.shape, **kw))):
        assert (np.isnan(got) == np.isnan(ref)).all() and (np.isinf(got) == np.isinf(ref)).all(), what + name
        m = np.isfinite(ref)
        assert m.all() != bool(plant)
        gu.assert_close(np.where(m, got, 0), np.where(m, ref, 0), tol, what + name)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", SEVERAL, ids=[c[0] for c in SEVERAL])
def test_several_tiles_per_block(case, layout, dtype):
    check_several(case, layout, dtype, ())


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", SEVERAL[:2], ids=[c[0] for c in SEVERAL[:2]])
def test_several_tiles_per_block_beside_a_non_finite_filter(case, layout, dtype):
    """Every tile of a block whose filter holds an infinity or NaN goes one output at a time, from pixels that the whole block staged."""
    check_several(case, layout, dtype, ((1, 2, 0, 0, np.inf), (20, 5, 2, 1, -np.inf), (250, 0, 1, 1, np.nan)))


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
def test_several_tiles_per_block_of_the_filter_gradient(layout, dtype):
    """Partials take at most 16 MiB: 28 of them at 64 channels a group, against 32 tiles of at most 256 positions."""
    case = ("filter_tiles", 4, 256, 256, 4, 43, 43, 3, 1, 2)
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    print("case", name, layout, dtype, dw.gconv_variant_name(d, 2), flush=True)
    assert dw.gconv_variant_name(d, 2) == "group_mfma16_bwd_filter"
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=81)
    assert dw.gconv_bwd_filter_workspace_bytes(d) // (w.size * 4) * 256 < dy.size // O
    _, _, dwt = run_gpu(case, layout, dtype, x, w, dy)
    ref = og.bwd_filter(x, dy, K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    gu.assert_close(gu.to_host(dwt), ref, gu.TOL_F32_FILTER, "bwd_filter " + name)

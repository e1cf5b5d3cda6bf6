"""The filter gradient of short launches in one kernel, against the CPU oracles: every filter size, strides, paddings, multipliers and group sizes, fewer and
more positions than lanes, pairs that are no whole number of wavefronts; infinities beside the padding.  A sum has up to 4 thousand products here
(fp32: sqrt(4000) * 2^-24 = 4e-6 of the rms term sum, inside 1e-4).  Then the kernels that take the same layers in longer launches (and that tests of
small layers ran before there was this one), with it switched off."""
import numpy as np
import pytest

import oracle
import paper_1803_09926_amd as dw
from oracle import gconv as og
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu
import test_gpu_flat
import test_gpu_flat_pairs
import test_gpu_gconv
import test_gpu_nhwc_any
import test_gpu_parity
import test_gpu_reduce
from test_gpu_nonfinite import assert_same, plant

pytestmark = pytest.mark.gpu
BOTH = pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
DTYPE = pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])


@pytest.fixture
def short():
    with dw.tuning_overrides({"DWCONV_TUNE_SHORT": 1}):
        yield


@pytest.fixture
def no_short():
    with dw.tuning_overrides({"DWCONV_TUNE_SHORT": 0}):
        yield


# N, Layer: C, H, W, K, stride, pad, mult
LAYERS = [
    (1, Layer("one_position", 5, 3, 3, 3, 1, 0)),
    (1, Layer("positions_64", 9, 8, 8)),                               # NCHW: a wavefront a pair
    (1, Layer("positions_65", 9, 13, 5)),
    (2, Layer("positions_256_many", 1100, 8, 16)),                     # NCHW: a wavefront a pair; NHWC: 16 pairs of a wavefront
    (3, Layer("odd", 13, 17, 19)),
    (2, Layer("s2_even", 22, 20, 16, 3, 2, 1)),
    (2, Layer("s3_pad0", 6, 22, 25, 3, 3, 0)),
    (2, Layer("pad_3", 7, 9, 8, 3, 1, 3)),                             # rows and columns of padding alone
    (2, Layer("m2", 6, 11, 14, 3, 1, 1, 2)),
    (2, Layer("m3_s2", 5, 15, 12, 3, 2, 1, 3)),
    (2, Layer("k5", 10, 14, 23, 5, 1, 2)),
    (3, Layer("k5_s2_pad0", 33, 13, 12, 5, 2, 0)),
    (2, Layer("k7", 12, 16, 15, 7, 1, 3)),
    (1, Layer("k7_s2", 260, 19, 18, 7, 2, 3)),
    (70, Layer("images", 8, 7, 7)),
]
# name, N, C, O, groups, H, W, K, stride, pad
GROUPS = [
    ("cg2", 2, 10, 10, 5, 13, 12, 3, 1, 1),
    ("cg4_og3", 3, 16, 12, 4, 11, 14, 3, 2, 1),
    ("cg3_og8", 1, 9, 24, 3, 12, 9, 5, 1, 2),
    ("cg32", 2, 64, 64, 2, 7, 8, 3, 1, 1),
    ("dense_k7", 1, 6, 10, 1, 9, 11, 7, 1, 3),
    ("cg8_s3", 2, 24, 24, 3, 16, 17, 5, 3, 1),
]


def _filter_gradient(d, layer, N, layout, dtype, x, dy):
    """dw through the entry point, from a workspace and an output that hold NaNs."""
    import torch
    xt, dyt = gu.to_dev(x, dtype), gu.to_dev(dy, dtype)
    shape = (layer.O, layer.K, layer.K) if layout == wl.NCHW else (layer.K, layer.K, layer.O)
    g = torch.full(shape, float("nan"), device="cuda")
    ws = torch.full((dw.bwd_filter_workspace_bytes(d) // 4,), float("nan"), device="cuda")
    assert ws.numel() == g.numel()                                     # one partial
    return gu.to_host(dw.bwd_filter(d, xt, dyt, g, ws)), g


@DTYPE
@BOTH
@pytest.mark.parametrize("N,layer", LAYERS, ids=[l.name for _, l in LAYERS])
def test_depthwise(gpu_lib, short, N, layer, layout, dtype):
    x, w, dy = wl.make_inputs(layer, N, layout, dtype, 8500 + layer.C)
    d = gu.desc_for(layer, N, layout, dtype)
    print("case", layer, N, layout, dtype, flush=True)
    kw = dict(K=layer.K, stride=layer.stride, pad=layer.pad, mult=layer.mult, layout=layout, nthreads=8)
    got, g = _filter_gradient(d, layer, N, layout, dtype, x, dy)
    gu.assert_close(got, oracle.bwd_filter(x, dy, **kw), gu.TOL_F32_FILTER, layer.name)
    alone = dw.bwd_filter_noalloc(d, gu.to_dev(x, dtype), gu.to_dev(dy, dtype), g.clone())
    assert (gu.to_host(alone) == got).all()
    if 0 < layer.pad < layer.K and layer.C > 1 and layer.Ho > 1:
        for x2, dy2 in ((x, plant(dy, layout, 0, 1, 0, 0, np.inf)), (plant(x, layout, N - 1, 1, layer.H - 1, layer.W - 1, -np.inf), dy)):
            got, _ = _filter_gradient(d, layer, N, layout, dtype, x2, dy2)
            assert_same(got, oracle.bwd_filter(x2, dy2, **kw), gu.TOL_F32_FILTER, layer.name)


@DTYPE
@BOTH
@pytest.mark.parametrize("case", GROUPS, ids=[c[0] for c in GROUPS])
def test_group(gpu_lib, short, case, layout, dtype):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    print("case", name, layout, dtype, flush=True)
    assert dw.gconv_bwd_filter_workspace_bytes(d) == O * (C // G) * K * K * 4
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=98)
    ref = og.bwd_filter(x, dy, K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    _, _, dwt = test_gpu_gconv.run_gpu(case, layout, dtype, x, w, dy)
    gu.assert_close(gu.to_host(dwt), ref, gu.TOL_F32_FILTER, name)


def test_chosen_for_short_launches_alone(gpu_lib):
    for layout in (wl.NCHW, wl.NHWC):
        one = lambda *a: dw.bwd_filter_workspace_bytes(dw.desc(*a, layout=layout)) == a[1] * a[4] ** 2 * 4
        assert one(3, 32, 9, 9, 3) and not one(64, 256, 56, 56, 3)
        with dw.tuning_overrides({"DWCONV_TUNE_SHORT": 0}):
            assert not one(3, 32, 9, 9, 3)


@DTYPE
@pytest.mark.parametrize("N,layer", test_gpu_flat.CASES, ids=[l.name for _, l in test_gpu_flat.CASES])
def test_any_width_kernels(gpu_lib, no_short, N, layer, dtype):
    test_gpu_flat.test_any_width_kernels_match_oracle(gpu_lib, N, layer, dtype)


@pytest.mark.parametrize("case", test_gpu_flat_pairs.CASES, ids=[c[1].name for c in test_gpu_flat_pairs.CASES])
def test_column_pairs(gpu_lib, no_short, case):
    N, layer = case
    assert dw.variant_name(gu.desc_for(layer, N, wl.NCHW, wl.BF16), 2).startswith("nchw_flat_bwd_filter")
    test_gpu_flat_pairs.test_column_pairs(case)


@DTYPE
@pytest.mark.parametrize("N,layer", test_gpu_nhwc_any.CASES, ids=[l.name for _, l in test_gpu_nhwc_any.CASES])
def test_any_channel_walks(gpu_lib, no_short, N, layer, dtype):
    test_gpu_nhwc_any.test_any_channel_walks_match_oracle(gpu_lib, N, layer, dtype)


@DTYPE
@BOTH
@pytest.mark.parametrize("N,layer", test_gpu_parity.AWKWARD, ids=[l.name for _, l in test_gpu_parity.AWKWARD])
def test_awkward_shapes(gpu_lib, no_short, N, layer, layout, dtype):
    test_gpu_parity.test_awkward_shapes_match_oracle(gpu_lib, N, layer, layout, dtype)


@DTYPE
@pytest.mark.parametrize("layout,N,layer", test_gpu_reduce.CASES, ids=[c[2].name for c in test_gpu_reduce.CASES])
def test_second_stage(gpu_lib, no_short, layout, N, layer, dtype):
    test_gpu_reduce.test_second_stage_matches_oracle(gpu_lib, layout, N, layer, dtype)


@DTYPE
@BOTH
@pytest.mark.parametrize("case", test_gpu_gconv.CASES, ids=[c[0] for c in test_gpu_gconv.CASES])
def test_group_walks(gpu_lib, no_short, case, layout, dtype):
    """(a tuning snapshot also leaves the walks the short launches that the 16x16 matrix instructions take otherwise)"""
    test_gpu_gconv.test_group_conv_matches_oracle(case, layout, dtype)

"""Infinities and NaNs beside the padding: a padded tap is no product, so that an infinite filter entry or dy value at the edge of an
image, or an infinite x value in its last row or column, leaves the results that it has no part in finite.  Every element is compared
with the CPU oracle: the same class (finite, +inf, -inf, NaN), and where finite the same value within the tolerance of gpu_util."""
import numpy as np
import pytest
import torch

import oracle
import oracle.gconv as og
import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu
from test_gpu_gconv_gemm import run_gpu

pytestmark = pytest.mark.gpu

LAYERS = [
    (wl.NCHW, 2, Layer("nchw_k3_odd", 11, 37, 37)),
    (wl.NCHW, 2, Layer("nchw_k3_s2", 11, 37, 75, 3, 2, 1)),
    (wl.NCHW, 2, Layer("nchw_k5_odd", 12, 41, 41, 5, 1, 2)),
    (wl.NCHW, 2, Layer("nchw_k5_s2", 12, 56, 55, 5, 2, 2)),
    (wl.NCHW, 3, Layer("nchw_k7", 24, 28, 29, 7, 1, 3)),
    (wl.NCHW, 2, Layer("nchw_m2", 10, 37, 37, 3, 1, 1, 2)),
    (wl.NHWC, 2, Layer("nhwc_k3_any", 30, 41, 40)),
    (wl.NHWC, 2, Layer("nhwc_k3_s2_odd", 33, 41, 40, 3, 2, 1)),
    (wl.NHWC, 2, Layer("nhwc_k5_s2", 32, 57, 56, 5, 2, 2)),
    (wl.NHWC, 2, Layer("nhwc_k7", 92, 28, 28, 7, 1, 3)),               # 4508 filter entries: four a lane in the second stage
    (wl.NHWC, 2, Layer("nhwc_m2_s2", 30, 40, 41, 3, 2, 1, 2)),
    (wl.NHWC, 1, Layer("nhwc_rows_in_parts", 64, 4, 278, 5, 1, 1)),    # partials of parts of a row
]
GROUPS = [("cg16", 2, 64, 64, 4, 14, 15, 3, 1, 1), ("cg16_s2", 2, 64, 64, 4, 28, 27, 3, 2, 1), ("cg8_s2", 2, 32, 32, 4, 21, 23, 3, 2, 1)]


def classes(a):
    a = np.asarray(a, dtype=np.float64)
    return np.where(np.isnan(a), 2, np.where(np.isinf(a), np.sign(a), 0.5))


def assert_same(got, ref, tol, what):
    cg, cr = classes(got), classes(ref)
    assert (cg == cr).all(), "%s: %d elements of another class" % (what, (cg != cr).sum())
    assert (cr != 0.5).any() and (cr == 0.5).any(), what + ": nothing to tell"
    m = cr == 0.5
    gu.assert_close(np.where(m, got, 0), np.where(m, ref, 0), tol, what)


def plant(a, layout, n, c, h, w, value):
    a = a.copy()
    a[(n, c, h, w) if layout == wl.NCHW else (n, h, w, c)] = value
    return a


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout,N,layer", LAYERS, ids=[c[2].name for c in LAYERS])
def test_padding_is_no_product(gpu_lib, layout, N, layer, dtype):
    d = gu.desc_for(layer, N, layout, dtype)
    print("case", layer, N, dtype, [dw.variant_name(d, i) for i in range(3)], flush=True)
    x, w, dy = wl.make_inputs(layer, N, layout, dtype, 8400 + layer.C)
    kw = dict(K=layer.K, stride=layer.stride, pad=layer.pad, mult=layer.mult, layout=layout, nthreads=8)
    tol = gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16
    w2 = w.copy()
    for o, kh, kwi, v in ((1, 0, 0, np.inf), (4, layer.K - 1, 1, -np.inf), (6, 1, layer.K - 1, np.nan)):
        w2[(o, kh, kwi) if layout == wl.NCHW else (kh, kwi, o)] = v
    dev = lambda *a: [gu.to_dev(t, dtype) for t in a]
    y, dx, _ = gu.gpu_passes(layer, N, layout, dtype, *dev(x, w2, dy))
    assert_same(gu.to_host(y), oracle.fwd(x, w2, **kw), tol, "fwd " + layer.name)
    assert_same(gu.to_host(dx), oracle.bwd_data(dy, w2, x_shape=x.shape, **kw), tol, "bwd_data " + layer.name)
    for what, x2, dy2 in (("dy in the first corner", x, plant(dy, layout, 0, 2, 0, 0, np.inf)),
                          ("dy in the last corner", x, plant(dy, layout, N - 1, 3, layer.Ho - 1, layer.Wo - 1, -np.inf)),
                          ("x in the last corner", plant(x, layout, 0, 1, layer.H - 1, layer.W - 1, np.inf), dy),
                          ("x in the first corner", plant(x, layout, N - 1, 1, 0, 0, np.inf), dy)):
        _, _, dwt = gu.gpu_passes(layer, N, layout, dtype, *dev(x2, w, dy2))
        assert_same(gu.to_host(dwt), oracle.bwd_filter(x2, dy2, **kw), gu.TOL_F32_FILTER, "bwd_filter " + layer.name + ", " + what)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout,N,layer", LAYERS, ids=[c[2].name for c in LAYERS])
def test_padding_is_no_product_in_the_kernels_of_longer_launches(gpu_lib, layout, N, layer, dtype):
    """The same layers without the one-launch filter gradient and with two channels a lane in the any-channel walks: kernels that do multiply with
    the padding, and a second stage that adds entries up again."""
    with dw.tuning_overrides({"DWCONV_TUNE_SHORT": 0, "DWCONV_TUNE_ANY_V": 2}):
        d = gu.desc_for(layer, N, layout, dtype)
        assert dw.bwd_filter_workspace_bytes(d) > layer.O * layer.K ** 2 * 4               # several partials
        test_padding_is_no_product(gpu_lib, layout, N, layer, dtype)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [wl.NCHW, wl.NHWC], ids=["nchw", "nhwc"])
@pytest.mark.parametrize("case", GROUPS, ids=[c[0] for c in GROUPS])
def test_padding_is_no_product_in_a_group(gpu_lib, case, layout, dtype):
    with dw.tuning_overrides({"DWCONV_TUNE_GROUP_GEMM": 1}):               # the matrix instructions also where a small launch is shorter without
        check_group(case, layout, dtype)


def check_group(case, layout, dtype):
    name, N, C, O, G, H, W, K, s, p = case
    d = dw.group_desc(N, C, H, W, K, s, p, G, O, layout, dtype)
    print("case", name, layout, dtype, [dw.gconv_variant_name(d, i) for i in range(3)], flush=True)
    if not all(dw.gconv_variant_name(d, i).startswith("group_mfma16") for i in range(3)):
        pytest.skip("not these kernels")
    x, w, dy = wl.make_group_inputs(N, C, O, G, H, W, K, s, p, layout, dtype, seed=79)
    kw = dict(K=K, stride=s, pad=p, groups=G, O=O, layout=layout, nthreads=8)
    tol = gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16
    w2 = w.copy()
    for o, ci, kh, kwi, v in ((1, 2, 0, 0, np.inf), (20, 5, 2, 1, -np.inf)):
        w2[(o, ci, kh, kwi) if layout == wl.NCHW else (kh, kwi, ci, o)] = v
    y, dx, _ = run_gpu(case, layout, dtype, x, w2, dy)
    assert_same(gu.to_host(y), og.fwd(x, w2, **kw), tol, "fwd " + name)
    assert_same(gu.to_host(dx), og.bwd_data(dy, w2, x_shape=x.shape, **kw), tol, "bwd_data " + name)
    Ho, Wo = (dy.shape[2], dy.shape[3]) if layout == wl.NCHW else (dy.shape[1], dy.shape[2])
    for what, x2, dy2 in (("dy", x, plant(dy, layout, 1, 17, 0, Wo - 1, np.inf)), ("x", plant(x, layout, 0, 3, H - 1, W - 1, np.inf), dy)):
        _, _, dwt = run_gpu(case, layout, dtype, x2, w, dy2)
        assert_same(gu.to_host(dwt), og.bwd_filter(x2, dy2, **kw), gu.TOL_F32_FILTER, "bwd_filter " + name + ", " + what)


SLOW = [
    (wl.NCHW, Layer("nchw_k3_odd", 64, 147, 147)),
    (wl.NCHW, Layer("nchw_k5_odd", 64, 75, 75, 5, 1, 2)),
    (wl.NHWC, Layer("nhwc_k5_s2", 64, 112, 112, 5, 2, 2)),
    (wl.NHWC, Layer("nhwc_k7", 64, 57, 57, 7, 1, 3)),
]


@pytest.mark.parametrize("layout,layer", SLOW, ids=[c[1].name for c in SLOW])
@pytest.mark.parametrize("what", ["every value a NaN", "one infinity a channel", "one infinity a channel and image", "every value an infinity"])
def test_an_overflowed_step_is_no_stall(gpu_lib, layout, layer, what):
    """The filter gradient of an overflowed step: as many milliseconds as the one-output-per-thread kernels would take at most (5 to
    50 times the finite step), not the hundreds that adding every entry up again from all of dy takes."""
    N = 32
    d = gu.desc_for(layer, N, layout, wl.F32)
    print("case", layer, what, dw.variant_name(d, 2), flush=True)
    x, w, dy = wl.make_inputs_device(layer, N, layout, wl.F32, 85)
    ws = torch.empty(dw.bwd_filter_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    dwt = torch.empty(w.shape, device="cuda")

    def ms(dy):
        dw.bwd_filter(d, x, dy, dwt, ws)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(); dw.bwd_filter(d, x, dy, dwt, ws); b.record(); b.synchronize()
        return a.elapsed_time(b)
    finite = ms(dy)
    assert torch.isfinite(dwt).all()
    bad = dy.clone()
    if what.startswith("every value"):
        bad[:] = float("nan") if "NaN" in what else float("inf")
    else:
        v = bad if "image" in what else bad[N // 2:N // 2 + 1]
        (v[:, :, 20, 30] if layout == wl.NCHW else v[:, 20, 30, :])[:] = float("inf")
    taken = ms(bad)
    print("finite %.3f ms, %s %.3f ms" % (finite, what, taken), flush=True)
    assert not torch.isfinite(dwt).any()
    assert taken < 10 + 50 * finite

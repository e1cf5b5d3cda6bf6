"""GPU parity of the bf16 3x3 walk on column pairs (rows of any even width) against the CPU oracle, element by element: whole planes and
bands, the narrowest rows it takes, rows of more than a wavefront, a last group of planes that is not full, multiplier 2 (forward); and the classes
of infinities and NaNs beside the padding, in the halves of the words that a lane does not use and in the filter."""
import numpy as np
import pytest

import oracle
import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu

# batch, layer
CASES = [
    (16, Layer("bands", 57, 74, 74, 3, 1, 1, 1)),
    (32, Layer("whole_planes", 61, 18, 38, 3, 1, 1, 1)),
    (33, Layer("one_row", 45, 1, 46, 3, 1, 1, 1)),
    (33, Layer("two_rows", 45, 2, 46, 3, 1, 1, 1)),
    (20, Layer("wide", 13, 19, 302, 3, 1, 1, 1)),                  # lanes of a row over several wavefronts
    (2, Layer("widest", 65, 5, 510, 3, 1, 1, 1)),
    (25, Layer("multiplier", 31, 39, 50, 3, 1, 1, 2)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[1].name for c in CASES])
def test_column_pairs(case):
    N, layer = case
    assert N * layer.O * (layer.W // 2) >= 32768 and layer.W >= 36
    d = gu.desc_for(layer, N, wl.NCHW, wl.BF16)
    print("case", layer.name, [dw.variant_name(d, i) for i in range(3)], flush=True)
    assert dw.variant_name(d, 0) == "nchw_flat_k3s1"
    gu.check_layer_full(layer, N, wl.NCHW, wl.BF16, seed=71)


def test_infinities_in_unused_halves():
    N, layer = 60, Layer("nonfinite", 30, 21, 50, 3, 1, 1, 1)
    x, w, dy = (a.copy() for a in wl.make_inputs(layer, N, wl.NCHW, wl.BF16, 72))
    x[0, 0, 0, 0] = np.inf; x[1, 1, 20, 49] = np.nan; x[0, 2, 15, 7] = -np.inf; x[0, 2, 18, 8] = np.nan
    dy[0, 3, 0, 49] = np.inf; dy[1, 3, 20, 0] = -np.inf; dy[0, 3, 10, 11] = np.nan
    w[4, 0, 2] = np.inf; w[5, 1, 1] = np.nan
    print("case", layer.name, flush=True)
    y, dx, _ = gu.gpu_passes(layer, N, wl.NCHW, wl.BF16, gu.to_dev(x, wl.BF16), gu.to_dev(w, wl.BF16), gu.to_dev(dy, wl.BF16))
    kw = dict(K=3, stride=1, pad=1, mult=1, layout=wl.NCHW, nthreads=8)
    for got, ref in ((gu.to_host(y), oracle.fwd(x, w, **kw)), (gu.to_host(dx), oracle.bwd_data(dy, w, x_shape=x.shape, **kw))):
        assert (np.isnan(got) == np.isnan(ref)).all() and (np.isinf(got) == np.isinf(ref)).all()
        m = np.isfinite(ref)
        assert not m.all()
        gu.assert_close(np.where(m, got, 0), np.where(m, ref, 0), gu.TOL_BF16, "finite part")


# The filter gradient takes pairs from rows of 64 on; with a multiplier several planes of dy meet one of x.  Planes of more than 40 KiB are bands, whose
# dy is in LDS beside them; of fewer rows the lanes read it.
FILTER_CASES = [
    (4, Layer("m2_bands", 64, 170, 130, 3, 1, 1, 2)),
    (4, Layer("m3_bands", 43, 170, 130, 3, 1, 1, 3)),
    (11, Layer("m2_few_rows", 15, 3, 200, 3, 1, 1, 2)),
    (10, Layer("m3_few_rows", 11, 4, 200, 3, 1, 1, 3)),
    (16, Layer("m2_narrowest", 33, 13, 64, 3, 1, 1, 2)),
    (6, Layer("m1_bands", 91, 170, 130, 3, 1, 1, 1)),
]


@pytest.mark.parametrize("case", FILTER_CASES, ids=[c[1].name for c in FILTER_CASES])
def test_filter_gradient_on_pairs(case):
    N, layer = case
    assert N * layer.O * (layer.W // 2) >= 32768 and layer.W >= 64
    d = gu.desc_for(layer, N, wl.NCHW, wl.BF16)
    print("case", layer.name, [dw.variant_name(d, i) for i in range(3)], flush=True)
    assert dw.variant_name(d, 2) == "nchw_flat_bwd_filter_k3s1"
    gu.check_layer_full(layer, N, wl.NCHW, wl.BF16, seed=73)


# Two columns a lane are rows of up to 1024: beyond 512 the passes on pairs (with a multiplier not the input gradient) and the generic kernels
# for the others.
WIDE_CASES = [
    (3, Layer("first", 43, 5, 514, 3, 1, 1, 1)),
    (2, Layer("middle", 49, 9, 702, 3, 1, 1, 1)),
    (2, Layer("last", 33, 2, 1022, 3, 1, 1, 1)),
    (2, Layer("bands", 33, 61, 1022, 3, 1, 1, 1)),
    (2, Layer("multiplier", 29, 7, 638, 3, 1, 1, 2)),
    (1, Layer("too_few", 5, 7, 638, 3, 1, 1, 1)),                  # a short launch: generic
    (2, Layer("odd", 65, 5, 515, 3, 1, 1, 1)),
]


@pytest.mark.parametrize("case", WIDE_CASES, ids=[c[1].name for c in WIDE_CASES])
def test_rows_of_more_than_512(case):
    N, layer = case
    d = gu.desc_for(layer, N, wl.NCHW, wl.BF16)
    names = [dw.variant_name(d, i) for i in range(3)]
    print("case", layer.name, names, flush=True)
    flat = ["nchw_flat_k3s1", "nchw_flat_k3s1_flip" if layer.mult == 1 else "generic", "nchw_flat_bwd_filter_k3s1"]
    assert names == (flat if layer.W % 2 == 0 and N * layer.O * (layer.W // 2) >= 32768 else ["generic"] * 3)
    gu.check_layer_full(layer, N, wl.NCHW, wl.BF16, seed=74)


@pytest.mark.parametrize("H", [21, 301], ids=["dy_by_lanes", "dy_in_lds"])
def test_filter_gradient_beside_infinities(H):
    N, layer = (34, Layer("nonfinite", 29, 21, 70, 3, 1, 1, 1)) if H == 21 else (32, Layer("nonfinite", 30, 301, 70, 3, 1, 1, 1))
    assert N * layer.O * (layer.W // 2) >= 32768
    x, w, dy = (a.copy() for a in wl.make_inputs(layer, N, wl.NCHW, wl.BF16, 75))
    x[0, 0, 0, 0] = np.inf; x[1, 1, H - 1, 69] = np.nan; x[0, 2, 15, 7] = -np.inf; x[0, 2, 18, 8] = np.nan; x[2, 6, 0, 69] = -np.inf
    dy[0, 3, 0, 69] = np.inf; dy[1, 3, H - 1, 0] = -np.inf; dy[0, 4, 10, 11] = np.nan; dy[3, 5, H - 1, 40] = np.inf
    print("case", layer.name, H, flush=True)
    _, _, g = gu.gpu_passes(layer, N, wl.NCHW, wl.BF16, gu.to_dev(x, wl.BF16), gu.to_dev(w, wl.BF16), gu.to_dev(dy, wl.BF16))
    got, ref = gu.to_host(g), oracle.bwd_filter(x, dy, K=3, stride=1, pad=1, mult=1, layout=wl.NCHW, nthreads=8)
    assert (np.isnan(got) == np.isnan(ref)).all() and (np.isinf(got) == np.isinf(ref)).all()
    m = np.isfinite(ref)
    assert not m.all()
    gu.assert_close(np.where(m, got, 0), np.where(m, ref, 0), gu.TOL_F32_FILTER, "finite part")

"""GPU parity of the fused backward pass on rows of any width (3x3, stride 1, "same" padding, multiplier 1) against the CPU oracle,
element by element: whole planes and bands, several planes and items a block, a last group of planes that is not full, rows of one
wavefront and more, planes of one band's rows and of fewer rows than are prefetched; and the classes of infinities and NaNs in x, dy and
the filter, which the zeros of the padding must not turn into NaNs."""
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
    (3, Layer("whole_planes", 29, 19, 19, 3, 1, 1, 1)),
    (2, Layer("bands", 7, 74, 74, 3, 1, 1, 1)),
    (1, Layer("one_plane", 1, 21, 17, 3, 1, 1, 1)),
    (5, Layer("few_rows", 13, 4, 37, 3, 1, 1, 1)),                 # fewer rows than are on their way
    (2, Layer("two_rows", 9, 2, 90, 3, 1, 1, 1)),
    (2, Layer("wide", 3, 33, 301, 3, 1, 1, 1)),                    # blocks of more than 256 lanes
    (40, Layer("several_items", 70, 15, 15, 3, 1, 1, 1)),
    (2, Layer("tall", 5, 301, 9, 3, 1, 1, 1)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[c[1].name for c in CASES])
def test_fused_backward_on_rows_of_any_width(case, dtype):
    N, layer = case
    d = gu.desc_for(layer, N, wl.NCHW, dtype)
    print("case", layer.name, dtype, dw.variant_name(d, 3), flush=True)
    assert dw.variant_name(d, 3) == "nchw_flat_bwd_fused_k3s1"
    gu.check_layer_full(layer, N, wl.NCHW, dtype, seed=61)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
def test_infinities_beside_the_padding(dtype):
    N, layer = 2, Layer("nonfinite", 6, 45, 51, 3, 1, 1, 1)
    assert dw.variant_name(gu.desc_for(layer, N, wl.NCHW, dtype), 3) == "nchw_flat_bwd_fused_k3s1"
    x, w, dy = (a.copy() for a in wl.make_inputs(layer, N, wl.NCHW, dtype, 62))
    x[0, 0, 0, 0] = np.inf; x[1, 1, 44, 50] = np.nan; x[0, 2, 20, 0] = -np.inf
    dy[0, 3, 0, 50] = np.inf; dy[1, 3, 44, 0] = -np.inf
    w[4, 0, 2] = np.inf; w[5, 1, 1] = np.nan
    print("case", layer.name, dtype, flush=True)
    dx, g = gu.gpu_bwd(layer, N, wl.NCHW, dtype, gu.to_dev(x, dtype), gu.to_dev(w, dtype), gu.to_dev(dy, dtype))
    kw = dict(K=3, stride=1, pad=1, mult=1, layout=wl.NCHW, nthreads=8)
    for got, ref, tol in ((gu.to_host(dx), oracle.bwd_data(dy, w, x_shape=x.shape, **kw), gu.TOL_F32 if dtype == wl.F32 else gu.TOL_BF16),
                          (gu.to_host(g), oracle.bwd_filter(x, dy, **kw), gu.TOL_F32_FILTER)):
        assert (np.isnan(got) == np.isnan(ref)).all() and (np.isinf(got) == np.isinf(ref)).all()
        m = np.isfinite(ref)
        assert not m.all()
        gu.assert_close(np.where(m, got, 0), np.where(m, ref, 0), tol, "finite part")

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

"""GPU parity of the NCHW row walk that takes both outputs of a channel (multiplier 2, 3x3, launches of 65536 lanes and more; filter
gradient: 1024 blocks) against the CPU oracle, element by element: row groups of two and four for the whole-line write-out, rows
that are whole lines, rows of 8-byte vectors, heights that leave a short last strip, and fp32 rows of one vector, which only the
whole-line write-out takes that way."""
import pytest

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu

# batch, layer
CASES = [
    (16, Layer("rows56", 96, 56, 56, 3, 1, 1, 2)),                 # groups of four rows
    (9, Layer("rows112", 48, 112, 112, 3, 1, 1, 2)),               # groups of two; lanes past the last plane
    (24, Layer("whole_lines", 128, 37, 32, 3, 1, 1, 2)),           # stored as they are
    (20, Layer("short_vectors", 96, 45, 44, 3, 1, 1, 2)),          # bf16: four columns a lane
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[c[1].name for c in CASES])
def test_both_outputs_of_a_channel(case, dtype):
    N, layer = case
    d = gu.desc_for(layer, N, wl.NCHW, dtype)
    print("case", layer.name, dtype, [dw.variant_name(d, i) for i in range(3)], flush=True)
    gu.check_layer_full(layer, N, wl.NCHW, dtype, seed=51)


# The launches above are large enough in fp32 (short strips).  These are whatever the strips: a lane for every vector of a row and plane of x.
# type, vector, batch, layer
WIDE = [
    (wl.BF16, 8, 36, Layer("rows56", 261, 16, 56, 3, 1, 1, 2)),             # bf16: groups of four rows
    (wl.BF16, 8, 64, Layer("rows32", 257, 16, 32, 3, 1, 1, 2)),             # groups of two
    (wl.BF16, 8, 100, Layer("rows40", 132, 17, 40, 3, 1, 1, 2)),            # stored as they are
    (wl.BF16, 4, 38, Layer("rows60", 115, 17, 60, 3, 1, 1, 2)),             # vectors of four columns
    (wl.F32, 4, 33, Layer("rows56", 146, 16, 56, 3, 1, 1, 2)),
    (wl.F32, 4, 205, Layer("rows4", 320, 16, 4, 3, 1, 1, 2)),               # one vector a row: groups of four rows
    (wl.F32, 4, 205, Layer("rows4_odd", 320, 19, 4, 3, 1, 1, 2)),          # and stored by themselves
]


@pytest.mark.parametrize("case", WIDE, ids=["%s_%s" % (c[3].name, "f32" if c[0] == wl.F32 else "bf16") for c in WIDE])
def test_both_outputs_whatever_the_strips(case):
    dtype, V, N, layer = case
    assert N * layer.C * (layer.W // V) >= 65536
    d = gu.desc_for(layer, N, wl.NCHW, dtype)
    print("case", layer.name, dtype, dw.variant_name(d, 0), flush=True)
    assert dw.variant_name(d, 0) == "nchw_rowwalk_k3s1"
    gu.check_layer_full(layer, N, wl.NCHW, dtype, seed=52)

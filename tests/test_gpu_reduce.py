"""Second stage of the filter gradient: the partials of stage 1 summed four entries a lane (entry counts of 2048 and more that are
a multiple of four) and one a lane (the others), against the CPU oracle.  Tolerances as in gpu_util."""
import pytest

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [
    (wl.NHWC, 5, Layer("entries_2052", 228, 20, 20)),                  # just above the line, last block a quarter full
    (wl.NHWC, 5, Layer("entries_2043", 227, 20, 20)),                  # just below it and no multiple of four
    (wl.NHWC, 5, Layer("entries_2075", 83, 20, 20, 5, 1, 2)),          # above it, no multiple of four
    (wl.NCHW, 1, Layer("one_partial", 300, 14, 14)),
    (wl.NHWC, 70, Layer("many_partials", 512, 14, 14)),
    (wl.NHWC, 3, Layer("wide", 4096, 7, 7)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout,N,layer", CASES, ids=[c[2].name for c in CASES])
def test_second_stage_matches_oracle(gpu_lib, layout, N, layer, dtype):
    d = gu.desc_for(layer, N, layout, dtype)
    print("case", layer, N, dtype, dw.variant_name(d, 2), flush=True)
    gu.check_layer_full(layer, N, layout, dtype, seed=8300 + layer.C + dtype)

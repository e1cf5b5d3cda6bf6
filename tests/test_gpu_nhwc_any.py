"""GPU parity of the NHWC row walks for any channel count, padding and multiplier (3x3, 5x5, 7x7; stride 1 and 2) against the CPU
oracle, element by element, at the edges of their tiling.  Tolerances as in gpu_util."""
import pytest

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [
    (2, Layer("k5_s2", 128, 28, 27, 5, 2, 2)),
    (3, Layer("k5_s2_odd_c", 13, 29, 30, 5, 2, 2)),
    (2, Layer("k7", 64, 28, 28, 7, 1, 3)),
    (2, Layer("k7_c_even", 30, 17, 41, 7, 1, 3)),
    (2, Layer("k7_s2", 36, 31, 32, 7, 2, 3)),
    (2, Layer("c_odd", 211, 14, 14)),
    (2, Layer("c_two", 2, 40, 41)),
    (1, Layer("c_one", 1, 75, 74)),
    (2, Layer("c_odd_s2", 37, 41, 40, 3, 2, 1)),
    (2, Layer("k5_c_odd", 31, 20, 20, 5, 1, 2)),
    (2, Layer("pad0", 16, 30, 29, 3, 1, 0)),
    (2, Layer("pad0_s2", 16, 30, 29, 3, 2, 0)),
    (2, Layer("pad3_k3", 16, 12, 13, 3, 1, 3)),                       # rows and columns of pure padding
    (2, Layer("pad6_k5_s2", 10, 12, 13, 5, 2, 6)),
    (2, Layer("m2_k5", 24, 20, 21, 5, 1, 2, 2)),
    (2, Layer("m2_s2", 24, 20, 21, 3, 2, 1, 2)),
    (2, Layer("m2_k7_s2", 12, 33, 20, 7, 2, 3, 2)),
    (2, Layer("m3", 10, 16, 17, 3, 1, 1, 3)),                         # (its input gradient stays generic)
    (1, Layer("tall", 6, 300, 5, 5, 2, 2)),                           # many strips
    (1, Layer("wide", 6, 5, 700, 7, 1, 3)),
    (40, Layer("rows_of_7_lanes", 2, 30, 7, 7, 1, 3)),                # blocks of one wavefront, most of it idle
    (2, Layer("rows_of_300_lanes", 6, 20, 100)),                      # blocks of 192
    (1, Layer("rows_in_parts", 97, 4, 278, 5, 1, 2)),                 # one image, few rows: the filter gradient splits the columns
    (31, Layer("images_of_9", 66, 3, 3, 7, 1, 3)),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,layer", CASES, ids=[l.name for _, l in CASES])
def test_any_channel_walks_match_oracle(gpu_lib, N, layer, dtype):
    d = gu.desc_for(layer, N, wl.NHWC, dtype)
    print("case", layer, N, dtype, [dw.variant_name(d, i) for i in range(3)], flush=True)
    # (short filter gradients run one launch of another kernel; here again with that switched off: test_gpu_short_filter)
    assert dw.variant_name(d, 0).startswith("nhwc_any") and dw.variant_name(d, 2).startswith(("nhwc_any", "nhwc_short"))
    gu.check_layer_full(layer, N, wl.NHWC, dtype, seed=8200 + layer.C + dtype)


# 5x5 and 7x7 with two channels a lane: beyond the sizes below which a lane takes one, and forced in small layers at the edges of the tiling
LARGE = [
    (11, Layer("k7_above", 226, 28, 28, 7, 1, 3)),
    (10, Layer("k5_s2_above", 230, 57, 56, 5, 2, 2)),
]
TWO = [c for c in CASES if c[1].K > 3 and c[1].mult == 1 and c[1].C % 2 == 0]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,layer", LARGE, ids=[l.name for _, l in LARGE])
def test_launches_of_many_lanes_match_oracle(gpu_lib, N, layer, dtype):
    d = gu.desc_for(layer, N, wl.NHWC, dtype)
    print("case", layer, N, dtype, [dw.variant_name(d, i) for i in range(3)], flush=True)
    need = dw.bwd_filter_workspace_bytes(d)
    for channels, same in ((1, False), (2, True)):                    # the partials tell which of the two is planned
        with dw.tuning_overrides({"DWCONV_TUNE_ANY_V": channels}):
            assert (dw.bwd_filter_workspace_bytes(d) == need) == same
    gu.check_layer_full(layer, N, wl.NHWC, dtype, seed=8250 + dtype)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,layer", TWO, ids=[l.name for _, l in TWO])
def test_two_channels_a_lane_match_oracle(gpu_lib, N, layer, dtype):
    with dw.tuning_overrides({"DWCONV_TUNE_ANY_V": 2, "DWCONV_TUNE_SHORT": 0}):
        test_any_channel_walks_match_oracle(gpu_lib, N, layer, dtype)

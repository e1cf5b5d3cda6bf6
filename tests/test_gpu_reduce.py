"""Second stage of the filter gradient: the partials of stage 1 summed four entries a lane (entry counts of 2048 and more that are
a multiple of four) and one a lane (the others), against the CPU oracle.  Tolerances as in gpu_util."""
import pytest

import torch

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


# A lane takes one partial each (up to 16 of 8192 entries and more, 32 of 4096, 64 of fewer), so that all its additions are in 64 bits.
GROUPS = [(wl.NCHW, 1, 240, 30, 30), (wl.NHWC, 1, 64, 30, 8)]                          # layout, N, C, H, groups: short launches of the row walks
WALKS = [(8, Layer("k7", 64, 14, 14, 7, 1, 3)), (8, Layer("k5_s2", 100, 20, 20, 5, 2, 2))]


def _partials_in_64_bits(d, call, need, x, dy, w):
    """The gradient is the sum of the partials that stage 1 leaves in the workspace, rounded once."""
    J = w.numel()
    ws = torch.full((need // 4,), float("nan"), device="cuda")
    g = torch.full(w.shape, float("nan"), device="cuda")
    assert 3 <= ws.numel() // J <= (16 if J >= 8192 else 32 if J >= 4096 else 64) and J >= 2048 and J % 4 == 0
    call(d, x, dy, g, ws)
    total = ws.reshape(-1, J).double().sum(0)
    # (a sum of 64 32-bit numbers in 64 bits, in another order, is 2^-47 of the largest off: one entry in 2^20 may round the other way)
    assert (g.flatten() != total.float()).double().mean().item() < 1e-3


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout,N,C,H,groups", GROUPS, ids=["nchw", "nhwc"])
def test_partials_of_the_group_kernels_meet_in_64_bits(gpu_lib, layout, N, C, H, groups, dtype):
    d = dw.group_desc(N, C, H, H, 3, 1, 1, groups, C, layout, dtype)
    print("case", layout, N, C, H, groups, dtype, dw.gconv_variant_name(d, 2), flush=True)
    assert dw.gconv_variant_name(d, 2) == "group_mfma16_bwd_filter"
    x, w, dy = wl.make_inputs_device(Layer("l", C, H, H, 3, 1, 1, 1, C // groups), N, layout, dtype, 8400 + dtype)
    _partials_in_64_bits(d, dw.gconv_bwd_filter, dw.gconv_bwd_filter_workspace_bytes(d), x, dy, w)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,layer", WALKS, ids=[l.name for _, l in WALKS])
def test_partials_of_the_any_channel_walks_meet_in_64_bits(gpu_lib, N, layer, dtype):
    with dw.tuning_overrides({"DWCONV_TUNE_SHORT": 0}):
        d = gu.desc_for(layer, N, wl.NHWC, dtype)
        print("case", layer, N, dtype, dw.variant_name(d, 2), flush=True)
        assert dw.variant_name(d, 2).startswith("nhwc_any")
        x, w, dy = wl.make_inputs_device(layer, N, wl.NHWC, dtype, 8400 + dtype)
        _partials_in_64_bits(d, dw.bwd_filter, dw.bwd_filter_workspace_bytes(d), x, dy, w)

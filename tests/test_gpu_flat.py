"""GPU parity of the NCHW any-width kernels (rows of any number of elements; 3x3, 5x5 and 7x7; stride 1 and 2; any padding)
against the CPU oracle, element by element, at the edges of their tiling.  Tolerances as in gpu_util (fp32 sums of up to 49
products in the forward and input-gradient passes; the filter gradient in fp32 whatever the storage type)."""
import pytest

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl
from paper_1803_09926_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu

CASES = [
    (3, Layer("whole_planes_odd", 37, 19, 19)),                        # a tile of several planes ends inside an image
    (2, Layer("bands_short_last", 11, 75, 74)),                        # bands of unequal height, segments at every alignment
    (1, Layer("one_plane_per_block", 5, 41, 147)),
    (1, Layer("wide_rows", 3, 9, 509)),                                # more lanes than 256
    (2, Layer("row_of_one", 9, 31, 1)),
    (2, Layer("s2_odd_both", 13, 37, 37, 3, 2, 1)),
    (2, Layer("s2_even_rows_odd", 13, 38, 75, 3, 2, 1)),
    (2, Layer("s2_pad0", 7, 40, 41, 3, 2, 0)),
    (2, Layer("pad2_k3", 7, 21, 22, 3, 1, 2)),
    (2, Layer("pad_above_filter", 6, 10, 11, 3, 1, 5)),                # rows and columns of pure padding
    (2, Layer("pad_above_filter_s2", 6, 10, 11, 5, 2, 6)),
    (2, Layer("k5_41", 12, 41, 41, 5, 1, 2)),
    (2, Layer("k5_rowwalk_width", 6, 40, 48, 5, 1, 2)),
    (4, Layer("k5_s2_planes", 21, 15, 14, 5, 2, 2)),
    (2, Layer("k5_s2_bands", 9, 57, 56, 5, 2, 2)),
    (3, Layer("k7", 24, 28, 28, 7, 1, 3)),
    (4, Layer("k7_pad1", 24, 30, 29, 7, 1, 1)),
    (3, Layer("k7_s2", 24, 57, 31, 7, 2, 3)),
    (2, Layer("k7_large", 16, 60, 59, 7, 1, 3)),
    (2, Layer("k5_row_of_one", 9, 31, 1, 5, 1, 2)),                    # bf16: the second column of the only lane is none
    (2, Layer("k7_s2_even", 10, 32, 30, 7, 2, 3)),                     # 15 outputs a row: 8 lanes of two columns, the last half used
    (1, Layer("k5_wide_rows", 3, 9, 511, 5, 1, 2)),
    (2, Layer("s2_pad2", 9, 40, 43, 3, 2, 2)),                         # input gradient: column pairs of an even padding, odd width
    (2, Layer("k5_s2_pad1", 9, 40, 42, 5, 2, 1)),                      # and of an odd padding
    (2, Layer("k7_s2_pad2", 9, 33, 34, 7, 2, 2)),
    (2, Layer("wide_s2", 5, 60, 155, 3, 2, 1)),                        # dy from LDS in bands
    (2, Layer("m2", 10, 37, 37, 3, 1, 1, 2)),                          # output planes 2c and 2c + 1 read input plane c
    (2, Layer("m2_k5_s2", 10, 29, 31, 5, 2, 2, 2)),
    (2, Layer("m3", 7, 23, 22, 3, 1, 1, 3)),
    (5, Layer("m2_k7", 12, 20, 21, 7, 1, 3, 2)),
    (1, Layer("few_tall_k7", 3, 149, 33, 7, 1, 3)),                    # few blocks: bands of four rows
    (2, Layer("few_tall_s2", 2, 146, 147, 3, 2, 1)),
    (1, Layer("few_tall_k5_m2", 2, 131, 30, 5, 1, 2, 2)),
    (1, Layer("few_short", 2, 5, 130, 5, 1, 2)),                       # one band that is not cut
    (2, Layer("few_k7", 8, 9, 9, 7, 1, 3)),                            # the forward pass of any size, the filter gradient generic
    (1, Layer("one_output_k7", 256, 7, 7, 7, 1, 0)),
    (3, Layer("narrow_bands", 10, 104, 4, 5, 2, 2)),                   # rows too short to cut bands
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N,layer", CASES, ids=[l.name for _, l in CASES])
def test_any_width_kernels_match_oracle(gpu_lib, N, layer, dtype):
    d = gu.desc_for(layer, N, wl.NCHW, dtype)
    print("case", layer, N, dtype, [dw.variant_name(d, i) for i in range(3)], flush=True)
    if layer.name != "k5_rowwalk_width" or dtype == wl.F32:
        assert dw.variant_name(d, 0).startswith("nchw_flat"), dw.variant_name(d, 0)
    gu.check_layer_full(layer, N, wl.NCHW, dtype, seed=8100 + layer.C + dtype)


@pytest.mark.parametrize("N,layer,flat", [(16, Layer("above", 656, 20, 20), True), (16, Layer("below", 655, 20, 20), False),
                                          (16, Layer("rows_of_24", 656, 20, 24), False)], ids=lambda v: getattr(v, "name", str(v)))
def test_bf16_rows_of_odd_quads(gpu_lib, N, layer, flat):
    """From 2^22 outputs on the bf16 3x3 layers whose rows are no whole number of 16-byte vectors."""
    d = gu.desc_for(layer, N, wl.NCHW, wl.BF16)
    for i in range(2):
        assert dw.variant_name(d, i).startswith("nchw_flat") == flat, dw.variant_name(d, i)
    gu.check_layer_full(layer, N, wl.NCHW, wl.BF16, seed=8200 + layer.C)


def test_rows_above_512_stay_with_the_row_walk(gpu_lib):
    layer = Layer("k5_516", 3, 20, 516, 5, 1, 2)
    d = gu.desc_for(layer, 1, wl.NCHW, wl.F32)
    for i in range(3):
        assert dw.variant_name(d, i).startswith("nchw_rowwalk"), dw.variant_name(d, i)
    gu.check_layer_full(layer, 1, wl.NCHW, wl.F32, seed=8250)

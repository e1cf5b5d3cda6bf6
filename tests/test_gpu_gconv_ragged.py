"""GPU parity of the 16x16 group kernels where channels are no whole number of vectors (NHWC: unaligned loads that reach into the next pixel, at the
tensor's end shifted) and where tiles are narrower than the rows (NCHW: runs of four columns from the multiple of four before a tile).
Against the CPU group oracle, element by element; tolerances as in test_gpu_gconv_gemm."""
import pytest

import paper_1803_09926_amd as dw
from paper_1803_09926_amd import workloads as wl

from test_gpu_gconv_gemm import matrix_instructions, test_mfma16_group_conv_matches_oracle as against_oracle        # noqa: F401
from test_gpu_nonfinite import check_group

pytestmark = pytest.mark.gpu

# name, N, C, O, groups, H, W, K, stride, pad
RAGGED = [
    ("c10", 4, 10, 10, 5, 19, 17, 5, 1, 2),
    ("c22_s2", 3, 22, 22, 11, 23, 20, 3, 2, 1),
    ("c30_k5", 2, 30, 30, 15, 17, 21, 5, 1, 2),
    ("c12", 5, 12, 12, 3, 30, 27, 3, 2, 1),                        # whole vectors in fp32 only
    ("c15_o20", 3, 15, 20, 5, 18, 16, 3, 1, 1),                    # odd channels: loads at odd elements
    ("c9_o33", 2, 9, 33, 1, 15, 19, 5, 2, 2),                      # outputs end inside a quad
    ("c34_o6", 3, 34, 6, 2, 14, 18, 3, 1, 1),                      # more input channels than a chunk
    ("one_image", 1, 11, 15, 1, 15, 17, 3, 1, 1),
    ("k1", 3, 18, 26, 2, 21, 17, 1, 1, 0),
    ("pixels_of_two", 2500, 2, 2, 1, 1, 1, 5, 1, 2),               # a vector spans pixels and images
]
SPLIT = [
    ("w65", 2, 16, 16, 4, 9, 65, 3, 1, 1),
    ("w70_pad0", 2, 12, 12, 3, 11, 70, 3, 1, 0),
    ("w98_pad2", 1, 16, 24, 2, 10, 98, 3, 1, 2),
    ("w131_k5", 2, 10, 10, 5, 9, 131, 5, 1, 2),
    ("w150_s2", 2, 32, 32, 4, 13, 150, 3, 2, 1),
    ("w149_s2_k5", 1, 24, 24, 3, 14, 149, 5, 2, 2),
    ("w200_pad3", 1, 16, 16, 1, 8, 200, 3, 1, 3),
    ("w137_c10_o12", 2, 20, 24, 2, 12, 137, 3, 1, 1),
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", RAGGED, ids=[c[0] for c in RAGGED])
def test_ragged_channels(case, dtype):
    against_oracle(case, wl.NHWC, dtype)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", SPLIT, ids=[c[0] for c in SPLIT])
def test_tiles_narrower_than_the_rows(case, dtype):
    against_oracle(case, wl.NCHW, dtype)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout,case", [(wl.NHWC, ("c30", 2, 30, 30, 5, 26, 23, 3, 1, 1)), (wl.NCHW, ("w71", 2, 24, 24, 4, 13, 71, 3, 1, 1))],
                         ids=["ragged", "split"])
def test_infinities_stay_in_their_group(layout, case, dtype):
    check_group(case, layout, dtype)

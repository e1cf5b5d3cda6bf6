"""The group planner on the host at the ends of what the 16x16 kernels stage: a pixel of more vectors than a block has lanes, one input
pixel, filters of about a compute unit's LDS.  It must return, name a variant and keep the partials within 64 MiB."""
import pytest

import paper_1803_09926_amd as dw


@pytest.mark.parametrize("dtype", [dw.F32, dw.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("layout", [dw.NCHW, dw.NHWC], ids=["nchw", "nhwc"])
def test_group_planner_at_its_limits(layout, dtype):
    for C in (1000, 1024, 1040, 1288, 2048, 2064, 4096, 8192, 65536):
        for groups in (1, 2, 8):
            for K, s, p in ((1, 1, 0), (1, 2, 0), (3, 1, 1), (5, 2, 2), (7, 1, 3)):
                for H, W in ((1, 1), (7, 7), (3, 300)):
                    d = dw.group_desc(2, C, H, W, K, s, p, groups, C, layout, dtype)
                    names = [dw.gconv_variant_name(d, i) for i in range(3)]
                    if C // groups * C * K * K < 1 << 31:
                        assert all(n.startswith("group_") for n in names), (C, groups, K, s, H, W, names)
                        assert dw.gconv_bwd_filter_workspace_bytes(d) <= max(64 << 20, 4 * C * (C // groups) * K * K)

"""Which kernel the library sends a layer to, asked on the host (no GPU): every form of a bf16 window that the kernel with operands straight into LDS is built for
reaches it, in both passes and at every size a call can have."""
import itertools

import pytest

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu


def _desc(n, c, h, w, k, r, s, stride, ph, pw):
    return lc.ConvDesc(n, c, h, w, k, r, s, stride, stride, ph, pw, lc.LC_BF16, lc.LC_NHWC)


@pytest.mark.parametrize("window", [(6, 6), (7, 7), (3, 11), (1, 33), (33, 1), (2, 40), (15, 15), (17, 31)], ids=str)
@pytest.mark.parametrize("stride", [1, 2, 3])
def test_windows_of_more_than_32_taps(window, stride):
    """Also as the phases of a strided window, which would otherwise be widened to fp32."""
    r, s = window
    for n, c, k in itertools.product((1, 7, 256), (8, 40, 64, 96, 504, 512), (8, 64, 200, 256, 1024)):
        d = _desc(n, c, 40, 44, k, r, s, stride, r // 2, s // 2)
        for which in (lc.LC_PASS_FWD, lc.LC_PASS_BWD_DATA):
            assert gu.route(d, which).startswith("conv_dma"), (d, which)
        assert gu.route(d, lc.LC_PASS_FWD, stats=True).startswith("conv_dma")
        assert lc.conv2d_fwd_stats_count(d) > 0

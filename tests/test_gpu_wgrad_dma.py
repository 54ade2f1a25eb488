"""GPU parity of the bf16 filter-gradient kernel whose operands go from memory straight into LDS: every tile it is built for, windows and strides
(pixels worked out per row) and plain 1x1 layers, one split (the kernel writes dw) and several, sizes that end inside tiles, stages and splits.
Against float64 on the same bf16 operands.  Bound per element: products are exact; sums of at most ceil(rows / 8) terms of the matrix instruction, a
rounding each, and the additions of the partial sums, 2^-23 of the sum of magnitudes apiece."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu

# n, c, h, w, k, window, stride, padding
SHAPES = [
    (3, 72, 9, 7, 136, 3, 1, 1),        # 128x64
    (5, 136, 14, 14, 264, 1, 1, 0),
    (9, 72, 15, 13, 200, 3, 2, 1),
    (7, 40, 13, 13, 96, 5, 1, 2),
    (4, 32, 11, 9, 72, 5, 2, 0),
    (19, 152, 19, 19, 160, 3, 1, 1),    # 64x128
    (33, 632, 13, 13, 424, 1, 1, 0),
    (20, 696, 5, 5, 56, 1, 1, 0),
    (11, 72, 18, 18, 648, 3, 1, 1),     # 128x128
    (29, 672, 9, 9, 952, 1, 1, 0),
    (25, 688, 10, 10, 136, 3, 1, 1),    # 128x256
    (48, 400, 19, 19, 520, 1, 1, 0),
    (38, 408, 11, 11, 144, 3, 1, 1),    # 256x128
    (52, 536, 19, 19, 392, 1, 1, 0),
    (40, 640, 17, 17, 24, 3, 1, 1),     # 64x256
    (3, 488, 11, 11, 944, 3, 1, 1),     # 256x64
    (3, 64, 1, 1, 2048, 1, 1, 0),       # a few rows of a fully connected layer
    (2, 64, 30, 2, 128, 1, 3, 0),       # a strided 1x1 window, images narrower than its steps
]
LARGE = [
    (203, 48, 30, 30, 136, 3, 1, 1),    # 256x256
    (219, 392, 42, 42, 136, 1, 1, 0),
    (72, 136, 49, 49, 136, 1, 1, 0),    # 256x64 and 64x256, plain
    (260, 136, 57, 57, 32, 1, 1, 0),
]


def _check(s):
    n, c, h, w, k, r, st, pad = s
    g = torch.Generator().manual_seed(11)
    x = torch.randn((n, h, w, c), generator=g).to(torch.bfloat16)
    d = lc.ConvDesc(n, c, h, w, k, r, r, st, st, pad, pad, lc.LC_BF16, lc.LC_NHWC)
    p, q = lc.conv2d_out_shape(d)
    dy = torch.randn((n, p, q, k), generator=g).to(torch.bfloat16)
    print(f"wgrad dma {s}", flush=True)
    ws = gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_WEIGHT))
    dw = torch.full((k, r, r, c), float("nan"), device=gu.DEV)
    lc.conv2d_bwd_weight(d, x.to(gu.DEV), dy.to(gu.DEV), dw, ws)
    torch.cuda.synchronize()
    ref = torch.zeros((k, c * r * r), dtype=torch.float64)
    mag = torch.zeros_like(ref)
    for i in range(0, n, 16):
        u = F.unfold(x[i:i + 16].double().permute(0, 3, 1, 2), r, padding=pad, stride=st).transpose(1, 2).reshape(-1, c * r * r)
        t = dy[i:i + 16].double().reshape(-1, k).t()
        ref += t @ u
        mag += t.abs() @ u.abs()
    order = lambda t: t.view(k, c, r, r).permute(0, 2, 3, 1)       # noqa: E731
    terms = -(-n * p * q // 8) + 64
    assert bool(((dw.cpu().double() - order(ref)).abs() <= terms * 2.0 ** -23 * order(mag)).all())
    return dw


@pytest.mark.parametrize("s", SHAPES + LARGE, ids=str)
def test_matches_float64(s):
    _check(s)


def test_infinities_stay_where_they_are():
    """An infinite gradient reaches its own filter only, an infinite activation the taps that read it."""
    n, c, hw, k = 4, 64, 9, 136
    x = torch.ones((n, hw, hw, c), dtype=torch.bfloat16)
    dy = torch.ones((n, hw, hw, k), dtype=torch.bfloat16)
    dy[-1, -1, -2, 135] = float("inf")
    x[0, 0, 0, 5] = float("inf")
    d = lc.ConvDesc(n, c, hw, hw, k, 3, 3, 1, 1, 1, 1, lc.LC_BF16, lc.LC_NHWC)
    dw = torch.full((k, 3, 3, c), float("nan"), device=gu.DEV)
    lc.conv2d_bwd_weight(d, x.to(gu.DEV), dy.to(gu.DEV), dw, gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_WEIGHT)))
    torch.cuda.synchronize()
    dw = dw.cpu().numpy()
    want = np.zeros((k, 3, 3, c), dtype=bool)
    want[:, :2, :2, 5] = True            # the corner pixel is read by the taps (0..1, 0..1)
    assert np.all(np.isfinite(dw[:135]) == ~want[:135])
    assert not np.any(np.isfinite(dw[135, :2, :, :]))              # taps inside the image at the last row but for its right neighbour

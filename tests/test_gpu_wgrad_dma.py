"""GPU parity of the bf16 filter-gradient kernel whose operands go from memory straight into LDS: every tile it is built for, windows and strides
(pixels worked out per row) and plain 1x1 layers, one split (the kernel writes dw) and several, sizes that end inside tiles, stages and splits.  Against float64
on the same bf16 operands, twice:
  * small whole numbers, whose sums are exact in fp32: the same bits in any order, so that a row lost or taken twice shows at any size;
  * normal numbers.  Products are exact and their signs random, so the roundings add up as their root: a running sum of L rows is rounded at most every eight rows (L / 16
    of its square, since a sum grows as it goes), one addition into the second set of sums is lost, the S splits' additions lose at most S / 2; each is 2^-24 of what is
    summed, whose deviation is the root of the sum of squares of the products.  Six deviations.
Results lie between guard bytes."""
import re

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu

# n, c, h, w, k, window, stride, padding; the tile that takes it
SHAPES = [
    ((3, 72, 9, 7, 136, 3, 1, 1), "128x64"),
    ((5, 136, 14, 14, 264, 1, 1, 0), "128x64"),
    ((9, 72, 15, 13, 200, 3, 2, 1), "128x64"),
    ((7, 40, 13, 13, 96, 5, 1, 2), "128x64"),
    ((4, 32, 11, 9, 72, 5, 2, 0), "128x64"),
    ((19, 152, 19, 19, 160, 3, 1, 1), "64x128"),
    ((33, 632, 13, 13, 424, 1, 1, 0), "64x128"),
    ((20, 696, 5, 5, 56, 1, 1, 0), "64x128"),
    ((11, 72, 18, 18, 648, 3, 1, 1), "128x128"),
    ((29, 672, 9, 9, 952, 1, 1, 0), "128x128"),
    ((25, 688, 10, 10, 136, 3, 1, 1), "128x256"),
    ((48, 400, 19, 19, 520, 1, 1, 0), "128x256"),
    ((38, 408, 11, 11, 144, 3, 1, 1), "256x128"),
    ((52, 536, 19, 19, 392, 1, 1, 0), "256x128"),
    ((40, 640, 17, 17, 24, 3, 1, 1), "64x256"),
    ((3, 488, 11, 11, 944, 3, 1, 1), "256x64"),
    ((3, 64, 1, 1, 2048, 1, 1, 0), "128x64"),      # a few rows of a fully connected layer
    ((2, 64, 30, 2, 128, 1, 3, 0), "128x64"),      # a strided 1x1 window, images narrower than its steps
]
LARGE = [
    ((203, 48, 30, 30, 136, 3, 1, 1), "256x256"),
    ((219, 392, 42, 42, 136, 1, 1, 0), "256x256"),
    ((72, 136, 49, 49, 136, 1, 1, 0), "256x64"),
    ((260, 136, 57, 57, 32, 1, 1, 0), "64x256"),
]


def _dw(d, x, dy, offset=0):
    print(f"wgrad dma {d}", flush=True)
    dw, guard = gu.guarded((d.k, d.r, d.s, d.c), torch.float32, offset=offset)
    lc.conv2d_bwd_weight(d, x.to(gu.DEV), dy.to(gu.DEV), dw, gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_WEIGHT)))
    torch.cuda.synchronize()
    guard()
    return dw.cpu()


def _sums(d, x, dy, squares=False):
    """dw in float64, and the sum of the squares of its products"""
    ref = torch.zeros((d.k, d.c * d.r * d.s), dtype=torch.float64)
    sq = torch.zeros_like(ref)
    for i in range(0, d.n, 16):
        u = F.unfold(x[i:i + 16].double().permute(0, 3, 1, 2), d.r, padding=d.pad_h, stride=d.stride_h).transpose(1, 2).reshape(-1, d.c * d.r * d.s)
        t = dy[i:i + 16].double().reshape(-1, d.k).t()
        ref += t @ u
        if squares:
            sq += t.square() @ u.square()
    order = lambda t: t.view(d.k, d.c, d.r, d.s).permute(0, 2, 3, 1)       # noqa: E731
    return order(ref), order(sq)


def _desc(s):
    n, c, h, w, k, r, st, pad = s
    return lc.ConvDesc(n, c, h, w, k, r, r, st, st, pad, pad, lc.LC_BF16, lc.LC_NHWC)


def _shapes(d):
    p, q = lc.conv2d_out_shape(d)
    return (d.n, d.h, d.w, d.c), (d.n, p, q, d.k)


@pytest.mark.parametrize("s,tile", SHAPES + LARGE, ids=str)
def test_matches_float64(s, tile):
    d = _desc(s)
    m = re.fullmatch(r"wgrad_dma (\d+x\d+) splits (\d+) sums (\d+)", gu.route(d, lc.LC_PASS_BWD_WEIGHT))
    assert m and m[1] == tile
    splits, rows = int(m[2]), int(m[3])
    g = torch.Generator().manual_seed(11)
    x, dy = (torch.randn(t, generator=g).to(torch.bfloat16) for t in _shapes(d))
    ref, sq = _sums(d, x, dy, squares=True)
    bound = 6 * 2.0 ** -24 * (rows / 16 + 2 + splits / 2) ** 0.5 * sq.sqrt()
    err = (_dw(d, x, dy).double() - ref).abs()
    assert bool((err <= bound).all()), float((err / (bound + 1e-30)).max())


@pytest.mark.parametrize("s,tile", SHAPES + LARGE, ids=str)
def test_whole_numbers_are_exact(s, tile):
    d = _desc(s)
    g = torch.Generator().manual_seed(12)
    x, dy = (torch.randint(-2, 3, t, generator=g).to(torch.bfloat16) for t in _shapes(d))
    assert 4 * dy.numel() // d.k < 1 << 24
    assert torch.equal(_dw(d, x, dy).double(), _sums(d, x, dy)[0])


def test_plain_layer_on_an_image_of_a_gibibyte():
    d = _desc((1, 64, 2950, 2950, 72, 1, 1, 0))
    assert gu.route(d, lc.LC_PASS_BWD_WEIGHT).startswith("wgrad_dma")
    g = torch.Generator(device=gu.DEV).manual_seed(14)
    x, dy = (torch.randint(-1, 2, t, generator=g, device=gu.DEV, dtype=torch.int8).to(torch.bfloat16) for t in _shapes(d))
    ref = torch.zeros((d.k, d.c), dtype=torch.float64, device=gu.DEV)
    for t, u in zip(dy.view(-1, d.k).split(1 << 20), x.view(-1, d.c).split(1 << 20)):
        ref += t.t().double().contiguous() @ u.double()
    assert torch.equal(_dw(d, x, dy).double().view(d.k, d.c), ref.cpu())


@pytest.mark.parametrize("s", [SHAPES[0][0], SHAPES[1][0], SHAPES[15][0]], ids=str)
def test_dw_aligned_to_four_bytes(s):
    d = _desc(s)
    g = torch.Generator().manual_seed(13)
    x, dy = (torch.randn(t, generator=g).to(torch.bfloat16) for t in _shapes(d))
    assert torch.equal(_dw(d, x, dy), _dw(d, x, dy, offset=4))


def test_infinities_stay_where_they_are():
    """An infinite gradient reaches its own filter only, an infinite activation the taps that read it; sums of infinite and finite numbers stay infinite
    however often they are taken over into the second set."""
    n, c, hw, k = 4, 64, 9, 136
    x = torch.ones((n, hw, hw, c), dtype=torch.bfloat16)
    dy = torch.ones((n, hw, hw, k), dtype=torch.bfloat16)
    dy[-1, -1, -2, 135] = float("inf")
    x[0, 0, 0, 5] = float("inf")
    d = _desc((n, c, hw, hw, k, 3, 1, 1))
    m = re.fullmatch(r"wgrad_dma \S+ splits 1 sums (\d+)", gu.route(d, lc.LC_PASS_BWD_WEIGHT))
    assert m and int(m[1]) < n * hw * hw                  # one split, several runs
    dw = _dw(d, x, dy).numpy()
    want = np.zeros((k, 3, 3, c), dtype=bool)
    want[:, :2, :2, 5] = True            # the corner pixel is read by the taps (0..1, 0..1)
    want[135, :2, :, :] = True           # taps inside the image at the last row but for its right neighbour
    assert np.all(np.isfinite(dw[:135]) == ~want[:135])
    assert np.all(dw[want] == np.inf)
    x[1, 4, 4, 7] = float("nan")
    dw = _dw(d, x, dy).numpy()
    assert np.all(np.isnan(dw[:, :, :, 7])) and not np.any(np.isnan(dw[:135, :, :, 8:]))

"""GPU parity of the bf16 3x3 kernel whose waves hold the whole filter in registers (64 channels to 33 to 64 filters, and the input gradients of 33 to 64 channels
from 64 filters): images that are one tile and several, a last tile of fewer rows, odd sizes, one column, wide rows of few, turns of 64 pixels in odd and even numbers, a round of
tiles that is not full and several rounds, and results of fewer than 64 columns.  Against float64 on the same bf16 operands.  Bound per element: one rounding to bf16
(2^-8 of the value, in which the fp32 sum on the other side of a rounding boundary is included) and the fp32 sums, a rounding every eight of the 576
terms, 2^-23 of the sum of magnitudes apiece."""
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu

# n, c, h, w, k
SHAPES = [
    (256, 64, 16, 16, 64),       # four turns
    (255, 64, 12, 21, 40),       # odd rows, 40 columns
    (128, 64, 20, 41, 64),       # two tiles of ten rows, seven turns
    (128, 64, 19, 41, 56),       # the last tile a row short
    (256, 64, 190, 1, 64),       # one column: a row of three pixels with its halo
    (128, 64, 4, 126, 48),       # two rows of a tile, four with the halo
    (500, 64, 16, 16, 64),       # two rounds, the second not full
    (70, 64, 56, 56, 64),        # seven tiles of eight rows, seven turns
    (250, 40, 16, 16, 64),       # backward-data from 64 filters
]


@pytest.mark.parametrize("s", SHAPES, ids=str)
def test_matches_float64(s, monkeypatch):
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1")     # read on every call; the library sends larger layers here
    n, c, h, w, k = s
    d = lc.ConvDesc(n, c, h, w, k, 3, 3, 1, 1, 1, 1, lc.LC_BF16, lc.LC_NHWC)
    gen = torch.Generator(device=gu.DEV).manual_seed(23)
    normal = lambda shape, std=1.0: (torch.randn(shape, generator=gen, device=gu.DEV) * std).to(torch.bfloat16)        # noqa: E731
    x, wt, dy = normal((n, h, w, c)), normal((k, 3, 3, c), (9 * c) ** -0.5), normal((n, h, w, k))
    print(f"conv held {s}", flush=True)

    def ref(a, b):                                       # a [n, h, w, ci], b [co, 3, 3, ci], tap by tap in float64
        pad, out = F.pad(a.double(), (0, 0, 1, 1, 1, 1)), 0
        for r in range(3):
            for q in range(3):
                out = out + pad[:, r:r + h, q:q + w].reshape(n * h * w, -1) @ b[:, r, q].double().t().contiguous()
        return out.view(n, h, w, -1)

    def check(got, a, b):
        bound = 2.0 ** -8 * ref(a, b).abs() + (-(-9 * a.shape[3] // 8) + 66) * 2.0 ** -23 * ref(a.abs(), b.abs())
        assert bool(((got.double() - ref(a, b)).abs() <= bound).all())

    def run(fn, which, a, shape):
        out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device=gu.DEV)
        fn(d, a, wt, out, gu.workspace(lc.conv2d_workspace_bytes(d, which)))
        torch.cuda.synchronize()
        return out

    y = run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, dy.shape)
    check(y, x, wt)
    dx = run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, x.shape)
    check(dx, dy, wt.flip(1, 2).permute(3, 1, 2, 0).contiguous())

    # the slab kernel adds in the same order
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1000000000")
    monkeypatch.setenv("LARSCONV_SLAB_MIN_TILES", "1")
    if 1 < w < 100:                                        # (that kernel takes no slabs so narrow or so wide)
        assert torch.equal(y.view(torch.int16), run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, dy.shape).view(torch.int16))
        assert torch.equal(dx.view(torch.int16), run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, x.shape).view(torch.int16))
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1")

    # with statistics: the same bits, and per column the sums of what was stored
    count = lc.conv2d_fwd_stats_count(d)
    assert count > 0
    stats = torch.full((count, k, 2), float("nan"), device=gu.DEV)
    y2 = run(lambda d_, a, b, out, ws: lc.conv2d_fwd_stats(d_, a, b, out, stats, ws), lc.LC_PASS_FWD, x, dy.shape)
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    rows, got = y.double().reshape(-1, k), stats.double().sum(0)
    assert bool(((got[:, 0] - rows.sum(0)).abs() <= 2e-5 * rows.abs().sum(0) + 1e-30).all())
    assert bool(((got[:, 1] - rows.square().sum(0)).abs() <= 2e-5 * rows.square().sum(0) + 1e-30).all())

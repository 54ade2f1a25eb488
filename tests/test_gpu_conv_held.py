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
        out, guard = gu.guarded(shape, torch.bfloat16)
        fn(d, a, wt, out, gu.workspace(lc.conv2d_workspace_bytes(d, which)))
        torch.cuda.synchronize()
        guard()
        return out

    assert (gu.route(d, lc.LC_PASS_FWD) == "conv3x3_held") == (c == 64) and (gu.route(d, lc.LC_PASS_BWD_DATA) == "conv3x3_held") == (k == 64)
    y = run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, dy.shape)
    check(y, x, wt)
    dx = run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, x.shape)
    check(dx, dy, wt.flip(1, 2).permute(3, 1, 2, 0).contiguous())

    # the slab kernel adds in the same order
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1000000000")
    monkeypatch.setenv("LARSCONV_SLAB_MIN_TILES", "1")
    if 1 < w < 100:                                        # (that kernel takes no slabs so narrow or so wide)
        assert gu.route(d, lc.LC_PASS_FWD if c == 64 else lc.LC_PASS_BWD_DATA) == "conv3x3_slab"
        assert torch.equal(y.view(torch.int16), run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, dy.shape).view(torch.int16))
        assert torch.equal(dx.view(torch.int16), run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, x.shape).view(torch.int16))
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1")

    # with statistics: the same bits, and per column the sums of what was stored
    count = lc.conv2d_fwd_stats_count(d)
    assert count > 0
    stats, guard = gu.guarded((count, k, 2), torch.float32)
    y2 = run(lambda d_, a, b, out, ws: lc.conv2d_fwd_stats(d_, a, b, out, stats, ws), lc.LC_PASS_FWD, x, dy.shape)
    guard()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    rows, got = y.double().reshape(-1, k), stats.double().sum(0)
    assert bool(((got[:, 0] - rows.sum(0)).abs() <= 2e-5 * rows.abs().sum(0) + 1e-30).all())
    assert bool(((got[:, 1] - rows.square().sum(0)).abs() <= 2e-5 * rows.square().sum(0) + 1e-30).all())


def test_infinities_and_nan_stay_where_they_are(monkeypatch):
    """An infinite or missing pixel reaches the outputs whose window holds it -- not those of the next image, whose halo it would be -- and a missing filter
    value its own filter and that filter's statistics."""
    monkeypatch.setenv("LARSCONV_HELD_MIN_TURNS", "1")
    n, h, w = 256, 16, 16
    d = lc.ConvDesc(n, 64, h, w, 64, 3, 3, 1, 1, 1, 1, lc.LC_BF16, lc.LC_NHWC)
    assert gu.route(d, lc.LC_PASS_FWD) == "conv3x3_held" and gu.route(d, lc.LC_PASS_FWD, stats=True) == "conv3x3_held"
    gen = torch.Generator(device=gu.DEV).manual_seed(29)
    x = torch.randn((n, h, w, 64), generator=gen, device=gu.DEV).to(torch.bfloat16)
    wt = (torch.randn((64, 3, 3, 64), generator=gen, device=gu.DEV) / 24).to(torch.bfloat16)
    bad = x.clone()
    bad[3, 0, 0, 63] = bad[7, h - 1, w - 1, 0] = float("inf")
    bad[9, h - 1, 5, 31] = bad[11, 4, w - 1, 32] = float("nan")
    want = torch.zeros((n, h, w), dtype=torch.bool, device=gu.DEV)
    for i, p, q in ((3, 0, 0), (7, h - 1, w - 1), (9, h - 1, 5), (11, 4, w - 1)):
        want[i, max(p - 1, 0):p + 2, max(q - 1, 0):q + 2] = True
    y, clean = torch.empty_like(x), torch.empty_like(x)
    lc.conv2d_fwd(d, x, wt, clean, None)
    lc.conv2d_fwd(d, bad, wt, y, None)
    torch.cuda.synchronize()
    assert torch.equal(~torch.isfinite(y), want[..., None].expand_as(y))
    assert torch.equal(y[~want].view(torch.int16), clean[~want].view(torch.int16))
    assert not torch.isnan(y[3]).any() and torch.isnan(y[9][want[9]]).all()

    filt = wt.clone()
    filt[5, 2, 0, 40] = float("nan")
    stats = torch.empty((lc.conv2d_fwd_stats_count(d), 64, 2), device=gu.DEV)
    lc.conv2d_fwd_stats(d, x, filt, y, stats, None)
    torch.cuda.synchronize()
    others = [i for i in range(64) if i != 5]
    assert torch.isnan(y[..., 5]).all() and torch.equal(y[..., others].view(torch.int16), clean[..., others].view(torch.int16))
    assert torch.isnan(stats[:, 5].sum(0)).all() and torch.isfinite(stats[:, others]).all()

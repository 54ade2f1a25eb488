"""GPU parity of the bf16 forward / backward-data kernel whose operands go from memory straight into LDS: every tile it is built for (192 to 256 rows of wide
results, 128x128, 128x64 with four and with two waves, 128x32), channels that are multiples of 64, nearly so (filled up with zeros) and any multiple of 8, tiles taken
whole and shared by blocks, filter counts that are no multiple of 8, and the stride grids of strided layers.  Against float64 on the same bf16 operands.  Bound
per element: one rounding to bf16 (2^-8 of the value, in which the fp32 sum on the other side of a rounding boundary is included) and the fp32
sums, a rounding every eight terms and the additions of parts, 2^-23 of the sum of magnitudes apiece."""
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu

# n, c, hw, k, window, stride
SHAPES = [
    (71, 8, 29, 184, 1, 1),        # 256x256
    (65, 64, 30, 136, 1, 1),
    (34, 64, 30, 288, 1, 1),       # 240
    (106, 16, 17, 504, 1, 1),
    (107, 64, 23, 136, 1, 1),      # 224
    (106, 8, 16, 312, 1, 1),
    (64, 64, 20, 264, 1, 1),       # 208
    (38, 8, 26, 344, 1, 1),
    (57, 64, 24, 152, 1, 1),       # 192
    (98, 8, 19, 152, 1, 1),
    (4, 256, 14, 256, 3, 1),       # 128x128
    (23, 8, 22, 144, 1, 1),
    (21, 576, 8, 104, 3, 1),       # tiles shared
    (76, 296, 6, 72, 3, 1),
    (2, 504, 7, 72, 3, 1),         # 504 channels as 512
    (37, 64, 7, 64, 5, 1),         # 128x64
    (7, 208, 5, 16, 3, 1),
    (2, 128, 5, 16, 3, 1),
    (62, 8, 26, 40, 1, 1),         # two waves
    (57, 64, 24, 16, 1, 1),        # 128x32
    (40, 32, 31, 32, 3, 1),
    (112, 544, 30, 56, 1, 1),
    (3, 64, 1, 1000, 1, 1),        # a fully connected layer of a few rows
    (5, 72, 9, 33, 3, 1),          # filter counts off the vector stores
    (3, 64, 10, 130, 1, 1),
    (2, 64, 13, 35, 3, 1),
    (6, 64, 15, 136, 1, 2),        # stride grids: one pixel in four, and the four phases of a window
    (5, 72, 11, 40, 3, 2),
    (3, 16, 12, 264, 3, 2),
    (2, 256, 9, 8, 5, 3),
    (4, 37, 10, 64, 1, 2),         # stride grids of odd and of even counts of channels
    (3, 38, 9, 64, 3, 2),
]


@pytest.mark.parametrize("s", SHAPES, ids=str)
def test_matches_float64(s):
    n, c, hw, k, r, st = s
    g = torch.Generator().manual_seed(17)
    d = lc.ConvDesc(n, c, hw, hw, k, r, r, st, st, r // 2, r // 2, lc.LC_BF16, lc.LC_NHWC)
    p, q = lc.conv2d_out_shape(d)
    x = torch.randn((n, hw, hw, c), generator=g).to(torch.bfloat16)
    w = (torch.randn((k, r, r, c), generator=g) / (c * r * r) ** 0.5).to(torch.bfloat16)
    dy = torch.randn((n, p, q, k), generator=g).to(torch.bfloat16)
    print(f"conv dma {s}", flush=True)

    def run(fn, which, a, b, shape):
        out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device=gu.DEV)
        ws = gu.workspace(lc.conv2d_workspace_bytes(d, which))
        fn(d, a.to(gu.DEV), b.to(gu.DEV), out, ws)
        torch.cuda.synchronize()
        return out.cpu()

    def check(got, ref, mag, terms):
        bound = 2.0 ** -8 * ref.abs() + (-(-terms // 8) + 66) * 2.0 ** -23 * mag
        assert bool(((got.double() - ref).abs() <= bound).all()), float(((got.double() - ref).abs() / (mag + 1e-30)).max())

    xn, wn, dyn = (t.double().permute(0, 3, 1, 2) for t in (x, w, dy))
    fwd = lambda a, b: F.conv2d(a, b, stride=st, padding=r // 2).permute(0, 2, 3, 1)                                             # noqa: E731
    bwd = lambda a, b: torch.nn.grad.conv2d_input(xn.shape, b, a, stride=st, padding=r // 2).permute(0, 2, 3, 1)                 # noqa: E731
    y = run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, w, dy.shape)
    check(y, fwd(xn, wn), fwd(xn.abs(), wn.abs()), c * r * r)
    check(run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, w, x.shape), bwd(dyn, wn), bwd(dyn.abs(), wn.abs()), k * r * r)

    # with statistics: the same bits, and per column the sums of what was stored
    count = lc.conv2d_fwd_stats_count(d)
    assert count > 0
    stats = torch.full((count, k, 2), float("nan"), device=gu.DEV)
    y2 = run(lambda d_, a, b, out, ws: lc.conv2d_fwd_stats(d_, a, b, out, stats, ws), lc.LC_PASS_FWD, x, w, dy.shape)
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    rows, got = y.double().reshape(-1, k), stats.cpu().double().sum(0)
    assert bool(((got[:, 0] - rows.sum(0)).abs() <= 2e-5 * rows.abs().sum(0) + 1e-30).all())
    assert bool(((got[:, 1] - rows.square().sum(0)).abs() <= 2e-5 * rows.square().sum(0) + 1e-30).all())

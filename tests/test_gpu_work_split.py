"""Parity of the forms in which a product's tiles are dealt to the chip: fewer tiles than compute units, each taken whole by a block; tiles shared
by several blocks in equal parts; the k-steps laid end to end over all blocks; whole rounds with a rest.  bf16 forward and backward-data against
float64 torch on the CPU.  Bound per element: one rounding to bf16 (2^-8 of the value, in which the fp32 sum on the other side of a rounding
boundary is included) and the fp32 sums, (2 * ceil(K / 16) + 66) roundings of 2^-23 of the sum of magnitudes."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu

# n, c, hw, k, window: tiles x k-steps of 128x128 forward (and backward-data)
SHAPES = [
    (16, 512, 7, 2048, 1),      # 112 x 16: whole tiles on an idle chip (28 x 64: shared)
    (2, 64, 56, 256, 1),        # 98 x 2, fewer k-steps than a shared tile needs
    (3, 512, 7, 512, 3),        # 8 x 144: many parts per tile
    (8, 256, 14, 256, 3),       # 26 x 72
    (1, 64, 5, 40, 3),          # one ragged tile
    (70, 128, 28, 320, 1),      # 429 rows x 3 columns: whole rounds and a rest
]


@pytest.mark.parametrize("s", SHAPES, ids=str)
def test_every_form_of_the_split_adds_up(s):
    n, c, hw, k, r = s
    g = torch.Generator().manual_seed(3)
    x = torch.randn((n, hw, hw, c), generator=g).to(torch.bfloat16)
    w = (torch.randn((k, r, r, c), generator=g) / np.sqrt(c * r * r)).to(torch.bfloat16)
    dy = torch.randn((n, hw, hw, k), generator=g).to(torch.bfloat16)
    d = lc.ConvDesc(n, c, hw, hw, k, r, r, 1, 1, r // 2, r // 2, lc.LC_BF16, lc.LC_NHWC)

    def run(fn, which, a, b, shape):
        out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device=gu.DEV)
        fn(d, a.to(gu.DEV), b.to(gu.DEV), out, gu.workspace(lc.conv2d_workspace_bytes(d, which)))
        torch.cuda.synchronize()
        return out.cpu().double()

    def check(got, ref, mag, terms):
        bound = 2.0 ** -8 * ref.abs() + (2 * -(-terms // 16) + 66) * 2.0 ** -23 * mag
        assert bool(((got - ref).abs() <= bound).all()), float(((got - ref).abs() / mag).max())

    xn, wn, dyn = (t.double().permute(0, 3, 1, 2) for t in (x, w, dy))
    fwd = lambda a, b: F.conv2d(a, b, padding=r // 2).permute(0, 2, 3, 1)                                            # noqa: E731
    bwd = lambda a, b: torch.nn.grad.conv2d_input(xn.shape, b, a, padding=r // 2).permute(0, 2, 3, 1)                # noqa: E731
    check(run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, w, dy.shape), fwd(xn, wn), fwd(xn.abs(), wn.abs()), c * r * r)
    check(run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, w, x.shape), bwd(dyn, wn), bwd(dyn.abs(), wn.abs()), k * r * r)


@pytest.mark.parametrize("s", [(41, 48, 7, 520), (17, 32, 44, 544), (40, 16, 7, 640), (3, 80, 28, 192), (2, 40, 31, 33)], ids=str)
def test_ranges_of_several_tiles_meet_inside_tiles(s):
    """fp32 forward 1x1 with one to five k-steps of 16 per tile: blocks of eight k-steps take whole tiles and share the ones their ranges meet in.  The bound
    of the fp32 sums, a rounding every two terms."""
    n, c, hw, k = s
    g = torch.Generator().manual_seed(5)
    x, w = torch.randn((n, hw, hw, c), generator=g), torch.randn((k, 1, 1, c), generator=g)
    d = lc.ConvDesc(n, c, hw, hw, k, 1, 1, 1, 1, 0, 0, lc.LC_F32, lc.LC_NHWC)
    y = torch.full((n, hw, hw, k), float("nan"), device=gu.DEV)
    lc.conv2d_fwd(d, x.to(gu.DEV), w.to(gu.DEV), y, gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_FWD)))
    torch.cuda.synchronize()
    ref, mag = x.double() @ w.double().view(k, c).t(), x.double().abs() @ w.double().abs().view(k, c).t()
    assert bool(((y.cpu().double() - ref).abs() <= (c // 2 + 4) * 2.0 ** -23 * mag).all())

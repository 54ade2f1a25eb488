"""GPU parity of the bf16 kernels that few blocks run on: forward and backward-data with four stages in flight (at most one block a compute unit,
eight k-steps and more: counts around the four stages' wrap, one tile to many, shared tiles and whole ones, whole and padded channel
chunks, pieces, ragged rows and columns, stride grids, statistics; 128x64 and 128x128 tiles) and filter gradients of 128x128 tiles by eight waves; and
shapes of the same kind just below eight k-steps a block.  test_conv_routes.py asks the library whether every form is met.  Reference: float64 on the CPU.

Bounds: as products are exact in fp32, a sum of n of them is off by n * 2^-24 of the sum of their sizes at most, in practice by its square
root: four times that; y and dx are rounded once more to bf16, 2^-8 of the value."""
import math

import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# n, h, w, c, k, window, stride: k-steps of 64 of the forward pass in the comment
LAYERS = [
    (1, 5, 7, 512, 128, 1, 1),        # 8, one tile
    (3, 11, 9, 576, 136, 1, 1),       # 9, ragged rows and columns
    (2, 13, 13, 64, 256, 3, 1),       # 9 from a window
    (1, 9, 10, 192, 100, 3, 1),       # 27, columns in pairs (statistics too)
    (1, 9, 10, 192, 97, 3, 1),        # odd columns: backward-data goes through fp32
    (2, 8, 8, 248, 128, 3, 1),        # channels filled up to 256
    (2, 8, 8, 88, 192, 3, 1),         # pieces
    (5, 14, 14, 256, 256, 3, 1),      # 36, shared tiles
    (4, 10, 10, 640, 512, 1, 2),      # stride grid
    (1, 28, 28, 512, 512, 3, 1),      # 72
    (1, 6, 6, 1032, 48, 1, 1),        # narrow tiles, pieces
    (1, 5, 7, 512, 97, 1, 1),         # odd columns
    (2, 8, 8, 504, 64, 3, 1),         # channels filled up to 512, shared tiles
    # 128x128 tiles
    (37, 7, 7, 512, 512, 3, 1),       # 72, shared
    (4, 28, 28, 256, 256, 3, 1),      # 36, shared
    (16, 14, 14, 504, 256, 3, 1),     # filled up, shared
    (37, 7, 7, 88, 512, 5, 1),        # pieces, shared
    (32, 7, 7, 1032, 2048, 1, 1),     # pieces, whole
    (32, 7, 7, 1024, 2044, 1, 1),     # columns in pairs, whole
    (37, 7, 7, 512, 500, 3, 1),       # columns in pairs, shared
    (32, 14, 14, 512, 2048, 1, 2),    # stride grid, shared
    (37, 14, 14, 1024, 2048, 1, 2),   # stride grid, whole
]


@pytest.mark.parametrize("n,h,w,c,k,r,s", LAYERS)
def test_few_blocks(n, h, w, c, k, r, s):
    g = torch.Generator().manual_seed(n * h + c + k)
    pad = r // 2
    d = lc.ConvDesc(n, c, h, w, k, r, r, s, s, pad, pad, lc.LC_BF16, lc.LC_NHWC)
    p, q = lc.conv2d_out_shape(d)
    x, wt, dy = (torch.randn(v, generator=g).to(torch.bfloat16) for v in ((n, h, w, c), (k, r, r, c), (n, p, q, k)))
    xd, wd, dyd = (t.to(DEV) for t in (x, wt, dy))
    y, dx, dw = torch.empty_like(dyd), torch.empty_like(xd), torch.empty(wt.shape, device=DEV)
    ws = torch.empty(max(256, *(lc.conv2d_workspace_bytes(d, m) for m in (lc.LC_PASS_FWD, lc.LC_PASS_BWD_DATA, lc.LC_PASS_BWD_WEIGHT))),
                     dtype=torch.uint8, device=DEV)
    lc.conv2d_fwd(d, xd, wd, y, ws)
    lc.conv2d_bwd_data(d, dyd, wd, dx, ws)
    lc.conv2d_bwd_weight(d, xd, dyd, dw, ws)

    def close(got, ref, size, terms, bf16):
        bad = (got.cpu().double() - ref).abs() - 4 * math.sqrt(terms) * 2.0 ** -24 * size - (ref.abs() * 2.0 ** -8 if bf16 else 0.0)
        assert bad.max().item() <= 0.0

    x4, w4, d4 = (t.double().permute(0, 3, 1, 2).contiguous().requires_grad_() for t in (x, wt, dy))
    ref = F.conv2d(x4, w4, None, s, pad)
    ref.backward(d4.detach())
    xa, wa = x4.detach().abs().requires_grad_(), w4.detach().abs().requires_grad_()
    size = F.conv2d(xa, wa, None, s, pad)
    size.backward(d4.detach().abs())
    back = lambda t: t.detach().permute(0, 2, 3, 1)
    close(y, back(ref), back(size), c * r * r, True)
    close(dx, back(x4.grad), back(xa.grad), k * r * r, True)
    close(dw, back(w4.grad), back(wa.grad), n * p * q, False)
    count = lc.conv2d_fwd_stats_count(d)
    if count:
        st, y2 = torch.empty((count, k, 2), device=DEV), torch.empty_like(y)
        lc.conv2d_fwd_stats(d, xd, wd, y2, st, ws)
        assert torch.equal(y, y2)
        v = y.double().view(-1, k)
        want = torch.stack([v.sum(0), v.square().sum(0)], 1)
        assert ((st.double().sum(0) - want).abs() <= 1e-5 * torch.stack([v.abs().sum(0), want[:, 1]], 1)).all()

"""GPU parity of the convolution passes where their large operands and results go past the caches: results of 64 MB and more (every kernel
that stores one so: tiles of conv_dma, held, slab, main and fp32 kernels, stride grids and the zeros between them, phases of a strided window, the first layer;
and results that do not: ragged columns, copies), rows of 256 MB and more that are read once (1x1 forward and backward-data to one tile of columns) and
filter gradients of one tile, whose stages go round the splits.  Row counts are no multiple of any tile.  Which form each shape is for stands beside it, and
test_conv_routes.py asks the library whether all of them are met.  Reference: plain products in float64 (1x1) or float32 (windows, by torch) of the same values, on the device.

Bounds: a sum of n products in fp32 is off by at most n * 2^-24 of the sum of their sizes, in practice by its square root: four times
that; a bf16 result is rounded once more, 2^-8 of the value."""
import math

import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rnd(shape, seed, dtype, std=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.randn(shape, generator=g, device=DEV).mul_(std).to(dtype)


def _ws(d, p):
    return torch.empty(max(256, lc.conv2d_workspace_bytes(d, p)), dtype=torch.uint8, device=DEV)


def _close(got, ref, size, n, bf16):
    bad = (got.double() - ref.double()).abs() - 4 * math.sqrt(n) * 2.0 ** -24 * size.max() - (ref.double().abs() * 2.0 ** -8 if bf16 else 0.0)
    assert bad.max().item() <= 0.0


# (images, h, w, c, k); 40, 100 and 97 columns end within a tile, 97 within a line
POINTWISE = [(1, 500, 503, 512, 40), (1, 500, 503, 512, 104), (1, 500, 503, 512, 256),                 # rows read once: 128x64, 128x128 and 256x256 tiles
             (1, 500, 503, 512, 32), (1, 500, 503, 32, 512), (1, 500, 503, 128, 512),                  # 128x32; backward-data to 32 and 128 columns
             (1, 1021, 979, 128, 64), (1, 801, 803, 120, 8), (1, 801, 803, 24, 104), (1, 801, 803, 8, 184), (1, 801, 803, 184, 8),   # gradients of one tile: 64x128 twice, 128x64, 256x64, 64x256
             (1, 801, 803, 72, 88), (1, 1281, 1283, 80, 80), (1, 801, 803, 96, 136), (1, 1001, 1003, 200, 72),      # 128x128 by eight waves and by four, 256x128, 128x256
             (1, 1281, 1283, 200, 136), (1, 801, 803, 72, 72),                                         # 256x256; a tile less than three fifths full
             (1, 801, 803, 64, 64),                                                                    # the main kernel's 256x64 tile
             (1, 601, 601, 64, 100), (1, 601, 601, 64, 97), (1, 331, 333, 24, 512), (1, 401, 403, 64, 256), (1, 401, 403, 256, 64)]


@pytest.mark.parametrize("dtype", [lc.LC_BF16, lc.LC_F32])
@pytest.mark.parametrize("n,h,w,c,k", POINTWISE)
def test_pointwise(dtype, n, h, w, c, k):
    t, bf16 = (torch.bfloat16, True) if dtype == lc.LC_BF16 else (torch.float32, False)
    d = lc.ConvDesc(n, c, h, w, k, 1, 1, 1, 1, 0, 0, dtype, lc.LC_NHWC)
    rows = n * h * w
    x, wt, dy = _rnd((n, h, w, c), 1, t), _rnd((k, 1, 1, c), 2, t, c ** -0.5), _rnd((n, h, w, k), 3, t)
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty((k, 1, 1, c), device=DEV)
    lc.conv2d_fwd(d, x, wt, y, _ws(d, lc.LC_PASS_FWD))
    lc.conv2d_bwd_data(d, dy, wt, dx, _ws(d, lc.LC_PASS_BWD_DATA))
    lc.conv2d_bwd_weight(d, x, dy, dw, _ws(d, lc.LC_PASS_BWD_WEIGHT))
    x2, w2, d2 = x.view(rows, c).double(), wt.view(k, c).double(), dy.view(rows, k).double()
    _close(dw.view(k, c), d2.t() @ x2, torch.full((), x2.square().sum(0).max().sqrt().item() * d2.square().sum(0).max().sqrt().item(), device=DEV), rows, False)
    aw = w2.abs()
    _close(y.view(rows, k), x2 @ w2.t(), x2.abs() @ aw.t(), c, bf16)
    _close(dx.view(rows, c), d2 @ w2, d2.abs() @ aw, k, bf16)
    if not lc.conv2d_fwd_stats_count(d):
        return
    st = torch.empty((lc.conv2d_fwd_stats_count(d), k, 2), device=DEV)
    y2 = torch.empty_like(y)
    lc.conv2d_fwd_stats(d, x, wt, y2, st, _ws(d, lc.LC_PASS_FWD))
    assert torch.equal(y, y2)
    want = torch.stack([y.view(rows, k).double().sum(0), y.view(rows, k).double().square().sum(0)], 1)
    scale = torch.stack([y.view(rows, k).double().abs().sum(0), want[:, 1]], 1)
    assert ((st.double().sum(0) - want).abs() <= 1e-5 * scale).all()


WINDOWS = [(160, 56, 56, 64, 64, 3, 1), (200, 56, 56, 32, 64, 3, 1), (3, 601, 603, 32, 64, 3, 1), (12, 211, 213, 32, 64, 3, 1),     # held, slab, main 256x64 and 128x64
           (12, 211, 213, 64, 64, 3, 1), (5, 301, 299, 64, 128, 3, 1), (3, 301, 299, 136, 128, 3, 1),                            # 128x64, 128x128, pieces
           (32, 130, 122, 128, 512, 1, 2), (64, 130, 122, 128, 128, 3, 2), (41, 224, 224, 3, 64, 7, 2),                          # stride grid, phases, the first layer
           (3, 211, 213, 64, 64, 3, 1), (5, 211, 213, 32, 64, 3, 1), (2, 301, 299, 64, 320, 3, 1), (2, 301, 299, 12, 200, 3, 1), (9, 130, 122, 128, 256, 1, 2),
           (9, 130, 122, 40, 264, 1, 2), (11, 224, 224, 3, 64, 7, 2)]


@pytest.mark.parametrize("dtype", [lc.LC_BF16, lc.LC_F32])
@pytest.mark.parametrize("n,h,w,c,k,r,s", WINDOWS)
def test_windows(dtype, n, h, w, c, k, r, s):
    t, bf16 = (torch.bfloat16, True) if dtype == lc.LC_BF16 else (torch.float32, False)
    if s == 2 and r == 1:
        c, k = k, c                                                # the stride grid is the large tensor
    d = lc.ConvDesc(n, c, h, w, k, r, r, s, s, r // 2, r // 2, dtype, lc.LC_NHWC)
    p, q = lc.conv2d_out_shape(d)
    x, wt, dy = _rnd((n, h, w, c), 4, t), _rnd((k, r, r, c), 5, t, (c * r * r) ** -0.5), _rnd((n, p, q, k), 6, t)
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    lc.conv2d_fwd(d, x, wt, y, _ws(d, lc.LC_PASS_FWD))
    lc.conv2d_bwd_data(d, dy, wt, dx, _ws(d, lc.LC_PASS_BWD_DATA))
    w4 = wt.double().permute(0, 3, 1, 2).contiguous().cpu()
    for i in (0, n - 1):                                           # the first and the last image, in float64 on the CPU
        xi, di = (v[i:i + 1].double().permute(0, 3, 1, 2).contiguous().cpu() for v in (x, dy))
        ref, size = (F.conv2d(a, b, None, s, r // 2).permute(0, 2, 3, 1) for a, b in ((xi, w4), (xi.abs(), w4.abs())))
        _close(y[i:i + 1].cpu(), ref, size, c * r * r, bf16)
        back = lambda a, b: F.conv_transpose2d(a, b, None, s, r // 2, output_padding=(h - ((p - 1) * s - 2 * (r // 2) + r), w - ((q - 1) * s - 2 * (r // 2) + r)))
        ref, size = (back(a, b).permute(0, 2, 3, 1) for a, b in ((di, w4), (di.abs(), w4.abs())))
        _close(dx[i:i + 1].cpu(), ref, size, k * r * r, bf16)

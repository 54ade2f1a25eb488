"""GPU parity of the gradient of a strided 1x1 convolution's input where the zeros between the stride grid are written by themselves: rows below, at and
around a block of 256 vectors, strides that differ, sizes that end on and off the grid, pixels that are not whole vectors, and a tensor whose zeros go
past the caches (64 MB).  dx holds NaN before the call: whatever is not written shows.  Off the grid zeros are exact; on it the bound is K roundings of the
products' sum (2^-24 each, doubled for the products themselves) and one bf16 rounding of the result (2^-8)."""
import pytest
import torch

from paper_1709_05011_amd import larsconv as lc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CASES = [(3, 5, 3, 16, 24, 2, 2), (2, 7, 8, 128, 32, 2, 2), (2, 9, 17, 60, 40, 2, 2), (1, 6, 51, 40, 16, 3, 2), (3, 8, 33, 64, 64, 1, 2), (2, 11, 64, 72, 8, 2, 1),
         (4, 14, 14, 256, 64, 2, 2), (2, 13, 15, 520, 32, 2, 2), (2, 10, 12, 130, 24, 2, 2), (5, 160, 176, 128, 64, 2, 2), (5, 321, 177, 128, 32, 2, 2)]


@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16])
@pytest.mark.parametrize("n,h,w,c,k,sh,sw", CASES)
def test_strided_pointwise_backward_data(dtype, n, h, w, c, k, sh, sw):
    t, bf16 = (torch.bfloat16, True) if dtype == lc.LC_BF16 else (torch.float32, False)
    d = lc.ConvDesc(n, c, h, w, k, 1, 1, sh, sw, 0, 0, dtype, lc.LC_NHWC)
    p, q = lc.conv2d_out_shape(d)
    g = torch.Generator(device=DEV).manual_seed(11)
    dy = torch.randn((n, p, q, k), generator=g, device=DEV).to(t)
    wt = torch.randn((k, 1, 1, c), generator=g, device=DEV).mul_(k ** -0.5).to(t)
    dx = torch.full((n, h, w, c), float("nan"), device=DEV, dtype=t)
    nb = lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_DATA)
    lc.conv2d_bwd_data(d, dy, wt, dx, torch.empty(max(nb, 16), dtype=torch.uint8, device=DEV))
    d2, w2 = dy.view(-1, k).double(), wt.view(k, c).double()
    ref, size = (d2 @ w2).view(n, p, q, c), (d2.abs() @ w2.abs()).view(n, p, q, c)
    got = dx[:, ::sh, ::sw].double()
    assert got.shape == ref.shape
    bad = (got - ref).abs() - 2 * k * 2.0 ** -24 * size - (ref.abs() * 2.0 ** -8 if bf16 else 0.0)
    assert bad.max().item() <= 0.0                                   # (NaN fails this)
    dx[:, ::sh, ::sw] = 0
    assert int((dx != 0).sum()) == 0                                  # (NaN != 0)

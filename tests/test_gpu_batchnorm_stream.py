"""GPU parity of the batch-norm passes where their streaming choices change: channel counts that a block of 64 vectors does not divide,
a last block that is partly past the end, tensors on both sides of the size from which the stream pass goes past the caches
(112 MB: one row less and one more) and from which the reduce pass does (200 MB over the tensors that are read again), and a channel count
that takes the loop kernel.  Reference: the same formulas in float64 on the device; for the joined pass's forms (ordinary accesses, past the caches
but for the last rows, past them with rows that are not whole lines of 128 bytes) the two plain calls, bit for bit.

Bounds: an fp32 value carries at most a handful of roundings of its terms (scale*x, shift, residual; in the backward pass dy and the two
sums over the rows, which are themselves sums of a few hundred fp32 values a thread): 2e-6 (34 * 2^-24) of the largest sum of the terms'
sizes.  A bf16 result is rounded once more: 2^-8 of the value."""
import pytest
import torch

from paper_1709_05011_amd import larsconv as lc

pytestmark = pytest.mark.gpu
DEV, EPS = "cuda:0", 1e-5

SMALL = [(1, 1, 1, 8), (2, 3, 5, 24), (1, 7, 9, 40), (3, 5, 5, 520), (5, 13, 11, 2056), (2, 1, 1, 8 * ((1 << 20) + 3))]
# (images, h, w, channels): fp32 sizes of 66, 112 less a row, 112 and a row, 135 and 217 MB (the reduce pass of a backward call reads two of them)
LARGE = [(1, 470, 489, 72), (1, 1, 388888, 72), (1, 1, 388889, 72), (1, 700, 669, 72), (1, 868, 869, 72)]
# the joined pass: fp32 sizes of 89, 120 and 217 MB, of which the last 105 stay in the caches; rows of whole lines and not; row counts that no tile divides
JOINED = [(1, 557, 623, 64), (3, 487, 323, 64), (1, 651, 653, 128), (1, 868, 869, 72), (1, 325, 323, 520)]


def _case(dtype, n, h, w, c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    t = torch.bfloat16 if dtype == lc.LC_BF16 else torch.float32
    rnd = lambda shape, std=1.0: torch.randn(shape, generator=g, device=DEV).mul_(std)
    shape = (n, h, w, c)
    return (rnd(shape).add_(0.25).to(t), rnd(shape, 1e-3).to(t), rnd(shape).to(t), 1.0 + rnd((c,), 0.1), rnd((c,), 0.1), t)


def _close(got, ref, terms, bf16):
    bad = (got.double() - ref).abs() - 2e-6 * terms.max() - (ref.abs() * 2.0 ** -8 if bf16 else 0.0)
    assert bad.max().item() <= 0.0, (bad.max().item(), terms.max().item())


@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16])
@pytest.mark.parametrize("n,h,w,c", SMALL + LARGE)
def test_passes_match_float64(dtype, n, h, w, c):
    if dtype == lc.LC_BF16 and (n, h, w, c) in LARGE:
        h *= 2                                                     # the same bytes
    x, dy, res, gamma, beta, t = _case(dtype, n, h, w, c, 7)
    bf16 = t == torch.bfloat16
    y, dx, d2 = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
    mean, inv, dgamma, dbeta = (torch.empty(c, device=DEV) for _ in range(4))
    ws = torch.empty(lc.batchnorm_workspace_bytes(n, c, h, w, lc.LC_NHWC), dtype=torch.uint8, device=DEV)
    rows = n * h * w
    x64, r64, d64 = (v.double().view(rows, c) for v in (x, res, dy))
    lc.batchnorm_fwd_t(dtype, x, gamma, beta, res, y, mean, inv, n, c, h, w, EPS, False, lc.LC_NHWC, ws)
    mu = x64.mean(0)
    var = (x64 - mu).square().mean(0)
    assert (mean.double() - mu).abs().max().item() <= 2e-6 * x64.abs().max().item()
    assert torch.allclose(inv.double(), 1.0 / torch.sqrt(var + EPS), rtol=2e-6 + 2e-6 * (x64.abs().max().item() ** 2 / EPS if rows < 8 else 1.0), atol=0)
    # everything after the statistics from the device's own: scale and shift as floats, so that the ReLU's decisions are the device's
    i64, m64, g64 = inv.double(), mean.double(), gamma.double()
    scale = (g64 * i64).float().double()
    shift = (beta.double() - m64 * (g64 * i64)).float().double()
    pre, terms = scale * x64 + shift, scale.abs() * x64.abs() + shift.abs()
    _close(y.view(rows, c), pre + r64, terms + r64.abs(), bf16)
    lc.batchnorm_fwd_t(dtype, x, gamma, beta, None, y, mean, inv, n, c, h, w, EPS, True, lc.LC_NHWC, ws)
    _close(y.view(rows, c), pre.clamp(min=0), terms, bf16)
    xh, wide = (x64 - m64) * i64, (x64.abs() + m64.abs()) * i64
    for relu in (False, True):
        lc.batchnorm_bwd_t(dtype, x, dy, gamma, beta, mean, inv, dx, dgamma, dbeta, n, c, h, w, relu, lc.LC_NHWC, ws)
        d = torch.where(pre > 0, d64, torch.zeros_like(d64)) if relu else d64
        s0, s1 = d.sum(0), (d * xh).sum(0)
        assert ((dbeta.double() - s0).abs() <= 2e-6 * d.abs().sum(0)).all()
        assert ((dgamma.double() - s1).abs() <= 2e-6 * (d.abs() * wide).sum(0)).all()
        a = g64.abs() * i64
        _close(dx.view(rows, c), g64 * i64 * (d - s0 / rows - xh * s1 / rows),
               a * (d.abs() + d.abs().sum(0) / rows + wide * (d.abs() * wide).sum(0) / rows), bf16)
    del pre, terms, xh, wide, d
    # the joined form: dy = (res > 0 ? dy + x : 0) written on the way, the sums left for the presummed backward
    lc.relu_add_bwd_bnsums_t(dtype, res, dy, x, d2, x, mean, inv, n, c, h, w, lc.LC_NHWC, ws)
    want = torch.where(res.float() > 0, dy.float() + x.float(), torch.zeros((), device=DEV)).to(t)
    assert torch.equal(d2, want)
    lc.batchnorm_bwd_presummed_t(dtype, x, d2, gamma, mean, inv, dx, dgamma, dbeta, n, c, h, w, lc.LC_NHWC, ws)
    lc.batchnorm_bwd_t(dtype, x, d2, gamma, beta, mean, inv, y, mean.clone(), inv.clone(), n, c, h, w, False, lc.LC_NHWC, ws)
    assert torch.equal(dx, y)


@pytest.mark.parametrize("dtype", [lc.LC_F32, lc.LC_BF16])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("n,h,w,c", JOINED)
def test_joined_pass_is_the_two_plain_calls(dtype, two, stride, n, h, w, c):
    if dtype == lc.LC_BF16:
        h *= 2
    x, _, y, gamma, beta, t = _case(dtype, n, h, w, c, 11)
    g = torch.Generator(device=DEV).manual_seed(12)
    small = [torch.randn((n, -(-h // stride), -(-w // stride), c), generator=g, device=DEV).to(t) for _ in range(1 + two)]
    grads = []
    for v in small:
        grads.append(torch.zeros_like(x) if stride > 1 else v)
        if stride > 1:
            grads[-1][:, ::stride, ::stride] = v
    mean, inv = torch.randn(c, generator=g, device=DEV).mul_(0.1), torch.rand(c, generator=g, device=DEV).add_(0.5)
    dg1, db1, dg2, db2 = (torch.empty(c, device=DEV) for _ in range(4))
    ws = torch.empty(lc.batchnorm_workspace_bytes(n, c, h, w, lc.LC_NHWC), dtype=torch.uint8, device=DEV)
    d1, d2, dx1, dx2 = (torch.full_like(x, float("nan")) for _ in range(4))
    lc.relu_add_bwd_bnsums_grid_t(dtype, y, small[0], small[1] if two else None, d1, x, mean, inv, n, c, h, w, stride, lc.LC_NHWC, ws)
    lc.batchnorm_bwd_presummed_t(dtype, x, d1, gamma, mean, inv, dx1, dg1, db1, n, c, h, w, lc.LC_NHWC, ws)
    lc.relu_add_bwd_t(dtype, y, grads[0], grads[1] if two else None, d2, x.numel())
    lc.batchnorm_bwd_t(dtype, x, d2, gamma, beta, mean, inv, dx2, dg2, db2, n, c, h, w, False, lc.LC_NHWC, ws)
    assert torch.equal(d1, d2) and torch.equal(dg1, dg2) and torch.equal(db1, db2) and torch.equal(dx1, dx2)

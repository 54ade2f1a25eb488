"""GPU parity of the fp32 passes that run on the bf16 matrix pipe, each operand as the sum of three bf16 values.

Checked against float64 torch on the CPU, element by element, with the bound that the arithmetic gives: a product's three dropped parts are
below 2^-24 of it together; each of the six kept ones is added with four roundings (one after eight terms, taken as 2^-24 each) to a sum over one
k-step of 32 reduction indices, and that sum with one rounding to the accumulator.  With the sums of stream-K pieces or batch splits (at most 64 more)
that is below (ceil(K / 32) + 90) * 2^-23 of the sum of magnitudes; _within() allows six roundings per k-step and 66:
|error| <= (6 * ceil(K / 32) + 66) * 2^-23 * sum |a| |b|, which the fp32 instructions of the forward pass (and of filter counts that are not multiples
of four, in backward-data) keep in practice as well.  Worst-case bounds are loose by the square root of the number of roundings, so the errors'
norm and mean are bounded too, over long reductions."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu

pytestmark = pytest.mark.gpu
NHWC = lc.LC_NHWC

# n, c, h, w, k, r, stride, pad: edges of tiles (128 rows, 64 and 128 columns), reduction remainders (32), channel counts below a k-step,
# result widths that are not multiples of four, strided results on a grid, stream-K pieces, and one whole tile only
SHAPES = [
    (1, 32, 16, 8, 128, 1, 1, 0), (1, 32, 16, 8, 64, 3, 1, 1), (3, 64, 13, 11, 129, 1, 1, 0), (2, 36, 9, 9, 65, 3, 1, 1),
    (2, 4, 15, 17, 33, 3, 1, 1), (5, 12, 7, 7, 62, 5, 1, 2), (2, 96, 14, 14, 130, 1, 2, 0), (1, 20, 6, 5, 4, 3, 1, 1),
    (4, 256, 7, 7, 256, 3, 1, 1), (40, 64, 28, 28, 256, 1, 1, 0), (2, 48, 12, 12, 96, 3, 2, 1), (1, 1024, 1, 1, 1000, 1, 1, 0),
]


def _desc(s):
    n, c, h, w, k, r, stride, pad = s
    return lc.ConvDesc(n, c, h, w, k, r, r, stride, stride, pad, pad, lc.LC_F32, NHWC)


def _conv64(x, w, s):
    """forward in float64; x, w NHWC / KRSC arrays"""
    xt, wt = (torch.from_numpy(np.ascontiguousarray(np.transpose(a, (0, 3, 1, 2)))).double() for a in (x, w))
    return F.conv2d(xt, wt, stride=s[6], padding=s[7]).permute(0, 2, 3, 1).numpy()


def _conv64_bwd(dy, w, s):
    dyt, wt = (torch.from_numpy(np.ascontiguousarray(np.transpose(a, (0, 3, 1, 2)))).double() for a in (dy, w))
    return torch.nn.grad.conv2d_input((s[0], s[1], s[2], s[3]), wt, dyt, stride=s[6], padding=s[7]).permute(0, 2, 3, 1).numpy()


def _conv64_wgrad(x, dy, s):
    xt, dyt = (torch.from_numpy(np.ascontiguousarray(np.transpose(a, (0, 3, 1, 2)))).double() for a in (x, dy))
    return torch.nn.grad.conv2d_weight(xt, (s[4], s[1], s[5], s[5]), dyt, stride=s[6], padding=s[7]).permute(0, 2, 3, 1).numpy()


def _data(s, seed, wide=False):
    """normal values; wide: magnitudes spread over 2^-40 .. 2^40"""
    rng = np.random.default_rng(seed)
    d = _desc(s)
    p, q = lc.conv2d_out_shape(d)

    def make(*shape):
        a = rng.standard_normal(shape)
        if wide:
            a = a * np.exp2(rng.integers(-40, 41, shape))
        return a.astype(np.float32)
    return d, make(s[0], s[2], s[3], s[1]), make(s[4], s[5], s[5], s[1]), make(s[0], p, q, s[4])


def _within(got, ref, mag, k, step=None):
    """step: reduction indices per rounding where the fp32 instructions may run (two of them per instruction)"""
    bound = (max(6 * -(-k // 32), -(-k // step) if step else 0) + 66) * 2.0 ** -23 * mag
    bad = ~(np.abs(got.astype(np.float64) - ref) <= bound)
    assert not bad.any(), (int(bad.sum()), np.max(np.abs(got - ref) / np.maximum(mag, 1e-300)))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("s", SHAPES, ids=str)
def test_all_three_passes_within_the_bound(s, wide):
    d, x, w, dy = _data(s, 11, wide)
    _within(gu.gpu_fwd(d, x, w), _conv64(x, w, s), _conv64(abs(x), abs(w), s), s[1] * s[5] ** 2)
    _within(gu.gpu_bwd_data(d, dy, w), _conv64_bwd(dy, w, s), _conv64_bwd(abs(dy), abs(w), s), s[4] * s[5] ** 2)
    _within(gu.gpu_bwd_weight(d, x, dy), _conv64_wgrad(x, dy, s), _conv64_wgrad(abs(x), abs(dy), s), dy.size // s[4])



def _norm_and_mean(got, ref):
    e = got.astype(np.float64) - ref
    return np.linalg.norm(e) / np.linalg.norm(ref), abs(e.mean()) / np.sqrt((ref * ref).mean())


def test_long_sums_round_once_per_k_step():
    """Whole tiles of 16 k-steps (784 of them on 256 compute units) and splits of 8 and 16.  A sum of n k-steps rounded once each to nearest (rms
    0.41 * 2^-24 of the running sum, which grows like a random walk) is off by sqrt(n / 2) * 0.41 * 2^-24 of its size, 0.7e-7 for n = 16, plus the roundings
    inside a k-step, 0.5e-7; six times four roundings per step give 3.2e-7.  The mean: what the instruction cuts always the same way, 24 times
    0.006 * 2^-24 of a k-step's sum, would be -5e-7 of the result for 6272 steps without the alternating sign."""
    s = (32, 64, 56, 56, 512, 1, 1, 0)
    d, x, w, dy = _data(s, 23)
    err, mean = _norm_and_mean(gu.gpu_bwd_data(d, dy, w), (dy.reshape(-1, 512).astype(np.float64) @ w.reshape(512, 64)).reshape(x.shape))
    assert err < 2e-7 and mean < 2e-8, (err, mean)
    for s, limit in (((64, 64, 56, 56, 256, 1, 1, 0), 2.5e-7), ((1, 1536, 64, 64, 1024, 1, 1, 0), 2e-7)):
        d, x, w, dy = _data(s, 29)
        x = np.maximum(x, 0)                                          # behind a ReLU
        ref = dy.reshape(-1, s[4]).T.astype(np.float64) @ x.reshape(-1, s[1])
        err, mean = _norm_and_mean(gu.gpu_bwd_weight(d, x, dy), ref.reshape(w.shape))
        assert err < limit and mean < 5e-8, (s, err, mean)


@pytest.mark.parametrize("c,k", [(128, 128), (60, 64), (68, 132)])
def test_each_of_the_six_products_counts(c, k):
    """Results that are one product each: all 24 bits of both operands matter (without the smallest of the kept products the error is above 2^-19)."""
    rng = np.random.default_rng(31)

    def full(*shape):                                                 # 24 significant bits, the lowest always set
        m = rng.integers(1 << 23, 1 << 24, shape) | 1
        return (m * np.exp2(rng.integers(-30, 10, shape))).astype(np.float32)
    n = 300
    d = lc.ConvDesc(n, c, 1, 1, k, 1, 1, 1, 1, 0, 0, lc.LC_F32, NHWC)
    w, v, at = full(k, 1, 1, c), full(n), rng.integers(0, k, n)
    dy = np.zeros((n, 1, 1, k), np.float32)
    dy[np.arange(n), 0, 0, at] = v
    ref = v[:, None].astype(np.float64) * w[at, 0, 0, :]
    got = gu.gpu_bwd_data(d, dy, w).reshape(n, c)
    assert (np.abs(got - ref) <= 2.0 ** -22 * np.abs(ref)).all(), np.max(np.abs(got / ref - 1))
    x, dy = np.zeros((n, 1, 1, c), np.float32), np.zeros((n, 1, 1, k), np.float32)
    x[7], dy[7] = full(1, 1, c), full(1, 1, k)
    ref = dy[7].reshape(k, 1).astype(np.float64) * x[7].reshape(1, c)
    got = gu.gpu_bwd_weight(d, x, dy).reshape(k, c)
    assert (np.abs(got - ref) <= 2.0 ** -22 * np.abs(ref)).all(), np.max(np.abs(got / ref - 1))


@pytest.mark.parametrize("e", [-112, -118, -124, -130])
@pytest.mark.parametrize("s", [(3, 64, 13, 11, 128, 1, 1, 0), (2, 36, 9, 9, 68, 3, 1, 1), (2, 96, 14, 14, 132, 1, 2, 0), (2, 20, 12, 12, 96, 3, 2, 1)], ids=str)
def test_the_smallest_numbers_keep_their_bits(s, e):
    """One operand of magnitude 2^e, down into fp32's subnormal numbers -- unscaled, the lower parts of its split fall below the smallest bf16, 2^-133 --
    against partners that keep the results normal.  As accurate as elsewhere: at most 20 k-steps, so below 1.5e-7 of the norm as derived above."""
    d, x, w, dy = _data(s, 41)

    def tiny(a):
        return (a * 2.0 ** e).astype(np.float32)
    up = np.float32(2.0 ** 60)
    for dy_, w_ in ((tiny(dy), w * up), (dy * up, tiny(w))):
        err, _ = _norm_and_mean(gu.gpu_bwd_data(d, dy_, w_), _conv64_bwd(dy_, w_, s))
        assert err < 1.5e-7, err
    for x_, dy_ in ((tiny(x), dy * up), (x * up, tiny(dy))):
        err, _ = _norm_and_mean(gu.gpu_bwd_weight(d, x_, dy_), _conv64_wgrad(x_, dy_, s))
        assert err < 1.5e-7, err


# The rows, filters and columns at which a filter gradient changes kernels (wide results, one 64x64 tile, few rows, filter counts that are not
# multiples of four), both sides of each line; n, c, hw, k, window, stride.
ROUTES = [
    (1, 64, 23, 64, 1, 1), (1, 64, 23, 62, 1, 1), (1, 32, 46, 64, 1, 2), (1, 32, 44, 64, 1, 2), (4, 32, 128, 64, 1, 2), (5, 32, 128, 64, 1, 2),
    (1, 68, 16, 64, 1, 1), (1, 68, 17, 64, 1, 1), (1, 64, 16, 68, 1, 1), (1, 64, 17, 66, 1, 1), (1, 8, 12, 64, 3, 1), (1, 8, 13, 64, 3, 1),
    (1, 2048, 16, 768, 1, 1), (1, 2048, 16, 764, 1, 1), (1, 2048, 17, 768, 1, 1), (1, 2732, 14, 64, 3, 1), (1, 2728, 14, 64, 3, 1), (2, 4, 56, 64, 3, 1), (1, 7, 28, 64, 1, 1), (3, 64, 56, 64, 1, 1),
]


@pytest.mark.parametrize("s", ROUTES, ids=str)
def test_filter_gradients_on_either_side_of_every_line(s):
    n, c, hw, k, r, stride = s
    d, x, _, dy = _data((n, c, hw, hw, k, r, stride, r // 2), 17)
    t = (n, c, hw, hw, k, r, stride, r // 2)
    _within(gu.gpu_bwd_weight(d, x, dy), _conv64_wgrad(x, dy, t), _conv64_wgrad(abs(x), abs(dy), t), dy.size // k, step=2)


def _same_where_not_finite(got, ref):
    """ref: float64 with infinities and NaN where fp32 arithmetic has them; the finite rest is compared by the caller"""
    ref32 = ref.astype(np.float32)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref32))
    inf = np.isinf(ref32)
    np.testing.assert_array_equal(got[inf], ref32[inf])
    return np.isfinite(ref32)


@pytest.mark.parametrize("s", [SHAPES[2], SHAPES[3], SHAPES[6], SHAPES[8]], ids=str)
def test_infinities_nans_and_the_largest_values_come_through_as_in_fp32(s):
    d, x, w, dy = _data(s, 5)
    rng = np.random.default_rng(6)

    def plant(a, values):
        a = a.copy()
        for v in values:
            a[tuple(rng.integers(0, m) for m in a.shape)] = v
        return a
    top = np.finfo(np.float32).max
    # +-inf and NaN in the activations (every row or pixel they reach), and a value whose bf16 rounding overflows
    with np.errstate(over="ignore", invalid="ignore"):
        for values in ([np.inf], [np.inf, -np.inf, np.nan], [top]):
            xs, ds = plant(x, values), plant(dy, values)
            small = (w * np.float32(0.01)).astype(np.float32)         # keeps a sum around the largest value finite
            ref, mag = _conv64(xs, small, s), _conv64(abs(xs), abs(small), s)
            got = gu.gpu_fwd(d, xs, small)
            ok = _same_where_not_finite(got, ref)
            _within(got[ok], ref[ok], mag[ok], s[1] * s[5] ** 2)
            ref, mag = _conv64_bwd(ds, small, s), _conv64_bwd(abs(ds), abs(small), s)
            got = gu.gpu_bwd_data(d, ds, small)
            ok = _same_where_not_finite(got, ref)
            _within(got[ok], ref[ok], mag[ok], s[4] * s[5] ** 2)
            xw = (x * np.float32(0.01)).astype(np.float32)
            ref, mag = _conv64_wgrad(xw, ds, s), _conv64_wgrad(abs(xw), abs(ds), s)
            got = gu.gpu_bwd_weight(d, xw, ds)
            ok = _same_where_not_finite(got, ref)
            _within(got[ok], ref[ok], mag[ok], dy.size // s[4])
        # ... and in a filter: one column of the result
        ws = plant(w, [np.inf])
        ref = _conv64(x, ws, s)
        got = gu.gpu_fwd(d, x, ws)
        ok = _same_where_not_finite(got, ref)
        _within(got[ok], ref[ok], _conv64(abs(x), abs(ws), s)[ok], s[1] * s[5] ** 2)


# Backward-data on the split kernel (the gathered channels, k, are a multiple of four) with results that are c wide: tile edges, widths that are not
# multiples of four, and every addressing it has -- k-steps inside one tap (k a multiple of 32), k-steps across taps, fewer channels than a k-step --
# each plain and with the result of a strided 1x1 on its grid, strided windows in phases, and tiles shared between blocks (long reductions).
RAGGED = [
    (2, 130, 9, 9, 32, 3, 1, 1), (3, 65, 13, 11, 64, 1, 1, 0), (2, 33, 9, 9, 36, 3, 1, 1), (2, 129, 7, 7, 20, 3, 1, 1), (1, 128, 11, 12, 4, 3, 1, 1),
    (2, 62, 14, 14, 64, 1, 2, 0), (2, 130, 14, 14, 20, 1, 2, 0), (2, 70, 14, 14, 100, 1, 2, 0), (2, 256, 10, 10, 32, 1, 2, 0), (2, 50, 12, 12, 96, 3, 2, 1),
    (1, 130, 10, 10, 512, 3, 1, 1), (1, 61, 9, 9, 640, 1, 1, 0), (2, 97, 13, 13, 324, 1, 2, 0),
]


@pytest.mark.parametrize("s", RAGGED, ids=str)
def test_ragged_results_of_every_addressing(s):
    d, x, w, dy = _data(s, 43)
    _within(gu.gpu_bwd_data(d, dy, w), _conv64_bwd(dy, w, s), _conv64_bwd(abs(dy), abs(w), s), s[4] * s[5] ** 2)
    _within(gu.gpu_bwd_weight(d, x, dy), _conv64_wgrad(x, dy, s), _conv64_wgrad(abs(x), abs(dy), s), dy.size // s[4])


def _plant(a, values, seed):
    a, rng = a.copy(), np.random.default_rng(seed)
    for v in values:
        a[tuple(rng.integers(0, m) for m in a.shape)] = v
    return a


NOT_FINITE = ([np.inf], [np.inf, -np.inf, np.nan], [np.finfo(np.float32).max], [np.float32(2.0 ** 120), np.float32(-2.0 ** 113)])


@pytest.mark.parametrize("s", RAGGED, ids=str)
def test_infinities_nans_and_the_largest_values_in_either_operand(s):
    """... of both passes: planted infinities, NaN, and values that the scaled split cannot carry come through as in fp32 arithmetic."""
    d, x, w, dy = _data(s, 47)
    x, w, dy = (a * np.float32(0.01) for a in (x, w, dy))             # keeps a sum around the largest value finite
    with np.errstate(over="ignore", invalid="ignore"):
        for i, values in enumerate(NOT_FINITE):
            for dy_, w_ in ((_plant(dy, values, i), w), (dy, _plant(w, values, i))):
                if s[5] > 1 and not np.isfinite(w_).all():
                    continue                # (taps outside the image: zero times the filter here, left out by the reference)
                ref, mag = _conv64_bwd(dy_, w_, s), _conv64_bwd(abs(dy_), abs(w_), s)
                got = gu.gpu_bwd_data(d, dy_, w_)
                ok = _same_where_not_finite(got, ref)
                _within(got[ok], ref[ok], mag[ok], s[4] * s[5] ** 2)
            for x_, dy_ in ((_plant(x, values, i), dy), (x, _plant(dy, values, i))):
                ref, mag = _conv64_wgrad(x_, dy_, s), _conv64_wgrad(abs(x_), abs(dy_), s)
                got = gu.gpu_bwd_weight(d, x_, dy_)
                ok = _same_where_not_finite(got, ref)
                _within(got[ok], ref[ok], mag[ok], dy.size // s[4], step=2)


def test_an_infinity_in_a_long_segment():
    """Whole tiles of 16 k-steps and splits of 16: the wave that meets the infinity computes its part again, the others keep theirs."""
    with np.errstate(over="ignore", invalid="ignore"):
        s = (32, 64, 56, 56, 512, 1, 1, 0)
        d, x, w, dy = _data(s, 53)
        dy = _plant(dy, [np.inf, -np.inf, np.nan], 1)
        a, b = dy.reshape(-1, 512).astype(np.float64), w.reshape(512, 64).astype(np.float64)
        ref, got = (a @ b).reshape(x.shape), gu.gpu_bwd_data(d, dy, w)
        ok = _same_where_not_finite(got, ref)
        _within(got[ok], ref[ok], (abs(a) @ abs(b)).reshape(x.shape)[ok], 512)
        s = (1, 1536, 64, 64, 1024, 1, 1, 0)
        d, x, w, dy = _data(s, 59)
        x = _plant(x, [np.inf, -np.inf, np.nan], 1)
        a, b = dy.reshape(-1, 1024).T.astype(np.float64), x.reshape(-1, 1536).astype(np.float64)
        ref, got = (a @ b).reshape(w.shape), gu.gpu_bwd_weight(d, x, dy)
        ok = _same_where_not_finite(got, ref)
        _within(got[ok], ref[ok], (abs(a) @ abs(b)).reshape(w.shape)[ok], 4096)


@pytest.mark.parametrize("s", [(3, 64, 13, 11, 128, 1, 1, 0), (2, 36, 9, 9, 65, 3, 1, 1), (2, 96, 14, 14, 132, 1, 2, 0)], ids=str)
def test_tensors_aligned_to_four_bytes_only(s):
    """The filter gradient's 8-byte loads and the 16-byte stores of backward-data's result on tensors that start 4 bytes past a 16-byte boundary."""
    d, x, w, dy = _data(s, 61)

    def off(a):
        t = torch.empty(a.size + 1, dtype=torch.float32, device=gu.DEV)
        t[1:].copy_(torch.from_numpy(a.reshape(-1)))
        return t[1:].view(a.shape)
    dw, dx = off(np.full_like(w, np.nan)), off(np.full_like(x, np.nan))
    lc.conv2d_bwd_weight(d, off(x), off(dy), dw, gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_WEIGHT)))
    lc.conv2d_bwd_data(d, gu.dev(dy), gu.dev(w), dx, gu.workspace(lc.conv2d_workspace_bytes(d, lc.LC_PASS_BWD_DATA)))
    torch.cuda.synchronize()
    _within(dw.cpu().numpy(), _conv64_wgrad(x, dy, s), _conv64_wgrad(abs(x), abs(dy), s), dy.size // s[4])
    _within(dx.cpu().numpy(), _conv64_bwd(dy, w, s), _conv64_bwd(abs(dy), abs(w), s), s[4] * s[5] ** 2)

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

# n, c, hw, k, window, stride; the tile, addressing and sharing of forward and of backward-data (phases: of the first)
SHAPES = [
    ((178, 24, 18, 136, 1, 1), "256x256 pieces", "128x32 pieces"),
    ((65, 64, 30, 136, 1, 1), "256x256 chunks", "conv_gemm_pk 128x64"),
    ((34, 64, 30, 288, 1, 1), "240x256 chunks", "conv_gemm_pk 128x64"),
    ((39, 24, 28, 272, 1, 1), "240x256 pieces", "128x32 pieces"),
    ((107, 64, 23, 136, 1, 1), "224x256 chunks", "conv_gemm_pk 128x64"),
    ((136, 24, 14, 264, 1, 1), "224x256 pieces", "128x32 pieces"),
    ((64, 64, 20, 264, 1, 1), "208x256 chunks", "conv_gemm_pk 128x64"),
    ((148, 24, 13, 264, 1, 1), "208x256 pieces", "128x32 pieces"),
    ((57, 64, 24, 152, 1, 1), "192x256 chunks", "conv_gemm_pk 128x64"),
    ((53, 24, 25, 136, 1, 1), "192x256 pieces", "128x32 pieces"),
    ((4, 256, 14, 256, 3, 1), "128x64 chunks shared", "128x64 chunks shared"),
    ((91, 24, 11, 136, 1, 1), "128x128 pieces", "128x32 pieces"),
    ((48, 64, 19, 72, 1, 1), "128x128 chunks", "conv_gemm_pk 128x64"),
    ((4, 256, 26, 200, 3, 1), "128x128 chunks shared", "128x64 pieces"),
    ((4, 504, 26, 72, 3, 1), "128x128 padded shared", "128x64 pieces"),
    ((7, 216, 28, 80, 3, 1), "128x128 pieces shared", "128x64 pieces"),
    ((9, 216, 25, 68, 3, 1), "128x128 pieces shared", "conv_gemm_split"),
    ((21, 576, 8, 104, 3, 1), "128x64 chunks shared", "128x64 pieces"),
    ((76, 296, 6, 72, 3, 1), "128x64 pieces shared", "128x64 pieces"),
    ((2, 504, 7, 72, 3, 1), "128x64 padded shared", "128x64 pieces"),      # 504 channels as 512
    ((37, 64, 7, 64, 5, 1), "128x64 chunks shared", "128x64 chunks shared"),
    ((7, 208, 5, 16, 3, 1), "128x32 pieces shared", "128x64 pieces"),
    ((2, 128, 5, 16, 3, 1), "128x32 chunks shared", "128x64 pieces"),
    ((1, 504, 3, 24, 3, 1), "128x32 padded shared", "128x64 pieces"),
    ((1, 240, 3, 20, 3, 1), "128x32 pieces shared", "conv_gemm_split"),
    ((9, 312, 30, 134, 3, 1), "128x64 padded", "conv_gemm"),
    ((40, 24, 41, 40, 5, 1), "128x64 two waves pieces", "128x32 pieces"),
    ((233, 128, 12, 56, 1, 1), "128x64 two waves chunks", "128x128 pieces"),
    ((54, 128, 25, 41, 1, 1), "128x64 two waves chunks", "conv_gemm"),
    ((43, 192, 23, 48, 5, 1), "128x64 two waves chunks shared", "128x128 pieces"),
    ((13, 496, 29, 33, 5, 1), "128x64 two waves pieces shared", "conv_gemm"),
    ((57, 128, 24, 16, 1, 1), "128x32 chunks", "conv_gemm_pk 128x128"),
    ((40, 32, 31, 32, 5, 1), "128x32 pieces", "128x32 pieces"),
    ((112, 544, 30, 56, 1, 1), "128x64 pieces", "256x256 pieces"),
    ((3, 64, 1, 1000, 1, 1), "128x64 chunks", "128x64 pieces"),      # a fully connected layer of a few rows
    ((5, 72, 9, 33, 3, 1), "128x64 pieces", "conv_gemm"),      # filter counts off the vector stores
    ((3, 64, 10, 130, 1, 1), "128x64 chunks", "conv_gemm"),
    ((2, 64, 13, 35, 3, 1), "128x64 chunks", "conv_gemm"),
    ((6, 64, 15, 136, 1, 2), "128x64 chunks", "128x64 pieces"),      # stride grids: one pixel in four, and the four phases of a window
    ((5, 72, 11, 40, 3, 2), "128x64 pieces", "128x64 pieces"),
    ((3, 16, 12, 264, 3, 2), "128x64 pieces", "128x32 pieces"),
    ((2, 256, 9, 8, 5, 3), "128x32 chunks shared", "128x64 pieces"),
    ((4, 37, 10, 64, 1, 2), "conv_gemm_pk 128x64", "128x64 chunks"),      # stride grids of odd and of even counts of channels
    ((3, 38, 9, 64, 3, 2), "128x64 pieces", "128x64 chunks"),
]
# windows of more than 32 taps: n, c, h, w, k, r, s, stride, pad_h, pad_w; the kernel of forward and of backward-data
LARGE_WINDOWS = [
    ((3, 64, 15, 14, 136, 7, 7, 1, 3, 3), "conv_dma 128x64 runs shared", "conv_dma 128x64 taps shared"),       # runs of 28 and 21 taps, split between blocks
    ((1, 504, 7, 7, 72, 7, 7, 1, 3, 3), "conv_dma 128x64 runs shared", "conv_dma 128x64 taps shared"),
    ((2, 40, 12, 13, 72, 7, 7, 1, 3, 3), "conv_dma 128x64 taps shared", "conv_dma 128x64 taps shared"),          # pieces of several taps in a k-step
    ((60, 64, 31, 31, 136, 3, 11, 1, 1, 5), "conv_dma 256x256 runs", "conv_dma 128x64 taps"),
    ((60, 8, 33, 33, 264, 6, 6, 1, 2, 3), "conv_dma 256x256 taps", "conv_dma 128x64 taps"),
    ((20, 128, 20, 20, 128, 7, 7, 1, 3, 3), "conv_dma 128x128 runs shared", "conv_dma 128x128 runs shared"),
    ((2, 64, 3, 50, 72, 1, 35, 1, 0, 20), "conv_dma 128x64 runs shared", "conv_dma 128x64 taps shared"),       # runs of 32 and 3 taps of a row; more padding than half of it
    ((2, 64, 6, 90, 64, 2, 70, 1, 1, 30), "conv_dma 128x64 runs shared", "conv_dma 128x64 runs shared"),
    ((2, 64, 50, 3, 64, 37, 1, 1, 18, 0), "conv_dma 128x64 runs shared", "conv_dma 128x64 runs shared"),
    ((2, 24, 50, 3, 40, 37, 1, 1, 18, 0), "conv_dma 128x64 taps", "conv_dma 128x64 taps shared"),
    ((3, 64, 5, 4, 72, 9, 9, 1, 4, 4), "conv_dma 128x64 runs shared", "conv_dma 128x64 taps shared"),          # larger than the image
    ((3, 16, 21, 19, 40, 13, 13, 2, 6, 6), "conv_dma 128x64 taps shared", "conv_dma 128x64 taps shared"),        # four phases of up to 49 taps
    ((2, 37, 16, 16, 64, 13, 12, 2, 5, 6), "conv_dma 128x64 taps shared", "conv_dma 128x64 runs shared"),      # odd counts of columns
    ((2, 64, 11, 11, 33, 7, 7, 1, 3, 3), "conv_dma 128x64 runs shared", "conv_gemm"),
]


NON_FINITE = [((4, 64, 14, 14, 136, 3, 3, 1, 1, 1), "chunks"), ((2, 504, 7, 7, 72, 3, 3, 1, 1, 1), "padded"), ((3, 40, 9, 9, 72, 3, 3, 1, 1, 1), "pieces"),
              ((2, 64, 9, 9, 72, 7, 7, 1, 3, 3), "runs"), ((2, 40, 9, 9, 72, 7, 7, 1, 3, 3), "taps"), ((4, 64, 15, 15, 136, 1, 1, 2, 0, 0), "chunks")]


@pytest.mark.parametrize("case", NON_FINITE, ids=str)
def test_infinities_and_nan_stay_where_they_are(case):
    """In the first and the last channel (beside those filled up with zeros), at corners (beside taps outside the image) and in the last pixel (beside rows past the
    end): they reach the float64 result's places and no others, and a missing filter value its own filter and that filter's statistics."""
    (n, c, h, w, k, r, s, st, ph, pw), form = case
    d = lc.ConvDesc(n, c, h, w, k, r, s, st, st, ph, pw, lc.LC_BF16, lc.LC_NHWC)
    assert gu.route(d, lc.LC_PASS_FWD).startswith("conv_dma") and form in gu.route(d, lc.LC_PASS_FWD).split()
    p, q = lc.conv2d_out_shape(d)
    g = torch.Generator().manual_seed(37)
    x, dy = torch.randn((n, h, w, c), generator=g).to(torch.bfloat16), torch.randn((n, p, q, k), generator=g).to(torch.bfloat16)
    wt = (torch.randn((k, r, s, c), generator=g) / (c * r * s) ** 0.5).to(torch.bfloat16)
    for t in (x, dy):
        t[0, 0, 0, -1] = t[1, 0, -1, 0] = float("inf")
        t[-1, -1, -1, -1] = float("nan")

    def run(fn, which, a, b, shape):
        out, guard = gu.guarded(shape, torch.bfloat16)
        fn(d, a.to(gu.DEV), b.to(gu.DEV), out, gu.workspace(lc.conv2d_workspace_bytes(d, which)))
        torch.cuda.synchronize()
        guard()
        return out.cpu()

    def check(got, ref):
        for kind in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(kind(got), kind(ref)), kind
        ok = torch.isfinite(ref)
        assert bool(((got.double() - ref).abs()[ok] <= 2.0 ** -7 * ref.abs()[ok] + 1e-4).all())

    nchw = lambda t: t.double().permute(0, 3, 1, 2)                                                                          # noqa: E731
    check(run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, wt, dy.shape), F.conv2d(nchw(x), nchw(wt), stride=st, padding=(ph, pw)).permute(0, 2, 3, 1))
    check(run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, wt, x.shape),
          torch.nn.grad.conv2d_input((n, c, h, w), nchw(wt), nchw(dy), stride=st, padding=(ph, pw)).permute(0, 2, 3, 1))

    x = torch.randn((n, h, w, c), generator=g).to(torch.bfloat16)
    wt[k // 2, 0, 0, c - 1] = float("nan")
    stats, guard = gu.guarded((lc.conv2d_fwd_stats_count(d), k, 2), torch.float32)
    y = run(lambda d_, a, b, out, ws: lc.conv2d_fwd_stats(d_, a, b, out, stats, ws), lc.LC_PASS_FWD, x, wt, dy.shape)
    guard()
    others = [i for i in range(k) if i != k // 2]
    assert torch.isnan(y[..., k // 2]).all() and torch.isfinite(y[..., others]).all()
    rows, sums = y.double().reshape(-1, k)[:, others], stats.cpu().double().sum(0)
    assert torch.isnan(sums[k // 2]).all()
    assert bool(((sums[others, 0] - rows.sum(0)).abs() <= 2e-5 * rows.abs().sum(0) + 1e-30).all())


def _check(d, seed=17):
    n, c, k, r, s, st, pad = d.n, d.c, d.k, d.r, d.s, (d.stride_h, d.stride_w), (d.pad_h, d.pad_w)
    g = torch.Generator().manual_seed(seed)
    p, q = lc.conv2d_out_shape(d)
    x = torch.randn((n, d.h, d.w, c), generator=g).to(torch.bfloat16)
    w = (torch.randn((k, r, s, c), generator=g) / (c * r * s) ** 0.5).to(torch.bfloat16)
    dy = torch.randn((n, p, q, k), generator=g).to(torch.bfloat16)

    def run(fn, which, a, b, shape):
        out, guard = gu.guarded(shape, torch.bfloat16)
        ws = gu.workspace(lc.conv2d_workspace_bytes(d, which))
        fn(d, a.to(gu.DEV), b.to(gu.DEV), out, ws)
        torch.cuda.synchronize()
        guard()
        return out.cpu()

    def check(got, ref, mag, terms):
        bound = 2.0 ** -8 * ref.abs() + (-(-terms // 8) + 66) * 2.0 ** -23 * mag
        assert bool(((got.double() - ref).abs() <= bound).all()), float(((got.double() - ref).abs() / (mag + 1e-30)).max())

    xn, wn, dyn = (t.double().permute(0, 3, 1, 2) for t in (x, w, dy))
    fwd = lambda a, b: F.conv2d(a, b, stride=st, padding=pad).permute(0, 2, 3, 1)                                             # noqa: E731
    bwd = lambda a, b: torch.nn.grad.conv2d_input(xn.shape, b, a, stride=st, padding=pad).permute(0, 2, 3, 1)                 # noqa: E731
    y = run(lc.conv2d_fwd, lc.LC_PASS_FWD, x, w, dy.shape)
    check(y, fwd(xn, wn), fwd(xn.abs(), wn.abs()), c * r * s)
    check(run(lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, dy, w, x.shape), bwd(dyn, wn), bwd(dyn.abs(), wn.abs()), k * r * s)

    # with statistics: the same bits, and per column the sums of what was stored
    count = lc.conv2d_fwd_stats_count(d)
    assert count > 0
    stats, guard = gu.guarded((count, k, 2), torch.float32)
    y2 = run(lambda d_, a, b, out, ws: lc.conv2d_fwd_stats(d_, a, b, out, stats, ws), lc.LC_PASS_FWD, x, w, dy.shape)
    guard()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    rows, got = y.double().reshape(-1, k), stats.cpu().double().sum(0)
    assert bool(((got[:, 0] - rows.sum(0)).abs() <= 2e-5 * rows.abs().sum(0) + 1e-30).all())
    assert bool(((got[:, 1] - rows.square().sum(0)).abs() <= 2e-5 * rows.square().sum(0) + 1e-30).all())


@pytest.mark.parametrize("s,fwd,bwd", SHAPES, ids=str)
def test_matches_float64(s, fwd, bwd):
    n, c, hw, k, r, st = s
    d = lc.ConvDesc(n, c, hw, hw, k, r, r, st, st, r // 2, r // 2, lc.LC_BF16, lc.LC_NHWC)
    print(f"conv dma {s}", flush=True)
    assert [gu.route(d, which).removeprefix("conv_dma ") for which in (lc.LC_PASS_FWD, lc.LC_PASS_BWD_DATA)] == [fwd, bwd]
    _check(d)


# images of a gibibyte: n, c, h, w, k, window, stride; the kernel of forward and, of the layer with c and k exchanged, of backward-data
FAR = [
    ((2, 64, 2950, 2900, 40, 3, 1), "conv_gemm_pk 256x64", "conv_gemm_pk 256x64"),
    ((2, 64, 2950, 2900, 72, 3, 1), "conv_dma 128x128 runs", "conv_dma 128x128 runs"),
    ((2, 40, 3300, 4200, 72, 3, 1), "conv_dma 128x128 taps", "conv_dma 128x128 taps"),
    ((2, 72, 2800, 2700, 264, 1, 1), "conv_dma 256x256 taps", "conv_dma 256x256 taps"),
    ((2, 128, 2100, 2050, 136, 3, 2), "conv_dma 256x256 runs", None),
]


@pytest.mark.parametrize("case", FAR, ids=str)
def test_images_of_a_gibibyte(case):
    """Small whole numbers, whose sums are exact in fp32: the float64 sums, rounded once.  The second image starts inside a tile."""
    (n, c, h, w, k, r, st), fwd, bwd = case
    g = torch.Generator(device=gu.DEV).manual_seed(19)
    numbers = lambda *t: torch.randint(-1, 2, t, generator=g, device=gu.DEV, dtype=torch.int8).to(torch.bfloat16)        # noqa: E731

    def run(d, fn, which, a, b, shape):
        out, guard = gu.guarded(shape, torch.bfloat16)
        fn(d, a, b, out, gu.workspace(lc.conv2d_workspace_bytes(d, which)))
        torch.cuda.synchronize()
        guard()
        return out

    def check(got, a, b):                                # b [k, r, s, c]
        p, q = got.shape[1:3]
        for i in range(n):
            pad = F.pad(a[i], (0, 0, r // 2, r // 2, r // 2, r // 2))
            for p0 in range(0, p, 256):
                m = min(256, p - p0)
                ref = sum(pad[u + st * p0:u + st * (p0 + m - 1) + 1:st, v:v + st * (q - 1) + 1:st].reshape(m * q, -1).double() @ b[:, u, v].double().t().contiguous()
                          for u in range(r) for v in range(r))
                assert torch.equal(got[i, p0:p0 + m].view(m * q, -1), ref.to(torch.bfloat16)), (i, p0)

    d = lc.ConvDesc(n, c, h, w, k, r, r, st, st, r // 2, r // 2, lc.LC_BF16, lc.LC_NHWC)
    print(f"conv dma far {d}", flush=True)
    assert gu.route(d, lc.LC_PASS_FWD) == fwd
    x, wt = numbers(n, h, w, c), numbers(k, r, r, c)
    check(run(d, lc.conv2d_fwd, lc.LC_PASS_FWD, x, wt, (n, *lc.conv2d_out_shape(d), k)), x, wt)
    if bwd:
        e = lc.ConvDesc(n, k, h, w, c, r, r, st, st, r // 2, r // 2, lc.LC_BF16, lc.LC_NHWC)
        assert gu.route(e, lc.LC_PASS_BWD_DATA) == bwd
        got = run(e, lc.conv2d_bwd_data, lc.LC_PASS_BWD_DATA, x, wt.permute(3, 1, 2, 0).contiguous(), (n, h, w, k))
        check(got, x, wt.flip(1, 2).contiguous())


@pytest.mark.parametrize("case", LARGE_WINDOWS, ids=str)
def test_windows_of_more_than_32_taps(case):
    (n, c, h, w, k, r, s, st, ph, pw), fwd, bwd = case
    d = lc.ConvDesc(n, c, h, w, k, r, s, st, st, ph, pw, lc.LC_BF16, lc.LC_NHWC)
    assert gu.route(d, lc.LC_PASS_FWD) == fwd and gu.route(d, lc.LC_PASS_BWD_DATA) == bwd
    print(f"conv dma large window {d}", flush=True)
    _check(d)

"""Which kernel the library sends a layer to, asked on the host (no GPU): every form of a bf16 window that the kernel with operands straight into LDS is built for
reaches it, in both passes and at every size a call can have, and the running sums of its filter gradients are as short as promised."""
import itertools
import random
import re

import pytest

from paper_1709_05011_amd import larsconv as lc

import gpu_util as gu


def _desc(n, c, h, w, k, r, s, stride, ph, pw):
    return lc.ConvDesc(n, c, h, w, k, r, s, stride, stride, ph, pw, lc.LC_BF16, lc.LC_NHWC)


@pytest.mark.parametrize("window", [(6, 6), (7, 7), (3, 11), (1, 33), (33, 1), (2, 40), (15, 15), (17, 31)], ids=str)
@pytest.mark.parametrize("stride", [1, 2, 3])
def test_windows_of_more_than_32_taps(window, stride):
    """Also as the phases of a strided window, which would otherwise be widened to fp32."""
    r, s = window
    for n, c, k in itertools.product((1, 7, 256), (8, 40, 64, 96, 504, 512), (8, 64, 200, 256, 1024)):
        d = _desc(n, c, 40, 44, k, r, s, stride, r // 2, s // 2)
        for which in (lc.LC_PASS_FWD, lc.LC_PASS_BWD_DATA):
            assert gu.route(d, which).startswith("conv_dma"), (d, which)
        assert gu.route(d, lc.LC_PASS_FWD, stats=True).startswith("conv_dma")
        assert lc.conv2d_fwd_stats_count(d) > 0


@pytest.mark.parametrize("c,k,r,stride", [(256, 256, 1, 1), (64, 72, 1, 1), (64, 64, 3, 1), (128, 256, 3, 1), (40, 40, 3, 1), (64, 128, 3, 2), (40, 24, 5, 1)])
def test_images_of_half_a_gibibyte_and_more(c, k, r, stride):
    """Two of them span more than the 2 GiB that a buffer's offsets reach; a tile does not.  At most 64 columns are faster in the main kernel's tile of 256 rows."""
    kernel = "conv_gemm_pk 256x64" if k <= 64 else "conv_dma"
    hw = int((1.2 * 2 ** 29 / c) ** 0.5)
    for n in (1, 3):
        d = _desc(n, c, hw, hw, k, r, r, stride, r // 2, r // 2)
        assert gu.route(d, lc.LC_PASS_FWD).startswith(kernel) and gu.route(d, lc.LC_PASS_FWD, stats=True).startswith(kernel)
        if stride == 1:
            assert gu.route(_desc(n, k, hw, hw, c, r, r, 1, r // 2, r // 2), lc.LC_PASS_BWD_DATA).startswith(kernel)


@pytest.mark.parametrize("c,k", [(64, 72), (64, 160), (256, 256), (512, 96)])
def test_filter_gradients_of_plain_layers_on_large_images(c, k):
    """A 1x1 layer's filter gradient reads rows of pixels, whatever image they are in: images of half a gibibyte and more are like any other."""
    hw = int((1.2 * 2 ** 29 / c) ** 0.5)
    for n in (1, 3):
        assert gu.route(_desc(n, c, hw, hw, k, 1, 1, 1, 0, 0), lc.LC_PASS_BWD_WEIGHT).startswith("wgrad_dma")


def _former_splits(d, rows):
    """The splits of the kernels that staged operands through registers: one round of 256 compute units with 4, 5 or 8 blocks each, 256 rows at least; 3x3 layers
    over multiples of 64 channels on wide images in two blocks per unit of 64 filters x 64 channels x nine taps."""
    j = d.r * d.s * d.c
    tiles = -(-d.k // (128 if d.k > 64 else 64)) * -(-j // (128 if j > 64 else 64))
    splits = min((4 if d.k > 64 and j > 64 else 8 if d.k <= 64 and j <= 64 else 5) * 256 // tiles, -(-rows // 256))
    if (d.r, d.s, d.stride_h, d.pad_h) == (3, 3, 1, 1) and d.c % 64 == 0 and d.k % 64 == 0 and d.w >= 24:
        splits = max(splits, min(512 // (d.c // 64 * (d.k // 64)), -(-d.n * (d.h + 1) * (d.w + 2) // 256)))
    return max(splits, 1)


def _additions(parts):
    """Adding equal parts in four interleaved sums: the share of the whole that each addition's result holds, summed."""
    each = parts // 4
    sums = [each + parts % 4, each, each, each]
    serial = sum(n * (n + 1) // 2 - 1 for n in sums if n)
    return (serial + (2 * parts if each else 0)) / parts


def test_sums_of_the_filter_gradient_are_no_longer_than_before():
    """The error of a sum in fp32 grows with the root of its rows.  No running sum holds more rows than a split of the former kernels did; one split in the
    place of several, whose additions are saved, may hold the 64 rows more per addition of everything that round as often."""
    rng, seen = random.Random(3), set()
    for _ in range(4000):
        unit = rng.choice([8, 32, 64])
        c, k = (max(unit, int(2 ** rng.uniform(3, 11)) // unit * unit) for _ in range(2))
        n, hw, r = int(2 ** rng.uniform(0, 9)), int(2 ** rng.uniform(2, 7)), rng.choice([1, 1, 3, 3, 3, 5])
        stride = rng.choice([1, 1, 1, 2])
        d = _desc(n, c, hw, hw, k, r, r, stride, r // 2, r // 2)
        m = re.fullmatch(r"wgrad_dma (\d+x\d+) splits (\d+) sums (\d+)", gu.route(d, lc.LC_PASS_BWD_WEIGHT))
        if not m:
            continue
        splits, sums = int(m[2]), int(m[3])
        p, q = lc.conv2d_out_shape(d)
        rows = n * p * q
        former = _former_splits(d, rows)
        limit = -(-rows // former)
        if splits == 1:
            limit += max(0.0, 64 * (_additions(former) - 1))
        assert sums <= limit, (d, m[0], former)
        seen.add(m[1])
    assert seen == {"256x256", "256x128", "128x256", "128x128", "256x64", "64x256", "128x64", "64x128"}


def test_few_columns_and_short_reductions_stay_with_the_main_kernel():
    for (n, c, hw, k, r), kernel in (((31, 16, 103, 48, 1), "conv_gemm_pk 128x64"), ((505, 32, 63, 32, 1), "conv_gemm_pk 256x64"), ((55, 16, 115, 48, 3), "conv_gemm_pk 128x64"),
                                     ((76, 64, 58, 64, 1), "conv_gemm_pk 128x64"), ((153, 64, 87, 64, 1), "conv_dma"), ((512, 64, 56, 64, 1), "conv_dma"),
                                     ((25, 16, 81, 16, 3), "conv_dma"), ((31, 24, 103, 72, 1), "conv_dma"), ((328, 16, 21, 608, 1), "conv_gemm_pk 128x128")):
        d = _desc(n, c, hw, hw, k, r, r, 1, r // 2, r // 2)
        assert gu.route(d, lc.LC_PASS_FWD).startswith(kernel), (d, gu.route(d, lc.LC_PASS_FWD))
        assert gu.route(d, lc.LC_PASS_FWD, stats=True).startswith(kernel)
        assert gu.route(_desc(n, k, hw, hw, c, r, r, 1, r // 2, r // 2), lc.LC_PASS_BWD_DATA).startswith(kernel)


def _layer(n, c, hw, k, r=1, stride=1, dtype=lc.LC_BF16, layout=lc.LC_NHWC):
    return lc.ConvDesc(n, c, hw, hw, k, r, r, stride, stride, r // 2, r // 2, dtype, layout)


@pytest.mark.parametrize("d,fwd,bwd", [
    (_layer(512, 128, 28, 512), True, True),
    (_layer(512, 256, 14, 256, 3), False, False),                       # 51 MB
    (_layer(512, 64, 56, 104), False, True),                            # rows of 208 bytes
    (_layer(512, 16, 56, 64), True, False),                             # two waves fill a line; rows of 32 bytes
    (_layer(512, 16, 28, 128), False, False),                           # reductions of 16 values to 128 columns: products that end before their stores
    (_layer(512, 8, 28, 256), False, False),
    (_layer(512, 16, 28, 640), False, False),
    (_layer(512, 128, 28, 128, 3, layout=lc.LC_NCHW), False, False),    # 103 MB that a transpose reads next
    (_layer(512, 128, 28, 512, layout=lc.LC_NCHW), True, False),        # 411 MB, 103 MB
    (_layer(256, 128, 28, 512, dtype=lc.LC_F32, layout=lc.LC_NCHW), True, False),
    (_layer(256, 128, 28, 512, dtype=lc.LC_F32), True, True),
    (_layer(256, 3, 224, 64, 7, 2), True, False),                       # the first layer, images of 77, 154 and 5 MB
    (_layer(512, 3, 224, 64, 7, 2), False, False),
    (_layer(16, 3, 224, 64, 7, 2), False, False),
], ids=str)
def test_results_that_go_past_the_caches(d, fwd, bwd):
    assert gu.route(d, lc.LC_PASS_FWD, form=True).endswith(" past") == fwd
    assert gu.route(d, lc.LC_PASS_BWD_DATA, form=True).endswith(" past") == bwd


@pytest.mark.parametrize("d,past", [(_layer(512, 512, 28, 1024, 1, 2), True), (_layer(256, 512, 28, 1024, 1, 2, lc.LC_F32), False),
                                    (_layer(256, 256, 56, 512, 1, 2, lc.LC_F32), False), (_layer(128, 512, 28, 256, 1, 2, lc.LC_F32), True),
                                    (_layer(64, 64, 56, 128, 1, 2, lc.LC_F32), False), (_layer(512, 64, 56, 64, 1, 2, lc.LC_F32), True)], ids=str)
def test_zeros_between_a_stride_grid_that_go_past_the_caches(d, past):
    """Not before a long fp32 product, nor where the caches hold them."""
    assert gu.route(d, lc.LC_PASS_BWD_DATA, form=True).endswith(", zeros past") == past


def test_shapes_of_few_blocks_meet_every_form():
    import test_gpu_conv_deep as deep

    seen = set()
    for n, h, w, c, k, r, s in deep.LAYERS:
        d = _desc(n, c, h, w, k, r, r, s, r // 2, r // 2)
        for which, out, columns, stats in ((lc.LC_PASS_FWD, "rows", k, False), (lc.LC_PASS_FWD, "stats", k, True), (lc.LC_PASS_BWD_DATA, "rows" if s == 1 else "grid", c, False)):
            m = re.fullmatch(r"conv_dma (128x\d+) (\w+)( shared)? four stages", gu.route(d, which, stats, form=True))
            if m:
                seen.add((m[1], m[2], out if columns % 8 == 0 or out != "rows" else "any", bool(m[3])))
        if "eight waves" in gu.route(d, lc.LC_PASS_BWD_WEIGHT, form=True):
            seen.add("eight waves")
    want = {"eight waves"} | {(t, i, o, True) for t in ("128x64", "128x128") for i in ("chunks", "padded") for o in ("rows", "stats")}
    want |= {(t, i, o, False) for t in ("128x64", "128x128") for i, o in (("chunks", "rows"), ("chunks", "stats"), ("chunks", "any"), ("pieces", "rows"), ("pieces", "stats"), ("chunks", "grid"))}
    want |= {("128x128", "pieces", "rows", True), ("128x128", "chunks", "any", True)}
    assert not want - seen, want - seen


def test_shapes_past_the_caches_meet_every_form():
    import test_gpu_conv_stream as stream

    seen = {lc.LC_BF16: set(), lc.LC_F32: set()}
    for dtype, forms in seen.items():
        for n, h, w, c, k in stream.POINTWISE:
            d = lc.ConvDesc(n, c, h, w, k, 1, 1, 1, 1, 0, 0, dtype, lc.LC_NHWC)
            forms |= {("fwd", gu.route(d, lc.LC_PASS_FWD, form=True)), ("bwd", gu.route(d, lc.LC_PASS_BWD_DATA, form=True)),
                      ("dw", re.sub(r" splits.*sums \d+", "", gu.route(d, lc.LC_PASS_BWD_WEIGHT, form=True)))}
        for n, h, w, c, k, r, s in stream.WINDOWS:
            if s == 2 and r == 1:
                c, k = k, c
            d = lc.ConvDesc(n, c, h, w, k, r, r, s, s, r // 2, r // 2, dtype, lc.LC_NHWC)
            forms |= {("fwd", gu.route(d, lc.LC_PASS_FWD, form=True)), ("bwd", gu.route(d, lc.LC_PASS_BWD_DATA, form=True))}
            if s == 2 and r > 1 and r < 7:
                forms.add(("phases", gu.route(d, lc.LC_PASS_BWD_DATA, form=True)))
    want = {("dw", f"wgrad_dma {t} around") for t in ("64x128", "128x64", "256x64", "64x256", "256x128", "128x256", "128x128", "256x256", "128x128 eight waves")}
    want |= {("dw", "wgrad_dma 128x128 eight waves")}
    want |= {("fwd", f"conv_dma {t} chunks once{p}") for t, p in (("128x64 two waves", ""), ("128x128", ""), ("128x32", ""), ("256x256", " past"))}
    want |= {("bwd", "conv_dma 128x32 chunks once"), ("bwd", "conv_dma 128x128 chunks once past")}
    want |= {("fwd", f"{f} past") for f in ("conv3x3_held", "conv3x3_slab", "conv_gemm_pk 256x64", "conv_gemm_pk 128x64", "conv_dma 128x64 two waves chunks", "conv_dma 128x128 chunks",
                                            "conv_dma 128x128 pieces", "conv_dma 256x256 chunks", "conv_dma 224x256 chunks", "conv_dma 240x256 chunks", "conv_dma 224x256 pieces", "conv_stem")}
    want |= {("bwd", "conv3x3_held past"), ("bwd", "conv_dma 128x128 chunks past, zeros past"), ("phases", "conv_dma 128x128 chunks past")}
    assert not want - seen[lc.LC_BF16], want - seen[lc.LC_BF16]
    want = {("fwd", "conv_stem past"), ("fwd", "conv_gemm_pk 128x64 past"), ("fwd", "conv_gemm_pk 128x128 past"), ("bwd", "conv_gemm_split past"), ("bwd", "conv_gemm_split past, zeros past"),
            ("phases", "conv_gemm_split past")}
    assert not want - seen[lc.LC_F32], want - seen[lc.LC_F32]


def test_filter_gradients_round_the_splits():
    """Large operands, one tile of which they fill three fifths; eight waves where a split is short."""
    for (n, hw, c, k, r), form in (((319, 56, 128, 64, 1), "around"), ((160, 56, 128, 64, 1), "around"), ((512, 28, 128, 64, 1), ""), ((512, 28, 96, 64, 1), ""), ((512, 56, 72, 72, 1), ""),
                                   ((512, 56, 72, 32, 1), ""), ((512, 56, 64, 256, 1), ""), ((37, 7, 512, 512, 3), "eight waves"), ((96, 21, 256, 448, 1), "eight waves"),
                                   ((256, 56, 200, 72, 1), ""), ((512, 28, 512, 128, 1), "")):
        m = re.fullmatch(r"wgrad_dma (\d+x\d+) splits \d+ sums \d+ ?(.*)", gu.route(_layer(n, c, hw, k, r), lc.LC_PASS_BWD_WEIGHT, form=True))
        assert m and m[2] == form, (n, hw, c, k, r, m and m[0])


@pytest.mark.parametrize("d,once", [(_layer(512, 512, 28, 128), True), (_layer(512, 256, 56, 64), True), (_layer(512, 64, 112, 32), False), (_layer(800, 64, 56, 64), False),
                                    (_layer(512, 128, 28, 128, 3), False), (_layer(256, 512, 28, 128), False), (_layer(512, 512, 28, 512), False)], ids=str)
def test_rows_read_once_come_past_the_caches(d, once):
    """Images of 256 MB and more under a 1x1 window of two k-steps and more, one tile of columns."""
    assert (" once" in gu.route(d, lc.LC_PASS_FWD, form=True)) == once

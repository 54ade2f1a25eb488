"""GPU parity of lars_step on a list long enough for the update pass that goes past the caches (12 million parameters and more): tensors that start
on a line of 128 bytes, on 16 bytes and on 4 bytes, sizes that end within a chunk, within a wave's vector and in single elements, with and
without bf16 copies; the same tensors in a short list, which take the ordinary accesses; and lists whose longest tensor fills part of a chunk, which
have blocks for that part only.  Reference: float64 on the device.  The ratio is
within 1e-6; v = momentum * v + ratio * (g + decay * w) is off by 1e-6 of the sum of its terms' sizes (that ratio's few roundings and its own four; in a tensor of one element
the terms may cancel), w = w - v by one more rounding, 4e-7 in all of the terms."""
import pytest
import torch

from paper_1709_05011_amd import larsconv as lc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ETA, MOMENTUM, DECAY, LR = 0.001, 0.9, 5e-4, 0.7


@pytest.mark.parametrize("big", [0, 13_000_003])
def test_update_matches_float64(big):
    _check([(300_000, 0), (70_001, 4), (4096, 1), (257, 0), (256, 4), (3, 0), (0, 0), (123_459, 2)] + ([(big, 0)] if big else []))


@pytest.mark.parametrize("longest", [1, 255, 256, 257, 512, 513, 1000, 1025, 2048, 2049, 4096, 4097])
def test_lists_of_short_tensors(longest):
    _check([(1, 0), (longest, 0), (0, 0), (max(1, longest - 1), 4), (longest, 1), (max(1, longest // 3), 0)] + [(max(1, longest - i), 0) for i in range(150)])


def _check(sizes):
    g = torch.Generator(device=DEV).manual_seed(3)
    made = []
    for m, off in sizes:                                           # off: floats past a 512-byte boundary
        made.append([torch.randn(m + off, generator=g, device=DEV).mul_(std)[off:] for std in (0.05, 1e-3, 1e-4)])
    w, gr, v = ([t[i] for t in made] for i in range(3))
    low = [torch.zeros(m + off, dtype=torch.bfloat16, device=DEV)[off:] if i % 2 == 0 else None for i, (m, off) in enumerate(sizes)]
    ref = []
    for a, b, c in made:
        a, b, c = a.double(), b.double(), c.double()
        nw, ng = a.norm(), b.norm()
        t = float(ETA * nw / (ng + DECAY * nw)) if a.numel() and nw > 0 else 1.0
        nv = MOMENTUM * c + LR * t * (b + DECAY * a)
        terms = MOMENTUM * c.abs() + LR * t * (b.abs() + DECAY * a.abs())
        ref.append((t, nv, a - nv, terms, terms + a.abs()))
    args = lc.LarsArgs(w, gr, v, w_lowp=low)
    trust = torch.empty(len(sizes), device=DEV)
    ws = torch.empty(lc.lars_workspace_bytes(args.numel), dtype=torch.uint8, device=DEV)
    lc.lars_step(args, ETA, MOMENTUM, DECAY, LR, trust, ws)
    for i, (t, nv, nw, v_terms, w_terms) in enumerate(ref):
        assert abs(trust[i].item() - t) <= 1e-6 * t
        if not nv.numel():
            continue
        assert (v[i].double() - nv).abs().max().item() <= 1e-6 * v_terms.max().item()
        assert (w[i].double() - nw).abs().max().item() <= 4e-7 * w_terms.max().item()
        if low[i] is not None:
            assert torch.equal(low[i], w[i].to(torch.bfloat16))

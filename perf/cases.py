"""The work a user of this library has it do, as measurable cases: single convolution layers through their three passes,
a convolution with its batch norm, a batch norm, the LARS update, and whole ResNet-50 training steps.

listed() names twelve of them at the sizes of this repository's own networks (ResNet-50 at the per-GPU batches of the
benchmark, 256 images in fp32 and 512 in bf16; one worker's smallest calls; a ragged batch); draw() gives others of the same
ranges.  prepare() makes what a training program holds before the call (tensors, workspace, argument lists), run() is one
pass through the public entry points of paper_1709_05011_amd, exact() the same results in 64-bit arithmetic from plain torch.
"""
import math

import torch
import torch.nn.functional as F

from paper_1709_05011_amd import larsconv as lc
from paper_1709_05011_amd import resnet_step
from paper_1709_05011_amd import synth

DEV = "cuda:0"
NHWC = lc.LC_NHWC
EPS = 1e-5
ETA, MOMENTUM, DECAY, LR = 0.001, 0.9, 5e-5, 0.5     # the benchmark's LARS coefficients (poly rate early in a run)


def _conv(name, dtype, n, hw, c, k, r, stride=1, groups=1):
    return {"name": name, "kind": "conv", "dtype": dtype, "n": n, "hw": hw, "c": c, "k": k, "r": r, "stride": stride, "groups": groups}


def listed():
    return [
        # ResNet-50's 3x3 layer of the 28x28 stage in fp32 at the benchmark's batch: the shape most of the fp32 step's time has
        _conv("conv_f32_3x3_28", "f32", 256, 28, 128, 128, 3),
        # the 56x56 expansion in fp32: few reduction steps per output tile, large tensors
        _conv("conv_f32_1x1_56", "f32", 256, 56, 64, 256, 1),
        # the strided projection into the 14x14 stage in fp32
        _conv("conv_f32_proj_s2", "f32", 256, 28, 512, 1024, 1, stride=2),
        # the smallest calls: a worker with two images (fine-tuning, a strongly scaled run), latency and launches
        _conv("conv_f32_small", "f32", 2, 14, 256, 256, 3),
        # mixed precision at the benchmark's batch: the 3x3 layer of the 14x14 stage
        _conv("conv_bf16_3x3_14", "bf16", 512, 14, 256, 256, 3),
        # mixed precision: a reducing 1x1 layer of the 28x28 stage
        _conv("conv_bf16_1x1_28", "bf16", 512, 28, 512, 128, 1),
        # a ragged batch (the last, incomplete one of an epoch) on the 7x7 stage
        _conv("conv_bf16_ragged", "bf16", 37, 7, 512, 512, 3),
        # a whole layer as a mixed-precision step runs it: convolution with statistics, batch norm + ReLU, both backward
        {"name": "layer_bf16_3x3_56", "kind": "layer", "dtype": "bf16", "n": 512, "hw": 56, "c": 64, "k": 64, "r": 3},
        # batch norm with the residual added, forward and backward, fp32
        {"name": "bn_f32_28", "kind": "bn", "dtype": "f32", "n": 256, "hw": 28, "c": 512, "residual": True},
        # the optimizer over ResNet-50's 161 parameter tensors
        {"name": "lars_resnet50", "kind": "lars", "tensors": 0, "most": 0},
        # a whole training step at an ordinary batch in fp32, and at the benchmark's batch in mixed precision
        {"name": "step_f32_b32", "kind": "step", "dtype": "f32", "n": 32},
        {"name": "step_bf16_b512", "kind": "step", "dtype": "bf16", "n": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo=16, hi=2048):
    c = _log_int(rng, lo, hi)
    unit = rng.choice([32, 32, 32, 8, 8, 1])          # networks take multiples of 32 mostly, odd counts now and then
    return max(unit, c // unit * unit)


def draw(rng):
    kind = rng.choice(["conv"] * 12 + ["layer"] * 3 + ["bn"] * 2 + ["lars"] * 2 + ["step"])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "step":
        return {"kind": "step", "dtype": dtype, "n": _log_int(rng, 2, 64)}
    if kind == "lars":
        return {"kind": "lars", "tensors": _log_int(rng, 1, 200), "most": _log_int(rng, 1000, 300000)}
    n, hw = _log_int(rng, 1, 512), _log_int(rng, 7, 112)
    c, k, r = _channels(rng), _channels(rng), rng.choice([1, 1, 3, 3, 3, 5])
    stride = 2 if r < 5 and rng.random() < 0.2 else 1
    groups = 2 if kind == "conv" and rng.random() < 0.1 else 1
    if kind != "conv":
        stride, c, k, r = 1, (c + 7) // 8 * 8, (k + 7) // 8 * 8, min(r, 3)
    if kind == "conv" and rng.random() < 0.1:
        hw, r, stride, groups = 1, 1, 1, 1             # a fully connected layer
    if groups == 2:
        c, k = 2 * ((c + 1) // 2), 2 * ((k + 1) // 2)
    # no dearer than the whole steps: at most 2^27 elements per tensor and 1.5e12 operations in the three passes
    while n > 1 and (n * hw * hw * max(c, k) > 1 << 27 or 6 * n * hw * hw // stride ** 2 * c * k * r * r // groups > 1.5e12):
        n = n * 3 // 4
    while 6 * n * hw * hw // stride ** 2 * c * k * r * r // groups > 1.5e12:
        c, k = max(8, c // 16 * 8), max(8, k // 16 * 8)
    if kind == "bn":
        return {"kind": "bn", "dtype": dtype, "n": n, "hw": hw, "c": k, "residual": rng.random() < 0.5}
    if kind == "layer":
        return {"kind": "layer", "dtype": dtype, "n": n, "hw": hw, "c": c, "k": k, "r": r}
    return {"kind": "conv", "dtype": dtype, "n": n, "hw": hw, "c": c, "k": k, "r": r, "stride": stride, "groups": groups}


# ---------------------------------------------------------------------------------------------- inputs

def _type(case):
    return (lc.LC_BF16, torch.bfloat16) if case.get("dtype") == "bf16" else (lc.LC_F32, torch.float32)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device=DEV).mul_(std)


def _workspace(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _desc(case):
    return lc.ConvDesc(case["n"], case["c"], case["hw"], case["hw"], case["k"], case["r"], case["r"], case.get("stride", 1),
                       case.get("stride", 1), case["r"] // 2, case["r"] // 2, _type(case)[0], NHWC, case.get("groups", 1))


def _conv_inputs(case, g):
    """x as it leaves a ReLU, He-normal filters, a gradient of the size a mean loss gives."""
    d, t = _desc(case), _type(case)[1]
    p, q = lc.conv2d_out_shape(d)
    x = _normal(g, (d.n, d.h, d.w, d.c)).clamp_(min=0).to(t)
    cg = d.c // d.groups
    w = _normal(g, (d.k, d.r, d.s, cg), math.sqrt(2.0 / (cg * d.r * d.s))).to(t)
    dy = _normal(g, (d.n, p, q, d.k), 1e-3).to(t)
    return d, t, x, w, dy


def _lars_sizes(case):
    if not case["tensors"]:
        return synth.resnet50_param_numels()
    sizes, m = [], case["most"]
    for i in range(case["tensors"]):                   # filters of many sizes with the vectors of their batch norms between them
        sizes.append(max(1, m >> (i % 7)) if i % 3 == 0 else 64 + (37 * i) % 449)
    return sizes


def _flat(g, sizes, std):
    """One buffer for a list of tensors, as data-parallel programs keep them; each starts on a 256-byte boundary."""
    flat = torch.zeros(sum((m + 63) // 64 * 64 for m in sizes), device=DEV)
    for t in _views(flat, sizes):
        t.copy_(_normal(g, t.shape, std))
    return flat


def _views(flat, sizes):
    views, at = [], 0
    for m in sizes:
        views.append(flat[at:at + m])
        at += (m + 63) // 64 * 64
    return views


def prepare(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind == "lars":
        sizes = _lars_sizes(case)
        w, gr, v = (_flat(g, sizes, std) for std in (0.05, 1e-4, 1e-6))
        return {"kind": kind, "args": lc.LarsArgs(*(_views(t, sizes) for t in (w, gr, v))), "w": w, "g": gr, "v": v, "sizes": sizes,
                "trust": torch.empty(len(sizes), device=DEV), "ws": _workspace(lc.lars_workspace_bytes(sizes))}
    if kind == "step":
        net, x, labels = _step_state(case, g)
        return {"kind": kind, "net": net, "x": x, "labels": labels}
    if kind == "bn":
        t = _type(case)[1]
        shape, c = (case["n"], case["hw"], case["hw"], case["c"]), case["c"]
        s = {"kind": kind, "case": dict(case), "dtype": _type(case)[0], "x": _normal(g, shape).to(t), "dy": _normal(g, shape, 1e-3).to(t),
             "res": _normal(g, shape).clamp_(min=0).to(t) if case["residual"] else None,
             "gamma": 1.0 + _normal(g, (c,), 0.1), "beta": _normal(g, (c,), 0.1)}
        s["y"], s["dx"] = torch.empty(shape, dtype=t, device=DEV), torch.empty(shape, dtype=t, device=DEV)
        s["mean"], s["inv"], s["dgamma"], s["dbeta"] = (torch.empty(c, device=DEV) for _ in range(4))
        s["ws"] = _workspace(lc.batchnorm_workspace_bytes(case["n"], c, case["hw"], case["hw"], NHWC))
        return s
    d, t, x, w, dy = _conv_inputs(case, g)
    s = {"kind": kind, "desc": d, "dtype": _type(case)[0], "x": x, "w": w, "dy": dy, "y": torch.empty_like(dy), "dx": torch.empty_like(x),
         "dw": torch.empty(w.shape, device=DEV)}
    need = max(lc.conv2d_workspace_bytes(d, p) for p in (lc.LC_PASS_FWD, lc.LC_PASS_BWD_DATA, lc.LC_PASS_BWD_WEIGHT))
    if kind == "layer":
        k, (p, q) = d.k, dy.shape[1:3]
        s["gamma"], s["beta"] = 1.0 + _normal(g, (k,), 0.1), _normal(g, (k,), 0.1)
        s["a"], s["dz"] = torch.empty_like(dy), torch.empty_like(dy)
        s["mean"], s["inv"], s["dgamma"], s["dbeta"] = (torch.empty(k, device=DEV) for _ in range(4))
        s["tiles"] = lc.conv2d_fwd_stats_count(d)
        s["stats"] = torch.empty(max(1, s["tiles"] * k * 2), device=DEV)
        s["sq"] = torch.empty(lc.conv2d_bwd_weight_sq_count(d), dtype=torch.float64, device=DEV)
        need = max(need, lc.batchnorm_workspace_bytes(d.n, k, p, q, NHWC))
    s["ws"] = _workspace(need)
    return s


def _step_params(net, g):
    """He-normal filters, scales near 1 but small at the end of each residual branch (as large-batch runs start), shifts near 0,
    a small classifier."""
    for name, p in net.params.items():
        if p.dim() == 4:
            p.copy_(_normal(g, p.shape, 0.01 if name == "fc.w" else math.sqrt(2.0 / (p.shape[1] * p.shape[2] * p.shape[3]))))
        elif name.endswith("gamma"):
            p.copy_((1.0 + _normal(g, p.shape, 0.1)) * (0.2 if ".c3." in name else 1.0))
        else:
            p.copy_(_normal(g, p.shape, 0.1))
        if name in net.lowp:
            net.lowp[name].copy_(p.to(torch.bfloat16))


def _step_state(case, g):
    dtype, t = _type(case)
    net = resnet_step.ResNetStep((64, 7, 2, 3), (64, 128, 256, 512), (3, 4, 6, 3), 1000, case["n"], (224, 224), device=DEV, dtype=dtype)
    _step_params(net, g)
    x = _normal(g, (case["n"], 224, 224, 3)).to(t)
    labels = torch.randint(0, 1000, (case["n"],), generator=g, device=DEV, dtype=torch.int32)
    return net, x, labels


# ---------------------------------------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "lars":
        lc.lars_step(s["args"], ETA, MOMENTUM, DECAY, LR, s["trust"], s["ws"])
        return {"trust": s["trust"], "w": s["w"], "v": s["v"]}
    if kind == "step":
        net = s["net"]
        loss = net.step(s["x"], s["labels"], ETA, MOMENTUM, DECAY, LR)
        return {"loss": loss, "logits": net.logits, "filters": {k: v for k, v in net.params.items() if v.dim() == 4}}
    ws = s["ws"]
    if kind == "bn":
        n, hw, c = s["case"]["n"], s["case"]["hw"], s["case"]["c"]
        lc.batchnorm_fwd_t(s["dtype"], s["x"], s["gamma"], s["beta"], s["res"], s["y"], s["mean"], s["inv"], n, c, hw, hw, EPS, True, NHWC, ws)
        # behind a residual the caller has taken dy through the ReLU already
        lc.batchnorm_bwd_t(s["dtype"], s["x"], s["dy"], s["gamma"], s["beta"], s["mean"], s["inv"], s["dx"], s["dgamma"], s["dbeta"], n, c,
                           hw, hw, s["res"] is None, NHWC, ws)
        return {"y": s["y"], "dx": s["dx"], "dgamma": s["dgamma"], "dbeta": s["dbeta"]}
    d = s["desc"]
    if kind == "conv":
        lc.conv2d_fwd(d, s["x"], s["w"], s["y"], ws)
        lc.conv2d_bwd_data(d, s["dy"], s["w"], s["dx"], ws)
        lc.conv2d_bwd_weight(d, s["x"], s["dy"], s["dw"], ws)
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    n, p, q, k = s["dy"].shape
    if s["tiles"]:
        lc.conv2d_fwd_stats(d, s["x"], s["w"], s["y"], s["stats"], ws)
        lc.batchnorm_fwd_pre(s["dtype"], s["y"], s["gamma"], s["beta"], None, s["a"], s["mean"], s["inv"], n, k, p, q, EPS, True, NHWC,
                             s["stats"], s["tiles"], ws)
    else:
        lc.conv2d_fwd(d, s["x"], s["w"], s["y"], ws)
        lc.batchnorm_fwd_t(s["dtype"], s["y"], s["gamma"], s["beta"], None, s["a"], s["mean"], s["inv"], n, k, p, q, EPS, True, NHWC, ws)
    lc.batchnorm_bwd_t(s["dtype"], s["y"], s["dy"], s["gamma"], s["beta"], s["mean"], s["inv"], s["dz"], s["dgamma"], s["dbeta"], n, k, p, q,
                       True, NHWC, ws)
    lc.conv2d_bwd_weight_sq(d, s["x"], s["dz"], s["dw"], s["sq"], ws)
    lc.conv2d_bwd_data(d, s["dz"], s["w"], s["dx"], ws)
    return {"a": s["a"], "dx": s["dx"], "dw": s["dw"], "dgamma": s["dgamma"], "dbeta": s["dbeta"]}


# ---------------------------------------------------------------------------------------------- what a pass cannot do without

def work(case):
    kind, es = case["kind"], 2 if case.get("dtype") == "bf16" else 4
    if kind == "lars":
        return {"bytes": 20.0 * sum(_lars_sizes(case)), "flops": 12.0 * sum(_lars_sizes(case))}
    if kind == "step":
        # three passes over every filter (two for the first layer), every convolution output written and read once each way
        convs = synth.resnet50_convs(case["n"]) + [synth.resnet50_fc(case["n"])]
        flops = sum(c.flops * (2 if c.name == "conv1" else 3) for c in convs)
        return {"bytes": 4.0 * es * sum(c.n * c.p * c.q * c.k for c in convs) + 20.0 * sum(synth.resnet50_param_numels()), "flops": float(flops)}
    if kind == "bn":
        m = case["n"] * case["hw"] ** 2 * case["c"]
        return {"bytes": float(es * m * (6 if case["residual"] else 5)), "flops": 20.0 * m}   # x, (residual), y; x, dy, dx
    c, k, r, g = case["c"], case["k"], case["r"], case.get("groups", 1)
    p = (case["hw"] + 2 * (r // 2) - r) // case.get("stride", 1) + 1
    nx, ny, nw = case["n"] * case["hw"] ** 2 * c, case["n"] * p * p * k, k * r * r * c // g
    flops = 6.0 * ny * (c // g) * r * r
    if kind == "conv":
        return {"bytes": float(es * (3 * nx + 3 * ny + 2 * nw) + 4 * nw), "flops": flops}
    return {"bytes": float(es * (3 * nx + 8 * ny + 2 * nw) + 4 * nw), "flops": flops + 20.0 * ny}


def tolerance(case):
    """About four times what other summation orders gave (the library's own comparison switches: no stream-K, no slab kernels, generic
    addressing) over the listed cases and 30 drawn ones."""
    kind, bf16 = case["kind"], case.get("dtype") == "bf16"
    if kind == "lars":
        return {"rel": 1e-6}
    if kind == "step":
        # measured 0.0043 (the bf16 logits; filters 1.6e-4) and 5.7e-6 (a filter behind a flipped ReLU)
        return {"rel": 0.017, "max": 0.08} if bf16 else {"rel": 2.5e-5, "max": 3e-3}
    if bf16:
        return {"rel": 3e-4, "max": 0.06}              # measured 5.2e-5; a value that rounds to its neighbour is 0.008 off, 0.015 at a ReLU
    return {"rel": 2e-6} if kind == "bn" else {"rel": 1.5e-5}   # convolutions: measured 3.8e-6 (43,600 terms)


# ---------------------------------------------------------------------------------------------- the same in 64 bits

def _unfold(x, r, stride, pad):
    """x [n, c, h, w] float64 -> [n * p * q, c * r * r]"""
    u = F.unfold(x, r, padding=pad, stride=stride) if r > 1 else x[:, :, ::stride, ::stride].flatten(2)
    return u.transpose(1, 2).reshape(-1, u.shape[1])


def _conv64(x, w, dy, d):
    """The three passes of one layer on float64 copies of the operands, some images at a time; dy may be None (forward only)."""
    G, cg, kg = d.groups, d.c // d.groups, d.k // d.groups
    p, q = lc.conv2d_out_shape(d)
    y = torch.empty((d.n, p, q, d.k), dtype=torch.float64, device=DEV)
    dx = torch.zeros((d.n, d.h, d.w, d.c), dtype=torch.float64, device=DEV) if dy is not None else None
    dw = torch.zeros((d.k, d.r, d.s, cg), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // max(1, p * q * cg * d.r * d.s))
    for g in range(G):
        wm = w[g * kg:(g + 1) * kg].double().permute(0, 3, 1, 2).reshape(kg, -1).contiguous()
        for i in range(0, d.n, step):
            xi = x[i:i + step, :, :, g * cg:(g + 1) * cg].double().permute(0, 3, 1, 2).contiguous()
            u, m = _unfold(xi, d.r, d.stride_h, d.pad_h), xi.shape[0]
            y[i:i + step, :, :, g * kg:(g + 1) * kg] = (u @ wm.t()).view(m, p, q, kg)
            if dy is None:
                continue
            dyi = dy[i:i + step, :, :, g * kg:(g + 1) * kg].double().reshape(-1, kg).contiguous()
            dw[g * kg:(g + 1) * kg] += (dyi.t() @ u).view(kg, cg, d.r, d.s).permute(0, 2, 3, 1)
            du = (dyi @ wm).view(m, p * q, -1).transpose(1, 2).contiguous()
            dx[i:i + step, :, :, g * cg:(g + 1) * cg] = F.fold(du, (d.h, d.w), d.r, padding=d.pad_h, stride=d.stride_h).permute(0, 2, 3, 1)
    return y, dx, dw


def _bn64(x, gamma, beta, dy, residual, relu_bwd):
    """Batch norm + ReLU forward, and its backward; x, dy [rows, c] float64."""
    m = x.shape[0]
    mean = x.mean(0)
    inv = 1.0 / torch.sqrt((x - mean).square().mean(0) + EPS)
    xh = (x - mean) * inv
    pre = xh * gamma + beta
    out = (pre if residual is None else pre + residual).clamp(min=0)
    if relu_bwd:
        dy = torch.where(pre > 0, dy, torch.zeros_like(dy))
    dbeta, dgamma = dy.sum(0), (dy * xh).sum(0)
    return out, gamma * inv * (dy - dbeta / m - xh * dgamma / m), dgamma, dbeta


def _lars64(w, g, v):
    nw, ng = w.norm(), g.norm()
    den = ng + DECAY * nw
    trust = ETA * nw / den if nw > 0 and den > 0 else torch.ones((), dtype=torch.float64, device=DEV)
    v = MOMENTUM * v + LR * trust * (g + DECAY * w)
    return w - v, v, trust


def _step64(case, seed):
    """ResNet-50 in float64: forward, autograd, and the update of the filters."""
    net, x, labels = _step_state(case, _gen(seed))
    par = {k: (net.lowp[k] if k in net.lowp else v).double().requires_grad_() for k, v in net.params.items()}

    def conv_bn(name, a, residual=None, relu=True):
        d, w = net.layers[name].desc, par[name + ".w"]
        u = _unfold(a, d.r, d.stride_h, d.pad_h)
        p, q = net.layers[name].out_hw
        z = u @ w.permute(0, 3, 1, 2).reshape(d.k, -1).t()
        mean = z.mean(0)
        out = (z - mean) / torch.sqrt((z - mean).square().mean(0) + EPS) * par[name + ".gamma"] + par[name + ".beta"]
        out = out.view(case["n"], p, q, d.k).permute(0, 3, 1, 2)
        if residual is not None:
            out = out + residual
        return out.clamp(min=0) if relu else out

    a = F.max_pool2d(conv_bn("stem", x.double().permute(0, 3, 1, 2)), 3, 2, 1)
    for name, proj in net.blocks:
        sc = conv_bn(name + ".proj", a, relu=False) if proj else a
        a = conv_bn(name + ".c3", conv_bn(name + ".c2", conv_bn(name + ".c1", a)), residual=sc)
    logits = a.mean((2, 3)) @ par["fc.w"].view(1000, -1).t() + par["fc.b"]
    loss = F.cross_entropy(logits, labels.long())
    loss.backward()
    names = [k for k, v in net.params.items() if v.dim() == 4]
    filters = {k: _lars64(net.params[k].double(), par[k].grad, torch.zeros_like(par[k]))[0].detach() for k in names}
    return {"loss": loss.detach().reshape(1), "logits": logits.detach(), "filters": filters}


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _step64(case, seed) if case["n"] <= 32 else None
    if kind == "lars":
        s = prepare(case, seed)
        w, gr, v = (s[k].double() for k in "wgv")
        trust = []
        for wi, gi, vi in zip(*(_views(t, s["sizes"]) for t in (w, gr, v))):
            wn, vn, t = _lars64(wi, gi, vi)
            wi.copy_(wn)
            vi.copy_(vn)
            trust.append(t)
        return {"trust": torch.stack(trust), "w": w, "v": v}
    if kind == "bn":
        s, c = prepare(case, seed), case["c"]
        res = s["res"].double().view(-1, c) if case["residual"] else None
        out, dx, dgamma, dbeta = _bn64(s["x"].double().view(-1, c), s["gamma"].double(), s["beta"].double(), s["dy"].double().view(-1, c), res,
                                       res is None)
        return {"y": out.view(s["x"].shape), "dx": dx.view(s["x"].shape), "dgamma": dgamma, "dbeta": dbeta}
    s = prepare(case, seed)
    d = s["desc"]
    if kind == "conv":
        y, dx, dw = _conv64(s["x"], s["w"], s["dy"], d)
        return {"y": y, "dx": dx, "dw": dw}
    y = _conv64(s["x"], s["w"], None, d)[0].to(s["y"].dtype).double()    # the convolution's output is stored in the layer's type
    out, dz, dgamma, dbeta = _bn64(y.view(-1, d.k), s["gamma"].double(), s["beta"].double(), s["dy"].double().view(-1, d.k), None, True)
    _, dx, dw = _conv64(s["x"], s["w"], dz.view(y.shape).to(s["y"].dtype), d)
    return {"a": out.view(y.shape), "dx": dx, "dw": dw, "dgamma": dgamma, "dbeta": dbeta}

"""What this library is timed on: the calls that training a network in fixed point consists of, at the sizes of the
benchmark's configurations and around them.

Kinds of cases:

  quantize  one tensor (activations, weights, gradients) to <wl,fl> with stochastic rounding; n elements
  gemm      quantize two matrices in one call, then their exact integer product (the benchmark's first configuration)
  search    the KL-divergence precision search over one weight tensor
  conv_fwd  the forward contraction of one layer on codes, requantized with ReLU
  conv_bwd  both gradient contractions of one layer, requantized
  switch    a precision switch of a whole network: gradient diversity of every layer's lookback window, then one batched
            KL search over all weight tensors
  alexnet   one training step (forward, backward, update) of the AlexNet-CIFAR chain
  resnet18  one training step of the ResNet-18-CIFAR graph with batch normalisation

Inputs are drawn on the GPU from the seed; distributions are those of the benchmark: activations max(N(0,1), 0), weights
N(0, 2/fan_in), gradients N(0, 0.25^2).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2107_13490_amd as pkg
from paper_2107_13490_amd import ConvDesc, Epilogue, LayerDesc, NodeDesc


# ---- the networks ---------------------------------------------------------------------------------------------------

def _alexnet(batch):
    """(name, conv geometry, relu, pool) of the five convolutions and three fully connected layers."""
    return [
        ("conv1", (batch, 32, 32, 3, 64, 3, 3, 1, 1), 1, 1),
        ("conv2", (batch, 16, 16, 64, 192, 3, 3, 1, 1), 1, 1),
        ("conv3", (batch, 8, 8, 192, 384, 3, 3, 1, 1), 1, 0),
        ("conv4", (batch, 8, 8, 384, 256, 3, 3, 1, 1), 1, 0),
        ("conv5", (batch, 8, 8, 256, 256, 3, 3, 1, 1), 1, 1),
        ("fc6", (batch, 1, 1, 4096, 4096, 1, 1, 1, 0), 1, 0),
        ("fc7", (batch, 1, 1, 4096, 4096, 1, 1, 1, 0), 1, 0),
        ("fc8", (batch, 1, 1, 4096, 10, 1, 1, 1, 0), 0, 0),
    ]


def _alexnet_word_lengths(seed):
    g = np.random.Generator(np.random.PCG64([seed, 0]))
    return [int(g.choice([4, 6, 8, 12, 16])) for _ in range(8)]


def _resnet18(batch):
    """(conv geometry, relu, bn, src, res, gap) of the 21 layers, in the order in which they run."""
    rows = [((batch, 32, 32, 3, 64, 3, 3, 1, 1), 1, 1, -1, -1, 0)]
    cin, size, last = 64, 32, 0
    for stage, cout in enumerate((64, 128, 256, 512)):
        for block in range(2):
            stride = 2 if stage > 0 and block == 0 else 1
            first = len(rows)
            rows.append(((batch, size, size, cin, cout, 3, 3, stride, 1), 1, 1, last, -1, 0))
            short = last
            if stride == 2:
                short = len(rows)
                rows.append(((batch, size, size, cin, cout, 1, 1, 2, 0), 0, 1, last, -1, 0))
                size //= 2
            rows.append(((batch, size, size, cout, cout, 3, 3, 1, 1), 1, 1, first, short, int(stage == 3 and block == 1)))
            last = len(rows) - 1
            cin = cout
    rows.append(((batch, 1, 1, 512, 100, 1, 1, 1, 0), 0, 0, last, -1, 0))
    return rows


def _resnet18_word_lengths(seed):
    g = np.random.Generator(np.random.PCG64([seed, 0]))
    return [int(g.integers(4, 17)) for _ in range(21)]


# ---- the cases ------------------------------------------------------------------------------------------------------

def _conv(kind, shape, fx, fw, fdy, zeros=0.0):
    n, h, w, c, k, r, s, stride, pad = shape
    return {"kind": kind, "n": n, "h": h, "w": w, "c": c, "k": k, "r": r, "s": s, "stride": stride, "pad": pad,
            "wl_x": fx, "wl_w": fw, "wl_dy": fdy, "zeros": zeros}


def listed():
    return [
        # the activations of a large batch (1024 x 32 x 32 x 64), two bytes per code
        {"name": "quantize_64M_12bit", "kind": "quantize", "n": 1 << 26, "wl": 12},
        # the benchmark's first configuration: a layer so small that launches and host work count
        {"name": "gemm_256_8bit", "kind": "gemm", "m": 256, "n": 256, "k": 256, "wl_a": 8, "wl_b": 8, "ta": False, "tb": False},
        # and its precision search, on a thin layer's weights, with the benchmark's fine bins
        {"name": "search_65536", "kind": "search", "n": 65536, "wl_lo": 2, "wl_hi": 16, "il": 2, "bins": 2048},
        # AlexNet's second convolution at batch 128: one int8 limb, both directions
        dict(_conv("conv_fwd", (128, 16, 16, 64, 192, 3, 3, 1, 1), 8, 8, 8), name="conv_fwd_8bit"),
        dict(_conv("conv_bwd", (128, 16, 16, 64, 192, 3, 3, 1, 1), 8, 8, 8), name="conv_bwd_8bit"),
        # a ResNet-18 block's convolution at batch 256: two limbs, pruned weights, both directions
        dict(_conv("conv_fwd", (256, 16, 16, 128, 128, 3, 3, 1, 1), 12, 12, 12, 0.5), name="conv_fwd_12bit"),
        dict(_conv("conv_bwd", (256, 16, 16, 128, 128, 3, 3, 1, 1), 12, 12, 12, 0.5), name="conv_bwd_12bit"),
        # sizes that fit no tile, a last partial batch, neighbouring layers of different word lengths
        dict(_conv("conv_fwd", (37, 15, 11, 48, 100, 3, 3, 2, 1), 8, 12, 12), name="conv_fwd_ragged_mixed"),
        # a layer that the controller has pushed above 16 bits: int32 codes
        dict(_conv("conv_fwd", (128, 16, 16, 64, 192, 3, 3, 1, 1), 24, 24, 24), name="conv_fwd_24bit"),
        # the precision switch of ResNet-18: lookback windows of 25 gradients, resolution as the paper has it
        {"name": "switch_resnet18", "kind": "switch", "net": "resnet18", "window": 25, "bins": 128, "wl_seed": 5},
        # whole training steps at the benchmark's batch sizes and word lengths
        {"name": "alexnet_step", "kind": "alexnet", "batch": 128, "wl_seed": 4},
        {"name": "resnet18_step", "kind": "resnet18", "batch": 256, "wl_seed": 5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_conv(rng, kind):
    while True:
        size = _log_int(rng, 1, 33)
        r = rng.choice((1, 3, 3, 5)) if size > 1 else 1
        stride = rng.choice((1, 1, 2)) if size > 2 else 1
        c = rng.choice((3, 16 * _log_int(rng, 1, 32), 16 * _log_int(rng, 1, 32), _log_int(rng, 8, 512)))
        k = rng.choice((10, 16 * _log_int(rng, 1, 32), 16 * _log_int(rng, 1, 32), _log_int(rng, 8, 512)))
        shape = (_log_int(rng, 8, 256), size, max(1, size - rng.choice((0, 0, 1, 3))), c, k, r, r, stride, r // 2)
        if shape[2] + 2 * shape[8] < r:
            continue
        if 2e7 <= _macs(shape) <= 1e10:
            break
    wide = rng.random() < 0.1 and kind == "conv_fwd" and _macs(shape) < 4e9
    if wide:
        wl = [rng.randint(17, 32)] * 3
    elif rng.random() < 0.5:
        wl = [rng.choice((4, 6, 8, 10, 12, 14, 16))] * 3
    else:
        wl = [rng.randint(4, 16) for _ in range(3)]
    return _conv(kind, shape, *wl, rng.choice((0.0, 0.3, 0.5)))


def draw(rng):
    kind = rng.choice(("quantize", "gemm", "search", "conv_fwd", "conv_fwd", "conv_bwd", "conv_bwd", "switch", "alexnet", "resnet18"))
    if kind == "quantize":
        return {"kind": kind, "n": _log_int(rng, 1000, 1 << 26), "wl": rng.randint(4, 16)}
    if kind == "gemm":
        dims = [_log_int(rng, 64, 2048) for _ in range(3)]
        if rng.random() < 0.5:
            dims = [max(16, d // 16 * 16) for d in dims]
        return {"kind": kind, "m": dims[0], "n": dims[1], "k": dims[2], "wl_a": rng.choice((4, 8, 12, 16)),
                "wl_b": rng.choice((4, 8, 12, 16)), "ta": rng.random() < 0.5, "tb": rng.random() < 0.5}
    if kind == "search":
        lo = rng.choice((2, 4))
        return {"kind": kind, "n": _log_int(rng, 2000, 1 << 24), "wl_lo": lo, "wl_hi": 16, "il": rng.randint(1, lo),
                "bins": _log_int(rng, 50, 2048)}
    if kind in ("conv_fwd", "conv_bwd"):
        return _draw_conv(rng, kind)
    if kind == "switch":
        return {"kind": kind, "net": rng.choice(("alexnet", "resnet18")), "window": rng.randint(1, 25), "bins": rng.randint(50, 150),
                "wl_seed": rng.randint(0, 99999)}
    top = 128 if kind == "alexnet" else 256
    return {"kind": kind, "batch": _log_int(rng, 8, top), "wl_seed": rng.randint(0, 99999)}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std):
    return torch.randn(shape, device="cuda", generator=g) * std


def _shape(case):
    return tuple(case[f] for f in ("n", "h", "w", "c", "k", "r", "s", "stride", "pad"))


def _macs(shape):
    d = ConvDesc(*shape)
    return float(d.n) * d.p * d.q * d.k * d.r * d.s * d.c


def _weights(g, k, r, s, c, zeros, gain=math.sqrt(2.0)):
    w = _normal(g, (k, r, s, c), gain / math.sqrt(r * s * c))
    if zeros:
        w[torch.rand((k, r, s, c), device="cuda", generator=g) < zeros] = 0.0
    return w


def _fl(wl):
    return wl - 3


def _prepare_conv(case, seed):
    g = _gen(seed)
    shape = _shape(case)
    d = ConvDesc(*shape)
    ctx = pkg.Context()
    fx, fw, fdy = ((case[f], _fl(case[f])) for f in ("wl_x", "wl_w", "wl_dy"))
    x = torch.relu(_normal(g, (d.n, d.h, d.w, d.c), 1.0))
    w = _weights(g, d.k, d.r, d.s, d.c, case["zeros"])
    s = {"kind": case["kind"], "ctx": ctx, "d": d, "fx": fx, "fw": fw, "fdy": fdy}
    s["x"], _ = ctx.quantize(x, *fx, stream=1)
    s["w"], _ = ctx.quantize(w, *fw, stream=2)
    if case["kind"] == "conv_fwd":
        need = ctx.workspace_bytes(pkg.CALL_CONV_FWD, conv=d, fa=fx, fb=fw)
        s["ep"] = Epilogue.requant(*fx, pkg.SR, seed, 10, relu=True)
        s["y"] = torch.empty((d.n, d.p, d.q, d.k), dtype=ctx.storage_dtype(fx[0]), device="cuda")
    else:
        s["dy"], _ = ctx.quantize(_normal(g, (d.n, d.p, d.q, d.k), 0.25), *fdy, stream=3)
        need = ctx.workspace_bytes(pkg.CALL_CONV_BACKWARD, conv=d, fa=fdy, fb=fw, fc=fx)
        s["ep_dx"] = Epilogue.requant(*fdy, pkg.SR, seed, 11)
        s["ep_dw"] = Epilogue.requant(*fw, pkg.SR, seed, 12)
        s["dx"] = torch.empty((d.n, d.h, d.w, d.c), dtype=ctx.storage_dtype(fdy[0]), device="cuda")
        s["dw"] = torch.empty((d.k, d.r, d.s, d.c), dtype=ctx.storage_dtype(fw[0]), device="cuda")
    ctx.reserve_workspace(need)
    return s


def _net_layers(case):
    """(conv geometry, word length) per layer of the case's network."""
    if case.get("net", case["kind"]) == "alexnet":
        return [(shape, wl) for (_, shape, _, _), wl in zip(_alexnet(case.get("batch", 128)), _alexnet_word_lengths(case["wl_seed"]))]
    return [(row[0], wl) for row, wl in zip(_resnet18(case.get("batch", 256)), _resnet18_word_lengths(case["wl_seed"]))]


def _prepare_switch(case, seed):
    g = _gen(seed)
    ctx = pkg.Context()
    masters, windows, outs, sums = [], [], [], []
    layers = _net_layers(case)
    for i, (shape, wl) in enumerate(layers):
        _, _, _, c, k, r, s = shape[:7]
        n = k * r * s * c
        masters.append(_weights(g, k, r, s, c, 0.3).view(-1))
        dt = ctx.storage_dtype(wl)
        lim = 1 << (wl - 1)
        gs, fmts = [], []
        for j in range(case["window"]):
            # codes fitted to the word length; their exponents move by a bit from batch to batch
            gs.append((_normal(g, (n,), 0.25 * lim)).round_().clamp_(-lim, lim - 1).to(dt))
            fmts.append((wl, (7 * i + 3 * j) % 3))
        windows.append((gs, fmts))
        outs.append(torch.empty(2, dtype=torch.float64, device="cuda"))
        sums.append(torch.empty(case["window"] + 2, dtype=torch.int64, device="cuda"))
    # what the last update of the weights left behind: their ranges
    ranges = torch.empty(2 * len(masters), dtype=torch.float32, device="cuda")
    ctx.quantize_batched(masters, [(wl, _fl(wl)) for _, wl in layers], list(range(1, len(masters) + 1)), ranges=ranges)
    ctx.reserve_for_layers([], kld_bins=None)
    ctx.reserve_workspace(ctx.workspace_bytes(pkg.CALL_KLD_SEARCH_BATCHED, kld_items=[(w.numel(), case["bins"]) for w in masters],
                                              wl_lo=4, wl_hi=16))
    return {"kind": "switch", "ctx": ctx, "masters": masters, "windows": windows, "outs": outs, "sums": sums,
            "ranges": [ranges[2 * i:2 * i + 2] for i in range(len(masters))], "bins": case["bins"], "seed": seed,
            "kld": torch.empty((len(masters), 13), dtype=torch.float64, device="cuda"),
            "sel": torch.empty((len(masters), 2), dtype=torch.int32, device="cuda")}


def _flat(sizes):
    """One flat fp32 parameter buffer and the 16-byte aligned views of its tensors."""
    buf = torch.zeros(sum((n + 3) // 4 * 4 for n in sizes), device="cuda")
    views, at = [], 0
    for n in sizes:
        views.append(buf[at:at + n])
        at += (n + 3) // 4 * 4
    return buf, views


def _prepare_net(case, seed):
    g = _gen(seed)
    batch, alex = case["batch"], case["kind"] == "alexnet"
    rows = _alexnet(batch) if alex else _resnet18(batch)
    shapes = [row[1] if alex else row[0] for row in rows]
    if alex:
        fmts = [(wl, wl - 3) for wl in _alexnet_word_lengths(case["wl_seed"])]
        layers = [LayerDesc(ConvDesc(*shape), relu, pool) for _, shape, relu, pool in rows]
    else:
        # a chain feeds each layer's codes to the next: fewer than 6 bits would saturate
        fmts = [(max(wl, 6), max(wl, 6) - 4) for wl in _resnet18_word_lengths(case["wl_seed"])]
        layers = [NodeDesc(ConvDesc(*shape), relu, 0, bn, src, res, gap) for shape, relu, bn, src, res, gap in rows]
    masters, ws = _flat([s[4] * s[5] * s[6] * s[3] for s in shapes])
    for w, s in zip(ws, shapes):
        w.copy_(_weights(g, s[4], s[5], s[6], s[3], 0.0, 1.5 if alex else 1.4).view(-1))
    state = {"kind": case["kind"], "masters": masters, "seed": seed}
    bn = None
    if not alex:
        widths = [s[4] for s, row in zip(shapes, rows) if row[2]]
        state["gammas"], gammas = _flat(widths)
        state["betas"], betas = _flat(widths)
        for t in gammas:
            t.fill_(1.0)
        it = iter(zip(gammas, betas))
        bn = [next(it) if row[2] else None for row in rows]
    ctx = pkg.Context()
    ctx.reserve_for_layers([(ConvDesc(*s), f, f, f) for s in shapes for f in ((8, 4), (16, 12))])
    net = pkg.Net(ctx, layers, ws, bn=bn)
    for l, f in enumerate(fmts):
        net.set_format(l, *f)
    net.quantize_weights(seed=seed)
    state["x"] = _normal(g, (batch, 32, 32, 3), 1.0)
    classes = shapes[-1][4]
    state["dl"] = torch.randint(-4, 4, (batch, classes), device="cuda", dtype=torch.int32, generator=g).to(
        ctx.storage_dtype(fmts[-1][0]))
    state["ctx"], state["net"] = ctx, net
    last = len(layers) - 1
    out = {"masters": masters, "logits": net.tensor(last, pkg.NT_A), "codes": [net.tensor(l, pkg.NT_QW) for l in range(last + 1)]}
    if not alex:
        out["gammas"], out["betas"] = state["gammas"], state["betas"]
    state["out"] = out
    return state


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("conv_fwd", "conv_bwd"):
        return _prepare_conv(case, seed)
    if kind == "switch":
        return _prepare_switch(case, seed)
    if kind in ("alexnet", "resnet18"):
        return _prepare_net(case, seed)
    g = _gen(seed)
    ctx = pkg.Context()
    if kind == "quantize":
        wl = case["wl"]
        return {"kind": kind, "ctx": ctx, "x": torch.relu(_normal(g, (case["n"],), 1.0)), "wl": wl, "fl": _fl(wl), "seed": seed,
                "out": torch.empty(case["n"], dtype=ctx.storage_dtype(wl), device="cuda"),
                "counters": torch.empty(2, dtype=torch.int64, device="cuda")}
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        a = _normal(g, (k, m) if case["ta"] else (m, k), 0.05)
        b = _normal(g, (n, k) if case["tb"] else (k, n), 0.05)
        fa, fb = (case["wl_a"], case["wl_a"] - 2), (case["wl_b"], case["wl_b"] - 2)
        ctx.reserve_workspace(ctx.workspace_bytes(pkg.CALL_GEMM, transA=int(case["ta"]), transB=int(case["tb"]), M=m, N=n, K=k,
                                                  fa=fa, fb=fb, lda=a.shape[1], ldb=b.shape[1]))
        qs = [torch.empty(t.shape, dtype=ctx.storage_dtype(f[0]), device="cuda") for t, f in ((a, fa), (b, fb))]
        bits = pkg.acc_bits(k, pkg.Fmt(*fa), pkg.Fmt(*fb))
        return {"kind": kind, "ctx": ctx, "ab": [a, b], "qs": qs, "fmts": [fa, fb], "ta": case["ta"], "tb": case["tb"], "seed": seed,
                "counters": torch.empty(4, dtype=torch.int64, device="cuda"), "ep": Epilogue.exact(),
                "c": torch.empty((m, n), dtype=torch.int32 if bits == 32 else torch.int64, device="cuda")}
    w = _normal(g, (case["n"],), 0.05)
    ctx.reserve_workspace(ctx.workspace_bytes(pkg.CALL_KLD_SEARCH, n=case["n"], wl_lo=case["wl_lo"], wl_hi=case["wl_hi"], bins=case["bins"]))
    return {"kind": kind, "ctx": ctx, "w": w, "case": dict(case), "seed": seed}


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "quantize":
        return ctx.quantize(s["x"], s["wl"], s["fl"], pkg.SR, s["seed"], 1, out=s["out"], counters=s["counters"])
    if kind == "gemm":
        qs, (fa, fb) = s["qs"], s["fmts"]
        ctx.quantize_batched(s["ab"], s["fmts"], [1, 2], pkg.SR, s["seed"], outs=qs, counters=s["counters"])
        ctx.fxp_gemm(qs[0], fa, qs[1], fb, s["ep"], s["ta"], s["tb"], out=s["c"])
        return {"a": qs[0], "b": qs[1], "counters": s["counters"], "c": s["c"]}
    if kind == "search":
        c = s["case"]
        r = ctx.kld_precision_search(s["w"], c["wl_lo"], c["wl_hi"], c["il"], c["bins"], 1e-2, seed=s["seed"], stream=2)
        return {"kld": r["kld"], "sel": r["sel"], "grid": r["grid"]}
    if kind == "conv_fwd":
        return ctx.conv_fwd(s["d"], s["x"], s["fx"], s["w"], s["fw"], s["ep"], out=s["y"])
    if kind == "conv_bwd":
        return ctx.conv_backward(s["d"], s["dy"], s["fdy"], s["w"], s["fw"], s["x"], s["fx"], s["ep_dx"], s["ep_dw"],
                                 out_dx=s["dx"], out_dw=s["dw"])
    if kind == "switch":
        for (gs, fmts), out, sums in zip(s["windows"], s["outs"], s["sums"]):
            ctx.gradient_diversity(gs, fmts, out=out, sums=sums)
        n = len(s["masters"])
        ctx.kld_precision_search_batched(s["masters"], [3] * n, [s["bins"]] * n, list(range(1, n + 1)), 4, 16, 1e-2, seed=s["seed"],
                                         kld=s["kld"], sel=s["sel"], ranges=s["ranges"])
        return {"diversity": s["outs"], "sums": s["sums"], "kld": s["kld"], "sel": s["sel"]}
    net = s["net"]
    net.forward(s["x"], seed=s["seed"])
    net.backward(s["dl"], 0, seed=s["seed"])
    net.update(0.01, 1e-5, 1e-4, seed=s["seed"])
    return s["out"]


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def _code_bytes(wl):
    return 1 if wl <= 8 else 2 if wl <= 16 else 4


def work(case):
    kind = case["kind"]
    if kind == "quantize":
        return {"bytes": case["n"] * (4 + _code_bytes(case["wl"])), "flops": 0}
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        codes = (_code_bytes(case["wl_a"]), _code_bytes(case["wl_b"]))
        bits = pkg.acc_bits(k, pkg.Fmt(case["wl_a"], 0), pkg.Fmt(case["wl_b"], 0))
        return {"bytes": m * k * (4 + codes[0]) + k * n * (4 + codes[1]) + m * n * bits // 8, "flops": 2.0 * m * n * k}
    if kind == "search":
        return {"bytes": 4 * case["n"] + 8 * (case["wl_hi"] - case["wl_lo"] + 1), "flops": 0}
    if kind in ("conv_fwd", "conv_bwd"):
        d = ConvDesc(*_shape(case))
        x, w, y = d.n * d.h * d.w * d.c, d.k * d.r * d.s * d.c, d.n * d.p * d.q * d.k
        bx, bw, bdy = (_code_bytes(case[f]) for f in ("wl_x", "wl_w", "wl_dy"))
        if kind == "conv_fwd":
            return {"bytes": x * bx + w * bw + y * bx, "flops": 2.0 * _macs(_shape(case))}
        return {"bytes": y * bdy + x * bx + w * bw + x * bdy + w * bw, "flops": 4.0 * _macs(_shape(case))}
    layers = _net_layers(case)
    sizes = [s[4] * s[5] * s[6] * s[3] for s, _ in layers]
    if kind == "switch":
        return {"bytes": sum(n * (4 + case["window"] * _code_bytes(wl)) for n, (_, wl) in zip(sizes, layers)), "flops": 0}
    # a step: every layer's three contractions (no data gradient below the first layer); activations and their gradients
    # written once and read once per use, master weights read and written, weight codes read twice and written
    nbytes, ops = 4.0 * case["batch"] * 32 * 32 * 3, 0.0
    for i, ((s, wl), n) in enumerate(zip(layers, sizes)):
        d, b = ConvDesc(*s), _code_bytes(max(wl, 6) if kind == "resnet18" else wl)
        y = d.n * d.p * d.q * d.k
        nbytes += n * (8 + 4 * b) + 6 * y * b
        ops += 2.0 * _macs(s) * (2 if i == 0 else 3)
    return {"bytes": nbytes, "flops": ops}


def tolerance(case):
    """Codes, sums, counters and updated weights follow exact integer rules and fp32 operations in a stated order: the
    same bits.  KL values and diversities are fp64 sums whose order is free."""
    return {"rel": 1e-9, "max": 1e-6} if case["kind"] in ("search", "switch") else "exact"

"""Timed workloads of the framework: what a training or inference program has it do.

A case is a dict of plain values; ``kind`` names the workload:

  conv      one convolution layer of a training step: forward, data gradient, filter gradient
  block     a residual bottleneck (1x1, 3x3, 1x1 with the fused bias / ReLU / skip tail), forward only, or the
            forward pass of one micro-batch and the whole backward pass of the one before
  aspp      the five parallel / closing convolutions of the atrous pyramid, three passes each
  head      the logits layer and the weighted loss with all their gradients, as four calls or as the fused one
  upsample  a stride-2 transposed convolution, three passes
  update    the layer-wise adaptive weight update of a list of filters

``listed()`` holds the fixed cases, ``draw(rng)`` makes one more of the same ranges.  ``prepare(case, seed)``
builds what a program has in hand before the call (all on the GPU), ``run(state)`` makes one pass through the
public entry points of ``paper_1810_01993_amd.api`` and returns its outputs, ``work(case)`` counts the bytes and
operations such a pass cannot do without, ``tolerance(case)`` says how far a correct result may be off,
``exact(case, seed)`` gives the outputs of a first pass as plain 64-bit torch computes them.
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_1810_01993_amd import api, layers, synth

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
CODES = {"f16": api.DL_F16, "bf16": api.DL_BF16}


# ---- the cases ---------------------------------------------------------------
def _conv(N, H, W, C, K, R, stride=1, pad=None, dil=1, dtype="f16", dw_f32=False):
    return {"kind": "conv", "N": N, "H": H, "W": W, "C": C, "K": K, "R": R, "stride": stride,
            "pad": dil * (R // 2) if pad is None else pad, "dil": dil, "dtype": dtype, "dw_f32": dw_f32}


def _block(N, H, W, C, width, dil, dtype, train):
    return {"kind": "block", "N": N, "H": H, "W": W, "C": C, "width": width, "dil": dil, "dtype": dtype, "train": train}


def listed():
    return [
        # the smallest layer anyone trains: one atrous 3x3 on a 96 x 144 map of 16 fields; launches and latency count
        dict(_conv(1, 96, 144, 16, 64, 3, dil=2), name="atrous_small"),
        # inference on one odd-sized tile through a bottleneck at output stride 16: the latency of a forward pass
        dict(_block(1, 45, 67, 1024, 256, 1, "f16", False), name="bottleneck_infer"),
        # training step of a bottleneck at output stride 16 (dilated), the shape most of the encoder's layers have
        dict(_block(2, 48, 72, 1024, 256, 2, "bf16", True), name="bottleneck_os16"),
        # the same at output stride 4: wide maps and few channels, bound by memory
        dict(_block(2, 192, 288, 256, 64, 1, "f16", True), name="bottleneck_os4"),
        # the first layer on all 16 fields at full resolution
        dict(_conv(2, 768, 1152, 16, 64, 7, stride=2, dtype="bf16"), name="stem"),
        # the first layer of a model trained on a few selected fields of an odd-sized region, fp32 filter gradients
        dict(_conv(2, 361, 577, 6, 64, 7, stride=2, dtype="f16", dw_f32=True), name="stem_few_fields"),
        # the atrous pyramid: small maps, very long reductions, dilations up to 18
        {"kind": "aspp", "N": 2, "H": 48, "W": 72, "C": 2048, "K": 256, "dtype": "bf16", "name": "aspp"},
        # a dense-block layer of the second network: 5x5, 32 new channels
        dict(_conv(2, 384, 576, 240, 32, 5, dtype="bf16"), name="dense5x5"),
        # an up-sampling layer of the decoder
        {"kind": "upsample", "N": 2, "H": 384, "W": 576, "C": 256, "K": 256, "dtype": "f16", "name": "upsample"},
        # logits and weighted loss at full resolution with all gradients
        {"kind": "head", "N": 2, "H": 768, "W": 1152, "C": 256, "fused": False, "weight_map": False, "dtype": "f16",
         "name": "logits_loss"},
        # the weight update of all 63 filters (40 M parameters) from fp16 gradients
        {"kind": "update", "count": 63, "width": 1.0, "grads": "f16", "momentum": True, "name": "update"},
        # the largest: a full-resolution decoder layer
        dict(_conv(2, 768, 1152, 304, 256, 3), name="decoder3x3"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _channels(rng, lo, hi):
    return max(8, int(round(_log(rng, lo, hi) / 8)) * 8)


def _map(rng, lo, hi):
    """Image height on a log scale, width about 1.5 times that; odd sizes among them."""
    h = int(_log(rng, lo, hi))
    return h, max(4, int(h * rng.uniform(1.3, 1.7)))


def draw(rng):
    kind = rng.choice(["conv", "conv", "conv", "few_fields", "block", "block", "aspp", "head", "upsample", "update"])
    dtype = rng.choice(["f16", "bf16"])
    if kind == "conv":
        while True:
            R = rng.choice([1, 1, 3, 3, 3, 5, 7])
            stride = rng.choice([1, 1, 1, 2])
            dil = rng.choice([1, 1, 1, 2, 6]) if R == 3 and stride == 1 else 1
            H, W = _map(rng, 24, 768)
            c = _conv(rng.choice([1, 2]), H, W, _channels(rng, 16, 512), _channels(rng, 16, 512), R, stride, None, dil, dtype,
                      rng.random() < 0.25)
            w = work(c)
            if w["flops"] < 9e11 and w["bytes"] < 2.5e9:
                return c
    if kind == "few_fields":
        H, W = _map(rng, 48, 500)
        R = rng.choice([3, 5, 7])
        return _conv(rng.choice([1, 2]), H, W, rng.choice([3, 4, 5, 6, 7, 9, 10, 11, 12, 13]), rng.choice([32, 48, 64]), R,
                     rng.choice([1, 2]) if H < 250 else 2, None, 1, dtype, rng.random() < 0.5)
    if kind == "block":
        width = rng.choice([64, 128, 256, 512])
        H, W = _map(rng, 24, {64: 220, 128: 160, 256: 110, 512: 72}[width])
        return _block(rng.choice([1, 2]), H, W, 4 * width, width, rng.choice([1, 2]), dtype, rng.random() < 0.7)
    if kind == "aspp":
        H, W = _map(rng, 20, 60)
        return {"kind": "aspp", "N": rng.choice([1, 2]), "H": H, "W": W, "C": rng.choice([512, 1024, 2048]), "K": 256,
                "dtype": dtype}
    if kind == "head":
        H, W = _map(rng, 96, 700)
        return {"kind": "head", "N": rng.choice([1, 2]), "H": H, "W": W, "C": rng.choice([64, 128, 240, 256]),
                "fused": rng.random() < 0.5, "weight_map": rng.random() < 0.3, "dtype": dtype}
    if kind == "upsample":
        H, W = _map(rng, 48, 400)
        return {"kind": "upsample", "N": rng.choice([1, 2]), "H": H, "W": W, "C": rng.choice([64, 128, 160, 256]),
                "K": rng.choice([64, 128, 160, 256]), "dtype": dtype}
    return {"kind": "update", "count": rng.randint(5, 63), "width": round(_log(rng, 0.2, 1.0), 3),
            "grads": rng.choice(["f16", "bf16", "f32"]), "momentum": rng.random() < 0.8}


# ---- shapes ------------------------------------------------------------------
def _desc(c, C=None, K=None, R=None, stride=None, pad=None, dil=None):
    """ConvDesc of a layer of case c; what is not given is taken from the case."""
    g = lambda v, name: c[name] if v is None else v                                              # noqa: E731
    R, s, p, d = g(R, "R"), g(stride, "stride"), g(pad, "pad"), g(dil, "dil")
    code = CODES[c["dtype"]]
    return api.ConvDesc(c["N"], c["H"], c["W"], g(C, "C"), g(K, "K"), R, R, s, s, p, p, d, d, code,
                        api.DL_F32 if c.get("dw_f32") else code)


def _aspp_layers(c):
    """(C, K, R, pad, dil) of the pyramid's 1x1, its three dilated 3x3 and the closing 1x1."""
    C, K = c["C"], c["K"]
    return [(C, K, 1, 0, 1), (C, K, 3, 6, 6), (C, K, 3, 12, 12), (C, K, 3, 18, 18), (5 * K, K, 1, 0, 1)]


def _block_descs(c):
    C, w, d = c["C"], c["width"], c["dil"]
    return (_desc(c, C, w, 1, 1, 0, 1), _desc(c, w, w, 3, 1, d, d), _desc(c, w, C, 1, 1, 0, 1))


def _filter_sizes(c):
    """Element counts of the first `count` filters of the segmentation network, channels scaled by `width`."""
    out = []
    for layer in layers.deeplab_layers():
        scale = lambda n: n if n <= 16 else max(8, int(n * c["width"] / 8) * 8)                   # noqa: E731
        out += [scale(layer.K) * layer.R * layer.S * scale(layer.C)] * layer.count
    return out[:c["count"]]


# ---- inputs --------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, shape, dtype, scale=1.0):
    return torch.randn(shape, generator=g, device="cuda").mul_(scale).to(dtype)


def _activations(g, shape, dtype):
    """Behind a ReLU: non-negative."""
    return torch.randn(shape, generator=g, device="cuda").abs_().to(dtype)


def _filter(g, K, R, C, dtype):
    return _randn(g, (K, R, R, C), dtype, math.sqrt(2.0 / (R * R * C)))


def _fields(g, N, H, W, C, dtype):
    """Smooth fields like climate variables on a grid."""
    coarse = torch.randn((N, C, H // 8 + 2, W // 8 + 2), generator=g, device="cuda")
    fine = F.interpolate(coarse, size=(H, W), mode="bilinear", align_corners=True)
    return fine.permute(0, 2, 3, 1).contiguous().mul_(1.5).to(dtype)


def _labels(g, N, H, W):
    """Connected patches: about 1.7 % of class 1 and 0.1 % of class 2, the rest background."""
    def top(share, cell):
        f = F.interpolate(torch.randn((N, 1, H // cell + 2, W // cell + 2), generator=g, device="cuda"), size=(H, W),
                          mode="bilinear", align_corners=True).reshape(-1)
        keep = max(1, int(share * f.numel()))
        return f >= f.kthvalue(f.numel() - keep + 1).values
    out = top(0.017, 24).to(torch.uint8)
    out[top(0.001, 10)] = 2
    return out.reshape(N, H, W)


def prepare(case, seed):
    c, g = case, _generator(seed)
    dt = DTYPES.get(case.get("dtype"))
    s = {"case": c}
    if c["kind"] == "conv":
        d = s["desc"] = _desc(c)
        P, Q = api.dl_conv_out_shape(d)
        first = c["R"] == 7 or c["C"] < 16
        s["x"] = (_fields if first else lambda g, N, H, W, C, dt: _activations(g, (N, H, W, C), dt))(g, c["N"], c["H"], c["W"], c["C"], dt)
        s["w"] = _filter(g, c["K"], c["R"], c["C"], dt)
        s["dy"] = _randn(g, (c["N"], P, Q, c["K"]), dt)
    elif c["kind"] == "block":
        C, w = c["C"], c["width"]
        s["descs"] = _block_descs(c)
        s["x"] = _activations(g, (c["N"], c["H"], c["W"], C), dt)
        s["w"] = (_filter(g, w, 1, C, dt), _filter(g, w, 3, w, dt), _filter(g, C, 1, w, dt))
        s["b"] = tuple(torch.randn(k, generator=g, device="cuda").mul_(0.2) for k in (w, w, C))
        if c["train"]:
            # the backward pass of the micro-batch before: its activations as its forward pass left them
            kept = lambda k: torch.randn((c["N"], c["H"], c["W"], k), generator=g, device="cuda").clamp_(min=0).to(dt)   # noqa: E731
            s["kept"] = (kept(C), kept(w), kept(w), kept(C))
            s["dy"] = _randn(g, (c["N"], c["H"], c["W"], C), dt)
    elif c["kind"] == "aspp":
        s["layers"] = []
        x = _activations(g, (c["N"], c["H"], c["W"], c["C"]), dt)
        for C, K, R, pad, dil in _aspp_layers(c):
            xi = x if C == c["C"] and len(s["layers"]) < 4 else _activations(g, (c["N"], c["H"], c["W"], C), dt)
            s["layers"].append((_desc(c, C, K, R, 1, pad, dil), xi, _filter(g, K, R, C, dt),
                                _randn(g, (c["N"], c["H"], c["W"], K), dt)))
    elif c["kind"] == "head":
        n = c["N"] * c["H"] * c["W"]
        s["desc"] = _desc(c, c["C"], 3, 1, 1, 0, 1)
        s["x"] = _activations(g, (c["N"], c["H"], c["W"], c["C"]), dt)
        s["w"] = _filter(g, 3, 1, c["C"], dt)
        s["labels"] = _labels(g, c["N"], c["H"], c["W"])
        s["cw"] = torch.tensor(synth.CLASS_WEIGHTS, dtype=torch.float32, device="cuda")
        # a loss scale, as in half-precision training: gradients of 1 / n would fall below fp16's range
        s["scale"] = 1024.0 / n
        s["map"] = s["cw"][s["labels"].long()].contiguous() if c["weight_map"] and not c["fused"] else None
    elif c["kind"] == "upsample":
        d = s["desc"] = _desc(c, c["C"], c["K"], 3, 2, 1, 1)
        P, Q = api.dl_conv_out_shape(d)
        s["x"] = _activations(g, (c["N"], P, Q, c["K"]), dt)
        s["w"] = _randn(g, (c["K"], 3, 3, c["C"]), dt, math.sqrt(2.0 / (9 * c["K"])))
        s["dy"] = _randn(g, (c["N"], c["H"], c["W"], c["C"]), dt)
    else:
        sizes = _filter_sizes(c)
        total = sum(sizes)
        gd = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[c["grads"]]
        s["flat_w"] = torch.randn(total, generator=g, device="cuda").mul_(0.05)
        s["flat_g"] = torch.randn(total, generator=g, device="cuda").mul_(0.5).to(gd)
        s["flat_v"] = torch.randn(total, generator=g, device="cuda").mul_(1e-4) if c["momentum"] else None
        split = lambda t: list(torch.split(t, sizes))                                            # noqa: E731
        s["w"], s["g"] = split(s["flat_w"]), split(s["flat_g"])
        s["v"] = split(s["flat_v"]) if c["momentum"] else None
    return s


# ---- one pass ------------------------------------------------------------------
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "conv":
        d = s["desc"]
        y = api.conv2d_fwd(d, s["x"], s["w"])
        dx = api.conv2d_bwd_data(d, s["dy"], s["w"])
        dw = api.conv2d_bwd_filter(d, s["x"], s["dy"])
        return y, dx, dw
    if kind == "block":
        (d1, d2, d3), (w1, w2, w3), (b1, b2, b3), x = s["descs"], s["w"], s["b"], s["x"]
        a1 = api.conv2d_fwd_bias_relu(d1, x, w1, b1, True)
        a2 = api.conv2d_fwd_bias_relu(d2, a1, w2, b2, True)
        y = api.conv2d_fwd_bias_add_relu(d3, a2, w3, b3, x, True)
        if not c["train"]:
            return y
        px, p1, p2, py = s["kept"]
        dz3, db3 = api.bias_relu_bwd(s["dy"], py, True)                  # also the skip connection's gradient
        da2 = api.conv2d_bwd_data(d3, dz3, w3)
        dw3 = api.conv2d_bwd_filter(d3, p2, dz3)
        dz2, db2 = api.bias_relu_bwd(da2, p2, True)
        da1 = api.conv2d_bwd_data(d2, dz2, w2)
        dw2 = api.conv2d_bwd_filter(d2, p1, dz2)
        dz1, db1 = api.bias_relu_bwd(da1, p1, True)
        dx = api.conv2d_bwd_data(d1, dz1, w1)
        dw1 = api.conv2d_bwd_filter(d1, px, dz1)
        return y, dz3, dx, dw1, dw2, dw3, db1, db2, db3
    if kind == "aspp":
        out = []
        for d, x, w, dy in s["layers"]:
            out += [api.conv2d_fwd(d, x, w), api.conv2d_bwd_data(d, dy, w), api.conv2d_bwd_filter(d, x, dy)]
        return out
    if kind == "head":
        d, x, w = s["desc"], s["x"], s["w"]
        if c["fused"]:
            return api.logits_ce_fused_fwd_bwd(x, w, s["labels"], s["cw"], s["scale"])
        z = api.conv2d_fwd(d, x, w)
        if s["map"] is not None:
            loss, dz = api.weighted_pixel_ce_map_fwd_bwd(z, s["labels"], s["map"], s["scale"])
        else:
            loss, dz = api.weighted_pixel_ce_fwd_bwd(z, s["labels"], s["cw"], s["scale"])
        return z, loss, dz, api.conv2d_bwd_data(d, dz, w), api.conv2d_bwd_filter(d, x, dz)
    if kind == "upsample":
        d = s["desc"]
        return (api.conv2d_transpose_fwd(d, s["x"], s["w"]), api.conv2d_transpose_bwd_data(d, s["dy"], s["w"]),
                api.conv2d_transpose_bwd_filter(d, s["x"], s["dy"]))
    rates = api.larc_sgd_step(s["w"], s["g"], s["v"], lr=0.01, trust=0.001, weight_decay=1e-4,
                              momentum=0.9 if c["momentum"] else 0.0)
    return s["flat_w"], s["flat_v"], rates


# ---- what a pass cannot do without ----------------------------------------------
def _extent(n, R, stride, pad, dil):
    return (n + 2 * pad - dil * (R - 1) - 1) // stride + 1


def work(case):
    c = case
    N = c.get("N", 0)
    if c["kind"] == "conv":
        P, Q = (_extent(c[a], c["R"], c["stride"], c["pad"], c["dil"]) for a in "HW")
        x, y, w = N * c["H"] * c["W"] * c["C"], N * P * Q * c["K"], c["K"] * c["R"] ** 2 * c["C"]
        # read x, dy, w; write y, dx, dw
        return {"bytes": 4 * x + 4 * y + 2 * w + (4 if c["dw_f32"] else 2) * w,
                "flops": 6.0 * N * P * Q * c["K"] * c["C"] * c["R"] ** 2}
    if c["kind"] == "block":
        n, C, w = N * c["H"] * c["W"], c["C"], c["width"]
        filters = 2 * C * w + 9 * w * w
        if not c["train"]:
            return {"bytes": 2 * (2 * n * C + filters), "flops": 2.0 * n * filters}
        # read x, dy, the kept activations and the filters; write y, the skip's gradient, dx and the filter gradients
        return {"bytes": 2 * (n * (7 * C + 2 * w) + 2 * filters), "flops": 6.0 * n * filters}
    if c["kind"] == "aspp":
        n, byts, flops, seen = N * c["H"] * c["W"], 0, 0.0, set()
        for C, K, R, _, _ in _aspp_layers(c):
            x_read = 0 if (C == c["C"] and "x" in seen) else n * C       # the first four layers share their input
            seen.add("x")
            byts += 2 * (x_read + n * C + 2 * n * K + 2 * K * R * R * C)
            flops += 6.0 * n * K * R * R * C
        return {"bytes": byts, "flops": flops}
    if c["kind"] == "head":
        n, C = N * c["H"] * c["W"], c["C"]
        # read x, labels, w (and the weight map); write dx, logits, dlogits, dw
        return {"bytes": n * (4 * C + 13 + (4 if c["weight_map"] and not c["fused"] else 0)) + 4 * 3 * C,
                "flops": 18.0 * n * C + 60.0 * n}
    if c["kind"] == "upsample":
        P, Q = (_extent(c[a], 3, 2, 1, 1) for a in "HW")
        x, y, w = N * P * Q * c["K"], N * c["H"] * c["W"] * c["C"], 9 * c["K"] * c["C"]
        return {"bytes": 2 * (2 * x + 2 * y + 2 * w), "flops": 54.0 * N * P * Q * c["K"] * c["C"]}
    n = sum(_filter_sizes(c))
    return {"bytes": n * (8 + (4 if c["grads"] == "f32" else 2) + (8 if c["momentum"] else 0)), "flops": 12.0 * n}


def tolerance(case):
    """Outputs are rounded once from fp32 sums: against float64 sums of the same inputs that is 2.1e-4 in fp16 and 1.7e-3
    in bf16 (2-norm; 4.9e-4 and 3.9e-3 of a single value).  Where a layer reads what another one has rounded, up to 3.1e-4
    and 2.5e-3, and single values whose terms cancel are off by more (0.017 and 0.16 of the tensor's root mean square)."""
    if case["kind"] == "update":
        return {"rel": 1e-5, "max": 1e-4}                               # fp32 norms summed in another order
    if case["kind"] in ("block", "head"):
        return {"rel": 1e-2, "max": 0.3} if case["dtype"] == "bf16" else {"rel": 1.2e-3, "max": 0.05}
    return {"rel": 7e-3, "max": 0.016} if case["dtype"] == "bf16" else {"rel": 8e-4, "max": 2e-3}


# ---- the same in 64 bits ----------------------------------------------------------
def _taps(H, W, P, Q, R, stride, pad, dil):
    """(r, s, rows, columns): the part of the zero-padded image that filter tap (r, s) meets, as slices."""
    cut = lambda t, n: slice(t * dil, t * dil + (n - 1) * stride + 1, stride)                       # noqa: E731
    return [(r, s, cut(r, P), cut(s, Q)) for r in range(R) for s in range(R)]


def _conv64(d, x, w, dy):
    """float64 (y, dx, dw) of the convolution d, tap by tap; what needs a missing operand is None."""
    P, Q = _extent(d.H, d.R, d.stride_h, d.pad_h, d.dil_h), _extent(d.W, d.S, d.stride_w, d.pad_w, d.dil_w)
    p = d.pad_h
    xp = None if x is None else F.pad(x.double(), (0, 0, p, p, p, p))
    g = None if dy is None else dy.double().reshape(-1, d.K)
    y = torch.zeros((d.N * P * Q, d.K), dtype=torch.float64, device="cuda") if x is not None and w is not None else None
    dxp = torch.zeros((d.N, d.H + 2 * p, d.W + 2 * p, d.C), dtype=torch.float64, device="cuda") if g is not None and w is not None else None
    dw = torch.zeros((d.K, d.R, d.S, d.C), dtype=torch.float64, device="cuda") if g is not None and x is not None else None
    for r, s, rows, cols in _taps(d.H, d.W, P, Q, d.R, d.stride_h, p, d.dil_h):
        xt = None if xp is None else xp[:, rows, cols].reshape(-1, d.C)
        wt = None if w is None else w[:, r, s].double().contiguous()
        if y is not None:
            y += xt @ wt.t()
        if dxp is not None:
            dxp[:, rows, cols] += (g @ wt).view(d.N, P, Q, d.C)
        if dw is not None:
            dw[:, r, s] = g.t() @ xt
    return (None if y is None else y.view(d.N, P, Q, d.K),
            None if dxp is None else dxp[:, p:p + d.H, p:p + d.W].contiguous(), dw)


def _block64(s, c):
    (d1, d2, d3), (w1, w2, w3), b = s["descs"], s["w"], [t.double() for t in s["b"]]
    a = (_conv64(d1, s["x"], w1, None)[0] + b[0]).clamp_(min=0)
    a = (_conv64(d2, a, w2, None)[0] + b[1]).clamp_(min=0)
    y = (_conv64(d3, a, w3, None)[0] + b[2] + s["x"].double()).clamp_(min=0)
    if not c["train"]:
        return y
    px, p1, p2, py = s["kept"]
    total = lambda t: t.reshape(-1, t.shape[-1]).sum(0)                                             # noqa: E731
    dz3 = s["dy"].double() * (py > 0)
    _, da2, dw3 = _conv64(d3, p2, w3, dz3)
    dz2 = da2 * (p2 > 0)
    _, da1, dw2 = _conv64(d2, p1, w2, dz2)
    dz1 = da1 * (p1 > 0)
    _, dx, dw1 = _conv64(d1, px, w1, dz1)
    return y, dz3, dx, dw1, dw2, dw3, total(dz1), total(dz2), total(dz3)


def _head64(s, c):
    n, C = c["N"] * c["H"] * c["W"], c["C"]
    x, w, lab = s["x"].double().view(n, C), s["w"].double().view(3, C), s["labels"].view(n).long()
    z = x @ w.t()
    weight = (s["cw"].double()[lab] if s["map"] is None else s["map"].double().view(n)) * s["scale"]
    lse = torch.logsumexp(z, 1)
    loss = (weight * (lse - z.gather(1, lab[:, None])[:, 0])).sum().view(1)
    dz = ((z - lse[:, None]).exp() - F.one_hot(lab, 3)) * weight[:, None]
    dx, dw = dz @ w, dz.t() @ x
    if c["fused"]:
        return z, loss, dz, dx.view(s["x"].shape), dw.view(s["w"].shape)
    z, dz = (t.view(c["N"], c["H"], c["W"], 3) for t in (z, dz))
    return z, loss, dz, dx.view(s["x"].shape), dw.view(s["w"].shape)


def _update64(s, c):
    lr, trust, decay, momentum = 0.01, 0.001, 1e-4, 0.9 if c["momentum"] else 0.0
    ws, vs, rates = [], [], []
    for i, (w, g) in enumerate(zip(s["w"], s["g"])):
        w, g = w.double(), g.double()
        local = trust * w.norm() / (g.norm() + decay * w.norm())
        rate = torch.clamp(local, max=lr)
        v = rate * (g + decay * w)
        if c["momentum"]:
            v = v + momentum * s["v"][i].double()
        ws.append(w - v)
        vs.append(v)
        rates.append(rate)
    return torch.cat(ws), torch.cat(vs) if c["momentum"] else None, torch.stack(rates)


def exact(case, seed):
    c, s = case, prepare(case, seed)
    kind = c["kind"]
    if kind == "conv":
        return _conv64(s["desc"], s["x"], s["w"], s["dy"])
    if kind == "block":
        return _block64(s, c)
    if kind == "aspp":
        return [t for d, x, w, dy in s["layers"] for t in _conv64(d, x, w, dy)]
    if kind == "head":
        return _head64(s, c)
    if kind == "upsample":
        y, dx, _ = _conv64(s["desc"], s["dy"], s["w"], s["x"])
        return dx, y, _conv64(s["desc"], s["dy"], None, s["x"])[2]
    return _update64(s, c)

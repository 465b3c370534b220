"""The work that users of the protected convolution have it do, as cases to time and to check.

Each case is one pass through the package's public entry points on device tensors: a protected
layer (``Layer.protected``), the same layer with soft errors in its output that the correction
chain repairs (``Layer.protected_fused``), or a whole network of protected layers
(``network.Chain``).  Layer shapes are those of the workloads (AlexNet, VGG-19, ResNet-18,
Darknet-19 and the single tiny layer), and drawn cases spread over the ranges these span: batch,
map size, channels, kernel, stride, grouping, bias and both data types.
"""
from __future__ import annotations

import math

import torch

import paper_2003_12203_amd as ft
import workloads as wl
from paper_2003_12203_amd import network, schemes

# the largest drawn layer: the flops and bytes of the largest listed single layers
MAX_FLOPS = 1.2e11
MAX_BYTES = 2.6e8


def _layer(name, n, ch, hw, m, r, stride=1, pad=0, dtype="f32", groups=1, bias=False, kind="protected", faults=""):
    return {"name": name, "kind": kind, "n": n, "ch": ch, "h": hw, "w": hw, "m": m, "r": r, "s": r,
            "stride": stride, "pad": pad, "dtype": dtype, "groups": groups, "bias": bias, "faults": faults}


def listed():
    return [
        # one small image layer: what a call costs when the arithmetic is nothing (launches, latency)
        _layer("tiny_f32", 4, 3, 32, 16, 3, 1, 1),
        # AlexNet's stem: three channels, an 11x11 kernel at stride 4
        _layer("alexnet_conv1_f32", 64, 3, 227, 96, 11, 4, 0),
        # AlexNet conv2 as published: two groups, a 5x5 kernel, with its bias
        _layer("alexnet_conv2_grouped_bias_f32", 64, 96, 27, 256, 5, 1, 2, groups=2, bias=True),
        # AlexNet conv4: odd 13x13 maps
        _layer("alexnet_conv4_f32", 64, 384, 13, 384, 3, 1, 1),
        # VGG-19's middle layers, the bulk of the headline network
        _layer("vgg19_v6_f32", 32, 256, 56, 256, 3, 1, 1),
        # VGG-19's last stage, with one image's outputs corrupted at one position (a row error,
        # which the correction chain locates and repairs)
        _layer("vgg19_v14_f32_row_error", 32, 512, 14, 512, 3, 1, 1, kind="erroneous", faults="row"),
        # Darknet-19's 1x1 bottlenecks: little arithmetic per byte
        _layer("darknet19_1x1_f32", 16, 512, 26, 256, 1),
        # ResNet-18's stem in bf16: the largest maps of the bf16 workloads
        _layer("resnet18_stem_bf16", 128, 3, 224, 64, 7, 2, 3, dtype="bf16"),
        # ResNet-18's third stage: many images of small maps
        _layer("resnet18_l3_bf16", 128, 256, 14, 256, 3, 1, 1, dtype="bf16"),
        # ResNet-18's projection shortcut: 1x1 at stride 2 onto 7x7 maps
        _layer("resnet18_proj_bf16", 128, 256, 14, 512, 1, 2, 0, dtype="bf16"),
        # VGG-19's 512-channel layers in bf16: the matrix cores' densest work
        _layer("vgg19_v10_bf16", 32, 512, 28, 512, 3, 1, 1, dtype="bf16"),
        # VGG-19 as one network of sixteen protected layers at a serving batch
        {"name": "vgg19_chain_bf16", "kind": "chain", "net": "vgg19", "n": 8, "dtype": "bf16"},
    ]


def _sizes(c):
    e = (c["h"] + 2 * c["pad"] - c["r"]) // c["stride"] + 1
    f = (c["w"] + 2 * c["pad"] - c["s"]) // c["stride"] + 1
    flops = 2.0 * c["n"] * c["m"] * e * f * (c["ch"] // c["groups"]) * c["r"] * c["s"]
    es = 4 if c["dtype"] == "f32" else 2
    kg = (c["ch"] // c["groups"]) * c["r"] * c["s"]
    # D and W read, O written; the encoded Cw1, Cw2 read; Cd1, Cd2 and the seven position arrays written
    b = es * (c["n"] * c["ch"] * c["h"] * c["w"] + c["m"] * kg + c["n"] * c["m"] * e * f)
    b += 8.0 * (2 * c["ch"] * c["r"] * c["s"] + 2 * c["ch"] * c["h"] * c["w"] + 7 * e * f)
    return e, f, flops, b


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_NETS = {"vgg19": 2, "alexnet": 1, "darknet19": 4}


def draw(rng):
    if rng.random() < 0.1:
        net = rng.choice(sorted(_NETS))
        dtype = rng.choice(["f32", "bf16"])
        # no more arithmetic than the listed network
        top = {"vgg19": 8 if dtype == "bf16" else 2, "alexnet": 64, "darknet19": 16 if dtype == "bf16" else 8}[net]
        return {"kind": "chain", "net": net, "n": _log(rng, 1, top), "dtype": dtype}
    while True:
        r = rng.choice([1, 1, 3, 3, 3, 3, 5, 7, 11])
        stride = rng.choice([1, 1, 1, 2, 4 if r > 3 else 1])
        pad = rng.choice([r // 2, r // 2, 0])
        h = _log(rng, 7, 227)
        w = h if rng.random() < 0.8 else _log(rng, 7, 227)
        kind = rng.random()
        if kind < 0.15:
            ch = 3
        elif kind < 0.8:
            ch = 32 * _log(rng, 1, 32)
        else:
            ch = _log(rng, 4, 512)
        m = 16 * _log(rng, 1, 64) if rng.random() < 0.8 else _log(rng, 4, 1024)
        groups = rng.choice([1, 1, 1, 1, 1, 1, 2, 4])
        if ch % groups or m % groups:
            groups = 1
        c = {"kind": "protected", "n": _log(rng, 1, 128), "ch": ch, "h": h, "w": w, "m": m, "r": r, "s": r,
             "stride": stride, "pad": pad, "dtype": rng.choice(["f32", "bf16"]), "groups": groups,
             "bias": rng.random() < 0.3, "faults": ""}
        if h + 2 * pad < r or w + 2 * pad < r:
            continue
        e, f, flops, b = _sizes(c)
        if flops > MAX_FLOPS or b > MAX_BYTES or flops < 1e6:
            continue
        if c["n"] >= 3 and m >= 3 and rng.random() < 0.15:
            c["kind"] = "erroneous"
            c["faults"] = rng.choice(["single", "row"])
        return c


def _specs(c):
    """The network's layers at the case's batch."""
    return [s.with_(n=c["n"], dtype=c["dtype"]) for s in wl.config(_NETS[c["net"]]).layers]


def _tuple(s):
    return (s.n, s.ch, s.h, s.w, s.m, s.r, s.s, s.stride, s.pad)


def _inputs(c, seed):
    """The input map, the filters and the biases, drawn on the device from the seed alone: maps
    from U(0, 1) (post-activation), filters He-normal, biases U(-0.1, 0.1)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    if c["kind"] == "chain":
        sp = _specs(c)
        shapes = [(s.m, s.ch, s.r, s.s) for s in sp]
        d_shape = (sp[0].n, sp[0].ch, sp[0].h, sp[0].w)
    else:
        shapes = [(c["m"], c["ch"] // c["groups"], c["r"], c["s"])]
        d_shape = (c["n"], c["ch"], c["h"], c["w"])
    D = torch.rand(d_shape, generator=g, device="cuda").to(dt)
    Ws = [(torch.randn(sh, generator=g, device="cuda") * math.sqrt(2.0 / (sh[1] * sh[2] * sh[3]))).to(dt)
          for sh in shapes]
    bias = None
    if c.get("bias"):
        bias = (torch.rand(c["m"], generator=g, device="cuda") - 0.5) * 0.2
    return D, Ws, bias


def prepare(case, seed):
    D, Ws, bias = _inputs(case, seed)
    if case["kind"] == "chain":
        net = network.Chain([_tuple(s) for s in _specs(case)], dtype=case["dtype"])
        net.set_weights(Ws)
        return {"case": case, "net": net, "D": D}
    lay = ft.Layer(case["n"], case["ch"], case["h"], case["w"], case["m"], case["r"], case["s"], case["stride"],
                   case["pad"], case["dtype"], groups=case["groups"])
    W = Ws[0]
    lay.encode_weights(W)
    if bias is not None:
        lay.set_bias(bias)
    faults = []
    if case["faults"]:
        faults = schemes.pattern(case["faults"], case["n"], case["m"], lay.E, lay.F)
    return {"case": case, "lay": lay, "D": D, "W": W, "O": lay.empty_output(), "faults": faults}


# the words of a report before the library's own: detected, n_flagged, status, resolved_by[7],
# n_fixes, cap_fixes
_REPORT_WORDS = 12


def run(state):
    if state["case"]["kind"] == "chain":
        net = state["net"]
        net.launch(state["D"])
        return {"output": net.outputs[-1],
                "reports": [lay.report.view(torch.int32)[:_REPORT_WORDS] for lay in net.layers]}
    lay = state["lay"]
    if state["case"]["kind"] == "erroneous":
        lay.protected_fused(state["D"], state["W"], state["O"], state["faults"])
    else:
        lay.protected(state["D"], state["W"], state["O"])
    out = {"O": state["O"], "report": lay.report.view(torch.int32)[:_REPORT_WORDS]}
    for k in ("cd1", "cd2", "co5", "co6", "co7", "so5", "so6", "so7", "q5"):
        out[k] = lay.buf[k]
    return out


def work(case):
    if case["kind"] != "chain":
        _, _, flops, b = _sizes(case)
        return {"bytes": b, "flops": flops}
    es = 4 if case["dtype"] == "f32" else 2
    sp = _specs(case)
    flops = b = 0.0
    for i, s in enumerate(sp):
        e = (s.h + 2 * s.pad - s.r) // s.stride + 1
        f = (s.w + 2 * s.pad - s.s) // s.stride + 1
        flops += 2.0 * s.n * s.m * e * f * s.ch * s.r * s.s
        b += es * s.m * s.ch * s.r * s.s
        if i == 0:
            b += es * s.n * s.ch * s.h * s.w
        if i == len(sp) - 1:
            b += es * s.n * s.m * e * f
    return {"bytes": b, "flops": flops}


def tolerance(case):
    # about four times the measured distance from 64 bits: fp32 outputs 1e-7 to 2.2e-6 (the longest
    # sums), bf16 outputs 1.7e-3 (their rounding), their sums up to 4e-3, a bf16 network's 5.4e-3
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 2e-2, "max": 0.4} if case["kind"] == "chain" else {"rel": 1e-2}


def _conv64(D, W, stride, pad, groups):
    """Eq. (1) in float64, one kernel tap at a time."""
    n, ch, h, w = D.shape
    m, cg, r, s = W.shape
    e, f = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1
    Dp = torch.nn.functional.pad(D, (pad, pad, pad, pad))
    mg = m // groups
    O = torch.zeros(n, groups, mg, e * f, dtype=torch.float64, device=D.device)
    step = max(1, int(2e8 // max(1, ch * e * f)))   # images at a time
    for i in range(r):
        for j in range(s):
            for n0 in range(0, n, step):
                X = Dp[n0:n0 + step, :, i:i + stride * (e - 1) + 1:stride, j:j + stride * (f - 1) + 1:stride]
                X = X.reshape(X.shape[0], groups, cg, e * f)
                for g in range(groups):
                    A = W[g * mg:(g + 1) * mg, :, i, j].contiguous()
                    O[n0:n0 + step, g] += torch.matmul(A, X[:, g].contiguous())
    return O.reshape(n, m, e, f)


def exact(case, seed):
    if work(case)["flops"] > 4e11:
        return None
    D, Ws, bias = _inputs(case, seed)
    X = D.double()
    if case["kind"] == "chain":
        sp = _specs(case)
        for i, s in enumerate(sp):
            X = _conv64(X, Ws[i].double(), s.stride, s.pad, 1)
            if i + 1 < len(sp):
                X = X.relu()
                k, st = network.pooling(X.shape[2], sp[i + 1].h)
                if k > 1:
                    X = torch.nn.functional.max_pool2d(X, k, st)
        return {"output": X, "reports": [None] * len(sp)}
    W = Ws[0].double()
    n, m, groups = case["n"], case["m"], case["groups"]
    mg, cg = m // groups, case["ch"] // groups
    wn = torch.arange(n, dtype=torch.float64, device=X.device)
    wm = torch.arange(m, dtype=torch.float64, device=X.device)
    O = _conv64(X, W, case["stride"], case["pad"], groups)
    cd1, cd2 = X.sum(0), (X * wn.view(-1, 1, 1, 1)).sum(0)
    # the filters' checksums, each group's side by side over the channels
    Wg = W.view(groups, mg, cg, case["r"], case["s"])
    cw1 = Wg.sum(1).reshape(1, case["ch"], case["r"], case["s"])
    cw2 = (Wg * wm.view(groups, mg, 1, 1, 1)).sum(1).reshape(1, case["ch"], case["r"], case["s"])

    def co(d, k):
        return _conv64(d.unsqueeze(0), k, case["stride"], case["pad"], 1).reshape(-1)

    out = {"O": O, "report": None, "cd1": cd1.reshape(-1), "cd2": cd2.reshape(-1),
           "co5": co(cd1, cw1), "co6": co(cd1, cw2), "co7": co(cd2, cw1)}
    if bias is not None:
        O += bias.double().view(1, -1, 1, 1)
    if case["faults"]:
        # the detected sums hold the planted faults as the output's type rounds them
        out.update(so5=None, so6=None, so7=None, q5=None)
    else:
        out["so5"] = O.sum((0, 1)).reshape(-1)
        out["so6"] = (O * wm.view(1, -1, 1, 1)).sum((0, 1)).reshape(-1)
        out["so7"] = (O * wn.view(-1, 1, 1, 1)).sum((0, 1)).reshape(-1)
        out["q5"] = (O * O).sum((0, 1)).sqrt().reshape(-1)
    return out

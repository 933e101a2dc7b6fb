"""The work that programs have this library do, as cases that can be timed.

A case is one block of a network as the training or the serving loop of a user runs it, through the tensor-level
functions of paper_1412_4564_amd.binding:

  train    forward (with the ReLU that follows, where `relu` is set), then the derivatives with respect to the input,
           the filters and the biases: one training step of a convolution block
  serve    conv_relu_forward alone: one block of a network that answers requests
  decoder  the convolution transpose block, forward and its three derivatives
  pool     the spatial pooling block, forward and derivative

Layer shapes are those of paper_1412_4564_amd.synth (the networks of the MatConvNet manual), sizes as in its notation:
x is H x W x D x N, w is Hf x Wf x Df x K.
"""
import math

import torch

from paper_1412_4564_amd import binding as B
from paper_1412_4564_amd import synth

PRECISION = {"fp32": B.MCN_PREC_FP32, "bf16": B.MCN_PREC_BF16, "bf16x3": B.MCN_PREC_FP32_BF16X3}


def _conv(kind, H, W, D, N, Hf, Wf, Df, K, stride=(1, 1), pad=(0, 0, 0, 0), precision="fp32", relu=False):
    return {"kind": kind, "H": H, "W": W, "D": D, "N": N, "Hf": Hf, "Wf": Wf, "Df": Df, "K": K, "Sh": stride[0],
            "Sw": stride[1], "Pt": pad[0], "Pb": pad[1], "Pl": pad[2], "Pr": pad[3], "precision": precision, "relu": relu}


def _layer(kind, name, **more):
    L = synth.LAYERS[name]
    return _conv(kind, L["H"], L["W"], L["D"], L["N"], L["Hf"], L["Wf"], L["Df"], L["K"], L["stride"], L["pad"], **more)


def _decoder(H, W, D, N, Hf, Wf, Kf, up=(1, 1), crop=(0, 0, 0, 0), precision="fp32"):
    return {"kind": "decoder", "H": H, "W": W, "D": D, "N": N, "Hf": Hf, "Wf": Wf, "Kf": Kf, "Uh": up[0], "Uw": up[1],
            "Ct": crop[0], "Cb": crop[1], "Cl": crop[2], "Cr": crop[3], "precision": precision}


def _pool(H, W, D, N, window, stride, pad, method):
    return {"kind": "pool", "H": H, "W": W, "D": D, "N": N, "Hp": window[0], "Wp": window[1], "Sh": stride[0], "Sw": stride[1],
            "Pt": pad[0], "Pb": pad[1], "Pl": pad[2], "Pr": pad[3], "method": method}


def listed():
    def named(name, case):
        return dict(case, name=name)

    t2, p3 = synth.CONVT_LAYERS["t2"], synth.POOL_LAYERS["p3"]
    return [
        # the smallest training step: a few images, odd plane, unequal strides and pads (latency and launches count)
        named("irregular small", _layer("train", "5c")),
        # serving one image: the deepest 3x3 block of a VGG-style network answering a single request
        named("one image", _conv("serve", 14, 14, 512, 1, 3, 3, 512, 512, (1, 1), (1, 1, 1, 1), relu=True)),
        # the middle block of a CIFAR-sized network, batch 100, with its ReLU
        named("cifar middle", _layer("train", "2b", relu=True)),
        # the first layer of the Krizhevsky-style network: three channels, 11x11 filters, stride 4
        named("first layer", _layer("train", "3a")),
        # its second layer: two filter groups, 5x5, with its ReLU
        named("two groups", _layer("train", "3b", relu=True)),
        # the large planes at the start of a VGG-style network, default precision: the largest case
        named("vgg 224", _layer("train", "4a")),
        # its middle, with operands rounded to bf16 (the option for those who trade precision for speed)
        named("vgg 56 bf16", _layer("train", "4b", precision="bf16", relu=True)),
        # its end, with operands split into two bf16 numbers (the option in between)
        named("vgg 14 split", _layer("train", "4c", precision="bf16x3")),
        # the first fully-connected layer, run as a 6x6 convolution
        named("fully connected", _layer("train", "5a")),
        # a 1x1 layer that reduces the channels
        named("pointwise", _layer("train", "5b")),
        # a decoder layer that doubles the resolution
        named("decoder", _decoder(t2["H"], t2["W"], t2["D"], t2["N"], t2["Hf"], t2["Wf"], t2["Kf"], t2["up"], t2["crop"])),
        # the pooling block after the first layer of the Krizhevsky-style network: overlapping 3x3 windows
        named("max pool", _pool(p3["H"], p3["W"], p3["D"], p3["N"], p3["window"], p3["stride"], p3["pad"], p3["method"])),
    ]


def _out(n, f, s, p0, p1):
    return (n + p0 + p1 - f) // s + 1


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Filter and channel counts: mostly multiples of 8, some odd."""
    c = _log(rng, lo, hi)
    return c if rng.random() < 0.3 else max(lo, (c + 4) // 8 * 8)


def _draw(rng):
    kind = rng.choice(["small", "serve", "cifar", "first", "groups", "deep", "deep", "deep", "fc", "pointwise", "decoder", "pool"])
    precision = rng.choice(["fp32", "fp32", "bf16", "bf16x3"])
    relu = rng.random() < 0.5
    if kind == "small":          # latency: up to a few megabytes
        f = (rng.randint(2, 5), rng.randint(2, 5))
        d = _channels(rng, 3, 32)
        return _conv("train", _log(rng, 12, 40), _log(rng, 12, 53), d, rng.randint(2, 8), f[0], f[1], d, _channels(rng, 16, 40),
                     (rng.randint(1, 3), rng.randint(1, 3)), tuple(rng.randint(0, 2) for _ in range(4)), "fp32", relu)
    if kind == "serve":          # one to four images through one block
        h = _log(rng, 7, 112)
        d = _channels(rng, 64, 512 if h < 60 else 128)
        f = rng.choice([1, 3, 3, 5])
        return _conv("serve", h, h + rng.randint(0, 3), d, rng.randint(1, 4), f, f, d, _channels(rng, 64, 512), (1, 1), (f // 2,) * 4,
                     precision, True)
    if kind == "cifar":          # small planes, 5x5, a batch of about a hundred
        d = _channels(rng, 16, 64)
        h = rng.choice([8, 16, 32, rng.randint(7, 32)])
        return _conv("train", h, h, d, rng.randint(50, 128), 5, 5, d, _channels(rng, 24, 96), (1, 1), (2, 2, 2, 2), "fp32", relu)
    if kind == "first":          # three channels, large filters and strides
        f, s = rng.choice([(11, 4), (7, 2), (5, 1), (5, 2)])
        h = _log(rng, 64, 227)
        return _conv("train", h, h, 3, _log(rng, 16, 128), f, f, 3, rng.choice([64, 96, _channels(rng, 32, 96)]), (s, s),
                     (rng.randint(0, f // 2),) * 4, "fp32", relu)
    if kind == "groups":         # two filter groups
        d, f = _channels(rng, 24, 96), rng.choice([3, 5])
        h = rng.randint(13, 31)
        return _conv("train", h, h, 2 * d, _log(rng, 16, 128), f, f, d, 2 * _channels(rng, 48, 128), (1, 1), (f // 2,) * 4, precision, relu)
    if kind == "deep":           # 3x3 layers of a deep network
        h = _log(rng, 10, 224)
        d = _channels(rng, 32, max(48, min(512, 14336 // h)))
        k = _channels(rng, 48, max(64, min(512, 14336 // h)))
        return _conv("train", h, h + rng.randint(0, 2), d, _log(rng, 8, 48), 3, 3, d, k, (1, 1), (1, 1, 1, 1), precision, relu)
    if kind == "fc":             # a filter as large as its input
        h, d = rng.randint(1, 7), _channels(rng, 128, 512)
        return _conv("train", h, h, d, _log(rng, 32, 256), h, h, d, _channels(rng, 500, 4096))
    if kind == "pointwise":      # 1x1
        return _conv("train", _log(rng, 7, 56), _log(rng, 7, 56), _channels(rng, 64, 512), _log(rng, 16, 64), 1, 1, 0, _channels(rng, 64, 256),
                     (1, 1), (0, 0, 0, 0), precision, relu)
    if kind == "decoder":        # twice the resolution
        h = rng.randint(9, 40)
        return _decoder(h, h, _channels(rng, 32, 256), _log(rng, 8, 32), 4, 4, _channels(rng, 32, 160), (2, 2), (1, 1, 1, 1), precision)
    method = rng.choice(["max", "max", "avg"])
    f, s = rng.choice([(2, 2), (3, 2), (3, 2), (3, 3)])
    return _pool(_log(rng, 12, 224), _log(rng, 12, 224), _channels(rng, 16, 96), _log(rng, 8, 128), (f, f), (s, s),
                 (0, rng.randint(0, f - 1), 0, rng.randint(0, f - 1)), method)


def draw(rng):
    """One more case of the same ranges, no costlier than the largest listed one."""
    most = work(_layer("train", "4a"))
    while True:
        case = _draw(rng)
        if case.get("Df") == 0:
            case["Df"] = case["D"]
        w = work(case)
        if w["bytes"] <= 0.9 * most["bytes"] and w["flops"] <= 0.9 * most["flops"]:
            return case


def _shapes(case):
    """x, w and y of a case, in the order of torch's axes (images, channels, columns, rows); w is None for pooling."""
    c = case
    x = (c["N"], c["D"], c["W"], c["H"])
    if c["kind"] == "decoder":
        ho = c["Uh"] * (c["H"] - 1) + c["Hf"] - c["Ct"] - c["Cb"]
        wo = c["Uw"] * (c["W"] - 1) + c["Wf"] - c["Cl"] - c["Cr"]
        return x, (c["D"], c["Kf"], c["Wf"], c["Hf"]), (c["N"], c["Kf"], wo, ho)
    fh, fw = (c["Hp"], c["Wp"]) if c["kind"] == "pool" else (c["Hf"], c["Wf"])
    ho, wo = _out(c["H"], fh, c["Sh"], c["Pt"], c["Pb"]), _out(c["W"], fw, c["Sw"], c["Pl"], c["Pr"])
    if c["kind"] == "pool":
        return x, None, (c["N"], c["D"], wo, ho)
    return x, (c["K"], c["Df"], c["Wf"], c["Hf"]), (c["N"], c["K"], wo, ho)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    xs, ws, ys = _shapes(case)

    def normal(shape, std=1.0):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std)

    s = {"case": dict(case), "x": normal(xs), "workspace": B.Workspace()}
    if ws is not None:           # He-scaled weights, small biases
        fan = ws[2] * ws[3] * (ws[1] if case["kind"] != "decoder" else ws[0])
        s["w"], s["b"] = normal(ws, (2.0 / fan) ** 0.5), normal((ys[1],), 0.1)
    if case["kind"] != "serve":
        s["dzdy"] = normal(ys)
    if case["kind"] == "train" and case["relu"]:
        # The activations that an earlier forward pass kept: the backward half takes its mask from them, so that a sum whose
        # last bit falls on the other side of zero does not change the derivatives.
        s["kept"] = normal(ys).clamp_(min=0.0)
    return s


def run(state):
    c, ws = state["case"], state["workspace"]
    x = state["x"]
    if c["kind"] == "pool":
        geometry = ((c["Hp"], c["Wp"]), (c["Sh"], c["Sw"]), (c["Pt"], c["Pb"], c["Pl"], c["Pr"]),
                    B.MCN_POOL_MAX if c["method"] == "max" else B.MCN_POOL_AVG)
        return {"y": B.pool_forward(x, *geometry), "dzdx": B.pool_backward(x, state["dzdy"], *geometry, workspace=ws)}
    w, b, precision = state["w"], state["b"], PRECISION[c["precision"]]
    if c["kind"] == "decoder":
        up, crop, dzdy = (c["Uh"], c["Uw"]), (c["Ct"], c["Cb"], c["Cl"], c["Cr"]), state["dzdy"]
        return {"y": B.convt_forward(x, w, b, up, crop, 1, precision, workspace=ws),
                "dzdx": B.convt_backward_data(x.shape, w, dzdy, up, crop, 1, precision, workspace=ws),
                "dzdf": B.convt_backward_filter(x, w.shape, dzdy, up, crop, 1, precision, workspace=ws),
                "dzdb": B.convt_backward_bias(x.shape, w.shape, dzdy, up, crop, 1, workspace=ws)}
    stride, pad = (c["Sh"], c["Sw"]), (c["Pt"], c["Pb"], c["Pl"], c["Pr"])
    if c["kind"] == "serve":
        return {"y": B.conv_relu_forward(x, w, b, stride, pad, precision, workspace=ws)}
    out, dzdy = {}, state["dzdy"]
    if c["relu"]:
        out["y"] = B.conv_relu_forward(x, w, b, stride, pad, precision, workspace=ws)
        dzdy, out["dzdb"] = B.conv_relu_backward_bias(x.shape, w.shape, state["kept"], dzdy, stride, pad, workspace=ws)
        out["dzdp"] = dzdy
        out["dzdw"] = B.conv_backward_filter(x, w.shape, dzdy, stride, pad, precision, workspace=ws)
    else:
        out["y"] = B.conv_forward(x, w, b, stride, pad, precision, workspace=ws)
        out["dzdw"], out["dzdb"] = B.conv_backward_filter_bias(x, w.shape, dzdy, stride, pad, precision, workspace=ws)
    out["dzdx"] = B.conv_backward_data(x.shape, w, dzdy, stride, pad, precision, workspace=ws)
    return out


def work(case):
    xs, ws, ys = _shapes(case)
    nx, ny = math.prod(xs), math.prod(ys)
    if case["kind"] == "pool":   # x and dzdy in, y and dzdx out (the average's derivative does not need x; its forward does)
        return {"bytes": 4.0 * (2 * nx + 2 * ny), "flops": float(ny * case["Hp"] * case["Wp"] + nx)}
    nw = math.prod(ws)
    if case["kind"] == "decoder":    # every input sample meets every tap of every output channel
        macs = nx * ws[1] * ws[2] * ws[3]
    else:                            # every output sample meets every tap of every channel of its group
        macs = ny * ws[1] * ws[2] * ws[3]
    if case["kind"] == "serve":
        return {"bytes": 4.0 * (nx + nw + ys[1] + ny), "flops": 2.0 * macs}
    # x, w, b and dzdy in; y, dzdx, dzdw and dzdb out; with the ReLU also the kept activations in and dzdp out
    relu = 2 * ny if case.get("relu") else 0
    return {"bytes": 4.0 * (2 * nx + 2 * nw + 2 * ys[1] + 2 * ny + relu), "flops": 6.0 * macs}


def tolerance(case):
    """Four times what the results differ by from sums in 64 bits, over the listed cases and a dozen drawn ones (2-norm, and
    largest difference): fp32 1.3e-6 and 6.7e-6, operands of two bf16 numbers 4.4e-6 and 3.7e-5, bf16 2.4e-3 and 1.9e-2."""
    if case["kind"] == "pool":   # windows that do not overlap only select; the others add a few numbers
        return "exact" if case["method"] == "max" and case["Sh"] == case["Hp"] and case["Sw"] == case["Wp"] else {"rel": 1e-6}
    return {"fp32": {"rel": 5e-6, "max": 4e-5}, "bf16x3": {"rel": 1.8e-5, "max": 1.5e-4}, "bf16": {"rel": 1e-2, "max": 8e-2}}[case["precision"]]


def _windows(case):
    """The taps of a window, in memory order: (column, row, and the slices of a padded plane that the tap meets over all windows)."""
    c = case
    fh, fw = (c["Hp"], c["Wp"]) if c["kind"] == "pool" else (c["Hf"], c["Wf"])
    ho, wo = _out(c["H"], fh, c["Sh"], c["Pt"], c["Pb"]), _out(c["W"], fw, c["Sw"], c["Pl"], c["Pr"])
    for fj in range(fw):
        for fi in range(fh):
            yield fj, fi, slice(fj, fj + (wo - 1) * c["Sw"] + 1, c["Sw"]), slice(fi, fi + (ho - 1) * c["Sh"] + 1, c["Sh"])


def _exact_pool(c, s):
    x, dzdy = s["x"].double(), s["dzdy"].double()
    pad = (c["Pt"], c["Pb"], c["Pl"], c["Pr"])
    inside = slice(c["Pl"], c["Pl"] + c["W"]), slice(c["Pt"], c["Pt"] + c["H"])
    dxp = torch.nn.functional.pad(torch.zeros_like(x), pad)
    if c["method"] == "max":
        xp = torch.nn.functional.pad(x, pad, value=-math.inf)
        y = torch.full_like(dzdy, -math.inf)
        which = torch.zeros(dzdy.shape, dtype=torch.int32, device=x.device)
        for t, (_, _, cols, rows) in enumerate(_windows(c)):
            v = xp[:, :, cols, rows]
            which.masked_fill_(v > y, t)
            y = torch.maximum(y, v)
        for t, (_, _, cols, rows) in enumerate(_windows(c)):
            dxp[:, :, cols, rows] += dzdy * (which == t)
    else:
        xp, ones = torch.nn.functional.pad(x, pad), torch.nn.functional.pad(torch.ones_like(x[:1, :1]), pad)
        y, count = torch.zeros_like(dzdy), 0
        for _, _, cols, rows in _windows(c):
            y += xp[:, :, cols, rows]
            count = count + ones[:, :, cols, rows]
        y /= count
        for _, _, cols, rows in _windows(c):
            dxp[:, :, cols, rows] += dzdy / count
    return {"y": y, "dzdx": dxp[:, :, inside[0], inside[1]]}


def _exact_conv(c, x, w, b, dzdy, bias):
    """Forward and the three derivatives as sums over the filter's taps; dzdy None: forward alone."""
    groups = x.shape[1] // w.shape[1]
    n, k, df = x.shape[0], w.shape[0], w.shape[1]
    kg = k // groups
    xp = torch.nn.functional.pad(x, (c["Pt"], c["Pb"], c["Pl"], c["Pr"]))
    taps = list(_windows(c))
    wo, ho = _out(c["W"], c["Wf"], c["Sw"], c["Pl"], c["Pr"]), _out(c["H"], c["Hf"], c["Sh"], c["Pt"], c["Pb"])
    y = torch.zeros((n, k, wo * ho), dtype=x.dtype, device=x.device)
    out = {}
    if dzdy is not None:
        p = dzdy.reshape(n, k, wo * ho)
        dxp, dw = torch.zeros_like(xp), torch.zeros_like(w)
    for fj, fi, cols, rows in taps:
        for g in range(groups):
            ch, ks = slice(g * df, (g + 1) * df), slice(g * kg, (g + 1) * kg)
            patch = xp[:, ch, cols, rows].reshape(n, df, wo * ho)
            f = w[ks, :, fj, fi].contiguous()
            y[:, ks] += torch.matmul(f, patch)
            if dzdy is not None:
                pg = p[:, ks].contiguous()
                dw[ks, :, fj, fi] = torch.matmul(pg, patch.transpose(1, 2).contiguous()).sum(0)
                dxp[:, ch, cols, rows] += torch.matmul(f.t().contiguous(), pg).reshape(n, df, wo, ho)
    out["y"] = (y + b[:, None]).reshape(n, k, wo, ho) if bias else y.reshape(n, k, wo, ho)
    if dzdy is not None:
        out["dzdx"] = dxp[:, :, c["Pl"]:c["Pl"] + c["W"], c["Pt"]:c["Pt"] + c["H"]]
        out["dzdw"], out["dzdb"] = dw, dzdy.sum((0, 2, 3))
    return out


def exact(case, seed):
    """What run() returns for these inputs, in 64 bits and plain torch (for every precision: of the inputs as they are)."""
    c, s = case, prepare(case, seed)
    if c["kind"] == "pool":
        return _exact_pool(c, s)
    x, w, b = s["x"].double(), s["w"].double(), s["b"].double()
    if c["kind"] == "decoder":
        # the transpose of a convolution that takes arrays of y's shape to arrays of x's: forward is its derivative with
        # respect to its input, and the other way round
        dzdy = s["dzdy"].double()
        back = {"kind": "train", "H": dzdy.shape[3], "W": dzdy.shape[2], "Hf": c["Hf"], "Wf": c["Wf"], "Sh": c["Uh"], "Sw": c["Uw"],
                "Pt": c["Ct"], "Pb": c["Cb"], "Pl": c["Cl"], "Pr": c["Cr"]}
        r = _exact_conv(back, dzdy, w, None, x, False)
        return {"y": r["dzdx"] + b[:, None, None], "dzdx": r["y"], "dzdf": r["dzdw"], "dzdb": dzdy.sum((0, 2, 3))}
    if c["kind"] == "serve":
        return {"y": _exact_conv(c, x, w, b, None, True)["y"].clamp_(min=0.0)}
    dzdy, out = s["dzdy"].double(), {}
    if c["relu"]:
        dzdy = out["dzdp"] = dzdy * (s["kept"] > 0)
    r = _exact_conv(c, x, w, b, dzdy, True)
    if c["relu"]:
        r["y"] = r["y"].clamp_(min=0.0)
    out.update(r)
    return out

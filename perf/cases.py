"""The work that users of this library have it do, as cases that can be timed and compared.

Four kinds, each through the entry points that a program calls:

  layer     one XConv2d layer in training: forward call and backward pass (output, input, weight and bias gradient)
  stack     a network of convolutions and ReLUs swapped by convert_net, forward and backward
  estimate  the C interface as a framework of its own would call it: probe in the forward pass, weight-gradient estimate
            in the backward pass, buffers kept by the caller
  volume    the same two calls for a volumetric (3-D) layer

The sizes are those of the benchmark layers C1..C5 and V2 (paper_2106_06998_amd/synth.py, bench.py) and generic ones.
"""
import itertools
import math

import torch

import paper_2106_06998_amd.layer as xlayer
from paper_2106_06998_amd import binding as xb

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _layer(name, B, cin, cout, h, w, k, stride, pad, r, dtype, probe="rademacher", mode="channel", layout="nchw", bias=True):
    return dict(name=name, kind="layer", B=B, cin=cin, cout=cout, h=h, w=w, k=k, stride=stride, pad=pad, r=r, dtype=dtype,
                probe=probe, mode=mode, layout=layout, bias=bias)


def _estimate(name, B, cin, cout, h, w, k, stride, pad, r, dtype, probe, layout="nchw"):
    return dict(name=name, kind="estimate", B=B, cin=cin, cout=cout, h=h, w=w, k=k, stride=stride, pad=pad, r=r, dtype=dtype,
                probe=probe, layout=layout)


def listed():
    return [
        # the smallest training step (C1): launches and the Python around them are what counts
        _layer("layer C1 f32", 4, 16, 16, 32, 32, 3, 1, 1, 8, "f32"),
        # a CIFAR-size layer in single precision (C2), Gaussian probing vectors
        _layer("layer C2 f32", 128, 64, 64, 32, 32, 3, 1, 1, 16, "f32", "gaussian"),
        # a residual network's downsampling layer in bfloat16 (C3)
        _layer("layer C3 bf16 stride 2", 64, 128, 256, 56, 56, 3, 2, 1, 32, "bf16", bias=False),
        # the largest benchmark layer in half precision (C5)
        _layer("layer C5 f16", 256, 256, 256, 28, 28, 3, 1, 1, 64, "f16"),
        # a bottleneck's 1x1 convolution: few operations for each byte
        _layer("layer 1x1 bf16", 64, 256, 64, 56, 56, 1, 1, 0, 32, "bf16", bias=False),
        # channels-last tensors, an odd image size and channel counts that are no powers of two
        _layer("layer channels-last bf16", 24, 96, 144, 45, 37, 3, 1, 1, 24, "bf16", layout="nhwc"),
        # the paper's probes over pixels and channels, where the stored state is B*r numbers
        _layer("layer multi f32", 64, 64, 64, 32, 32, 3, 1, 1, 16, "f32", "gaussian", mode="multi"),
        # a converted network: six convolutions with sign-bit ReLUs in half the bytes
        dict(name="stack bf16", kind="stack", B=128, c=64, h=32, w=32, depth=6, r=16, dtype="bf16", probe="rademacher", mode="channel"),
        # the C interface alone on the smallest benchmark layer (C1)
        _estimate("estimate C1 f32", 4, 16, 16, 32, 32, 3, 1, 1, 8, "f32", "rademacher"),
        # ... at high resolution (C4: U-Net-like layers)
        _estimate("estimate C4 f32", 8, 64, 64, 256, 256, 3, 1, 1, 16, "f32", "gaussian"),
        # ... and on the headline layer (C5)
        _estimate("estimate C5 f16", 256, 256, 256, 28, 28, 3, 1, 1, 64, "f16", "rademacher"),
        # a volumetric layer on a CT-like patch (V2)
        dict(name="volume V2 f16", kind="volume", B=1, cin=128, cout=128, d=48, h=48, w=48, k=3, stride=1, pad=1, r=32, dtype="f16",
             probe="rademacher", layout="nchw"),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v / step) * step))


def _channels(rng, lo=16, hi=256):
    """Mostly multiples of 8, as networks have them; one in four is any number."""
    return _log_int(rng, lo, hi, 8 if rng.random() < 0.75 else 1)


def _drawn(rng):
    kind = rng.choice(["layer", "layer", "layer", "estimate", "estimate", "stack", "volume"])
    dtype = rng.choice(["f32", "bf16", "f16"])
    probe = rng.choice(["rademacher", "gaussian"])
    if kind == "stack":
        h = _log_int(rng, 14, 64)
        return dict(kind=kind, B=_log_int(rng, 8, 128), c=_log_int(rng, 32, 128, 8), h=h, w=h, depth=rng.randint(2, 8),
                    r=rng.choice([4, 8, 16]), dtype=dtype, probe=probe, mode=rng.choice(["channel", "channel", "multi"]))
    cin, cout = _channels(rng), _channels(rng)
    r = rng.choice([v for v in (4, 8, 12, 16, 24, 32, 64) if 2 * v <= cin])
    if kind == "volume":
        h = _log_int(rng, 12, 64)
        return dict(kind=kind, B=rng.choice([1, 1, 2, 4]), cin=cin, cout=cout, d=_log_int(rng, 12, 64), h=h, w=h + rng.choice([0, 0, -3, 4]),
                    k=3, stride=1, pad=1, r=r, dtype=dtype, probe=probe, layout=rng.choice(["nchw", "nchw", "nhwc"]))
    h = _log_int(rng, 7, 256)
    w = h if rng.random() < 0.6 else _log_int(rng, max(7, h // 2), min(256, 2 * h))
    k = rng.choice([1, 3, 3, 3, 3, 5])
    case = dict(kind=kind, B=_log_int(rng, 2, 256), cin=cin, cout=cout, h=h, w=w, k=k, stride=rng.choice([1, 1, 1, 2]), pad=k // 2, r=r,
                dtype=dtype, probe=probe, layout=rng.choice(["nchw", "nchw", "nhwc"]))
    if kind == "layer":
        case.update(mode=rng.choice(["channel", "channel", "channel", "multi"]), bias=rng.random() < 0.6)
    return case


def _cost(case):
    """Seconds, roughly, that decide whether a drawn case is too large."""
    w = work(case)
    s = w["flops"] / (1.2e14 if case["dtype"] == "f32" else 1e15) + w["bytes"] / 4e12
    if case.get("mode") == "multi":        # the probing vectors are drawn in each pass, one for each value of an image
        values = case["c"] * case["depth"] if case["kind"] == "stack" else case["cin"]
        s += 2e-11 * values * case["h"] * case["w"] * case["r"]
    return s


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _drawn(rng)
        if _cost(case) <= most:
            return case


def _out(n, case):
    return (n + 2 * case["pad"] - case["k"]) // case["stride"] + 1


def work(case):
    """Bytes and operations of one pass: every input read once, every output written once, the estimator's own operations."""
    s = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "stack":
        c, n = case["c"], case["B"] * case["h"] * case["w"]
        one = dict(case, kind="layer", cin=c, cout=c, k=3, stride=1, pad=1, bias=True)
        flops = case["depth"] * work(one)["flops"] - 2.0 * n * c * c * 9      # the first layer's input needs no gradient
        # the input, the output and its gradient; the weights, biases and their gradients
        return dict(bytes=3.0 * n * c * s + case["depth"] * 2 * (c * c * 9 + c) * s, flops=flops)
    B, cin, cout, r = case["B"], case["cin"], case["cout"], case["r"]
    d, do, kd = (case["d"], _out(case["d"], case), case["k"]) if case["kind"] == "volume" else (1, 1, 1)
    q, p, k2 = B * d * case["h"] * case["w"], B * do * _out(case["h"], case) * _out(case["w"], case), case["k"] ** 2 * kd
    x, y, wt = float(q * cin * s), float(p * cout * s), cout * cin * k2
    if case["kind"] in ("estimate", "volume"):
        # the stored probe output passes from one call to the other in the caller's buffer: written once, read once
        return dict(bytes=x + y + 4.0 * wt + 2.0 * q * r * s, flops=2.0 * q * cin * r + 2.0 * p * cout * r * k2 + 2.0 * wt * r)
    if case["mode"] == "multi":
        est = 2.0 * q * cin * r + 2.0 * p * cout * r + 2.0 * (p // B) * r * cout * cin * k2
    else:
        est = 2.0 * q * cin * r + 2.0 * p * cout * r * k2 + 2.0 * wt * r
    return dict(bytes=2 * x + 2 * y + 2.0 * (wt + (cout if case["bias"] else 0)) * s, flops=4.0 * p * cout * cin * k2 + est)


def tolerance(case):
    """Outputs rounded to the storage type from fp32 sums; the stored probe output is rounded to it too."""
    return {"rel": {"f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}[case["dtype"]]}


class _State:
    pass


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(1 + seed)
    td = DTYPES[case["dtype"]]
    kind = case["kind"]
    s = _State()
    s.kind, s.seed = kind, seed

    def normal(shape, std, relu=False):
        t = torch.randn(shape, device=DEV, generator=g)
        return (t.relu_() if relu else t).mul_(std).to(td)

    if kind == "stack":
        c, shape = case["c"], (case["B"], case["c"], case["h"], case["w"])
        mods = []
        for _ in range(case["depth"]):
            mods += [torch.nn.Conv2d(c, c, 3, padding=1, device=DEV, dtype=td), torch.nn.ReLU()]
        s.net, _ = xlayer.convert_net(torch.nn.Sequential(*mods), r=case["r"], probe=case["probe"], mode=case["mode"], relu=True)
        with torch.no_grad():
            for m in s.net:
                if isinstance(m, xlayer.XConv2d):
                    m.base_seed += 1000 * seed
                    m.weight.copy_(normal(m.weight.shape, (2.0 / (9 * c)) ** 0.5))
                    m.bias.copy_(normal(m.bias.shape, 0.1))
        s.params = list(s.net.parameters())
        s.x, s.dy = normal(shape, 1.0, relu=True), normal(shape, 0.1)
        return s

    B, cin, cout, h, w, k = (case[n] for n in ("B", "cin", "cout", "h", "w", "k"))
    if kind == "volume":
        nhwc = case["layout"] == "nhwc"
        xs, ys = (case["d"], h, w), tuple(_out(n, case) for n in (case["d"], h, w))
        s.x = normal((B, *xs, cin) if nhwc else (B, cin, *xs), 1.0, relu=True)
        s.dy = normal((B, *ys, cout) if nhwc else (B, cout, *ys), 0.1)
        s.desc = xb.make_desc3d(B, cin, cout, case["d"], h, w, k, case["stride"], case["pad"], case["r"], case["dtype"], case["probe"],
                                seed, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
        s.xt = xb.alloc_bytes(xb.xconv3d_xt_bytes(s.desc), DEV)
        s.ws_probe = xb.alloc_bytes(xb.xconv3d_workspace_bytes(s.desc, xb.XCONV_OP_PROBE), DEV)
        s.ws = xb.alloc_bytes(xb.xconv3d_workspace_bytes(s.desc, xb.XCONV_OP_ESTIMATE), DEV)
        s.dw = torch.empty((cout, cin, k, k, k), dtype=torch.float32, device=DEV)
        return s

    ho, wo = _out(h, case), _out(w, case)
    nhwc = case["layout"] == "nhwc"
    if kind == "estimate":
        s.x = normal((B, h, w, cin) if nhwc else (B, cin, h, w), 1.0, relu=True)
        s.dy = normal((B, ho, wo, cout) if nhwc else (B, cout, ho, wo), 0.1)
        s.desc = xb.make_desc(B, cin, cout, h, w, k, case["stride"], case["pad"], case["r"], case["dtype"], case["probe"], seed,
                              xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
        s.xt = xb.alloc_xt(s.desc, DEV)
        s.ws_probe = xb.alloc_ws(s.desc, xb.XCONV_OP_PROBE, DEV)
        s.ws = xb.alloc_ws(s.desc, xb.XCONV_OP_ESTIMATE, DEV)
        s.dw = torch.empty((cout, cin, k, k), dtype=torch.float32, device=DEV)
        return s

    fmt = torch.channels_last if nhwc else torch.contiguous_format
    s.layer = xlayer.XConv2d(cin, cout, k, r=case["r"], stride=case["stride"], padding=case["pad"], bias=case["bias"], probe=case["probe"],
                             mode=case["mode"], base_seed=seed, device=DEV, dtype=td)
    with torch.no_grad():
        s.layer.weight.copy_(normal(s.layer.weight.shape, (2.0 / (cin * k * k)) ** 0.5))
        if case["bias"]:
            s.layer.bias.copy_(normal(s.layer.bias.shape, 0.1))
    s.x = normal((B, cin, h, w), 1.0, relu=True).contiguous(memory_format=fmt).requires_grad_(True)
    s.dy = normal((B, cout, ho, wo), 0.1).contiguous(memory_format=fmt)
    s.wanted = [s.x] + list(s.layer.parameters())
    return s


def run(s):
    # the stored probe output is not returned: its layout is the library's own, and the gradient is computed from all of it
    if s.kind == "estimate":
        xb.xconv_probe_fwd(s.desc, s.x, s.xt, None, s.ws_probe)
        xb.xconv_dw_estimate(s.desc, s.dy, s.xt, None, s.dw, s.ws)
        return s.dw
    if s.kind == "volume":
        xb.xconv3d_probe_fwd(s.desc, s.x, s.xt, None, s.ws_probe)
        xb.xconv3d_dw_estimate(s.desc, s.dy, s.xt, None, s.dw, s.ws)
        return s.dw
    # the layers draw fresh probing vectors at every call; counted from here, the same ones for every pass on this state
    xlayer._calls = itertools.count(1)
    if s.kind == "stack":
        y = s.net(s.x)
        return [y] + list(torch.autograd.grad(y, s.params, s.dy))
    y = s.layer(s.x)
    return [y] + list(torch.autograd.grad(y, s.wanted, s.dy))

"""The work whose speed matters here: what a program that runs pattern-pruned networks has the
library do, as it does it - layers encoded once, then called through ``binding.Layer`` /
``binding.Stack`` on tensors that live on the GPU, in the launch configuration the library
chooses by itself (no autotuner run, no table of tuned configurations).

A case is a dict of plain values:

``kind``   "layer"  pattern- and connectivity-pruned 3x3 layer, fp32, bias + ReLU
           "f16"    the same layer on binary16 storage
           "dense"  unpruned 3x3 layer, fp32 (the first layer of a pruned network)
           "dw"     depthwise pattern-pruned layer, fp32
           "dw_f16" depthwise on binary16 storage
           "stack"  VGG-16-shaped chain of the 13 layers with its five fused poolings
other keys  ``n`` images; ``h`` x ``w`` input; ``c_in`` / ``c_out`` channels; ``stride``; ``pad``;
            ``keep`` share of kernels that connectivity pruning leaves (1/3.6 in the paper's
            networks); ``patterns`` size of the pattern library; ``pool`` fused 2x2 max pooling;
            ``width`` (stack) divides the VGG-16 channel counts
"""

import math

import torch

from paper_2001_00138_amd import binding as B
from paper_2001_00138_amd import workloads as wl

PAPER_KEEP = 1 / 3.6


def _conv(name, kind, n, c_in, c_out, h, w, stride=1, pad=1, keep=PAPER_KEEP, patterns=8, pool=False):
    case = {"kind": kind, "n": n, "c_in": c_in, "c_out": c_out, "h": h, "w": w, "stride": stride, "pad": pad,
            "keep": keep, "patterns": patterns, "pool": pool}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: one 16-channel layer on one 32x32 image, where launch cost is everything
        _conv("small_layer", "layer", 1, 16, 16, 32, 32, keep=0.5),
        # one camera frame through all CONV layers of a VGG-16-shaped network: the paper's headline latency
        {"name": "stack_one_image", "kind": "stack", "n": 1, "h": 224, "w": 224, "width": 1},
        # the same network as a throughput service runs it, 64 images at a time: the largest case
        {"name": "stack_batch", "kind": "stack", "n": 64, "h": 224, "w": 224, "width": 1},
        # an ordinary layer in the middle of such a network, called by itself
        _conv("layer_batch", "layer", 64, 256, 256, 56, 56),
        # sizes that fit nothing: channel counts, rows and columns that are no multiples of anything
        _conv("layer_ragged", "layer", 6, 100, 75, 45, 61),
        # the last stage of a ResNet-50-shaped network: many channels on 7x7 planes
        _conv("layer_small_planes", "layer", 64, 512, 512, 7, 7),
        # the downsampling layer of such a network
        _conv("layer_stride2", "layer", 64, 128, 128, 56, 56, stride=2),
        # the first layer, which pruning leaves alone: three channels in, large planes out
        _conv("dense_first_layer", "dense", 64, 3, 64, 224, 224, keep=1.0),
        # MobileNet-V2-shaped depthwise layers: a large fp32 one, and small odd planes on binary16
        _conv("depthwise", "dw", 64, 144, 144, 56, 56, keep=1.0),
        _conv("depthwise_f16_small_planes", "dw_f16", 64, 960, 960, 7, 7, keep=1.0),
        # weights and activations kept in half precision, as the paper's GPU runs keep them: a
        # batch, and one image
        _conv("f16_batch", "f16", 64, 128, 128, 56, 56),
        _conv("f16_one_image", "f16", 1, 256, 256, 28, 28),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size of [lo, hi]: as often a multiple of 8 as not."""
    v = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        v = max(lo, (v + 4) // 8 * 8)
    return min(v, hi)


def draw(rng):
    kind = rng.choices(["layer", "f16", "dense", "dw", "dw_f16", "stack"], [8, 4, 1, 3, 2, 2])[0]
    if kind == "stack":
        side = rng.choice([64, 96, 128, 160, 192, 224])
        return {"kind": "stack", "n": _log_int(rng, 1, 32), "h": side, "w": side, "width": rng.choice([1, 2, 4])}
    stride = rng.choice([1, 1, 1, 2])
    pad = rng.choice([1, 1, 1, 1, 0])
    n = _log_int(rng, 1, 64)
    h = _log_int(rng, 7, 224)
    w = h if rng.random() < 0.5 else min(224, max(7, int(h * rng.uniform(0.6, 1.6))))
    if kind in ("dw", "dw_f16"):
        c = _size(rng, 16, 960)
        n = max(1, min(n, 100_000_000 // (c * h * w)))
        return _conv(None, kind, n, c, c, h, w, stride, pad, keep=1.0)
    if kind == "dense":
        c_in, c_out = rng.choice([1, 3, 4]), _size(rng, 16, 96)
        n = max(1, min(n, 150_000_000 // (c_out * h * w)))
        return _conv(None, kind, n, c_in, c_out, h, w, stride, pad, keep=1.0)
    c_in, c_out = _size(rng, 16, 512), _size(rng, 16, 512)
    keep = rng.choice([PAPER_KEEP, PAPER_KEEP, PAPER_KEEP, 0.5, 1.0])
    n = max(1, min(n, 100_000_000 // (max(c_in, c_out) * h * w), int(4e10 // (8 * keep * c_in * c_out * h * w))))
    pool = kind == "layer" and stride == 1 and h >= 8 and w >= 8 and rng.random() < 0.2
    return _conv(None, kind, n, c_in, c_out, h, w, stride, pad, keep, rng.choice([6, 8, 8, 8, 12]), pool)


# ---------------------------------------------------------------------------
# shapes
# ---------------------------------------------------------------------------

_VGG = [(64, False), (64, True), (128, False), (128, True), (256, False), (256, False), (256, True),
        (512, False), (512, False), (512, True), (512, False), (512, False), (512, True)]


def _stack_layers(case):
    """(c_in, c_out, h, w, pool) of every layer; the first one is not pruned."""
    c_in, h, w, out = 3, case["h"], case["w"], []
    for c, pool in _VGG:
        c_out = c // case["width"]
        out.append((c_in, c_out, h, w, pool))
        if pool:
            h, w = h // 2, w // 2
        c_in = c_out
    return out


def _out_hw(case):
    return tuple((case[k] + 2 * case["pad"] - 3) // case["stride"] + 1 for k in ("h", "w"))


def _kept(c_in, c_out, keep):
    return int(round(c_in * c_out * keep))


# ---------------------------------------------------------------------------
# what the program has in hand before the call
# ---------------------------------------------------------------------------

def _encode(gen, c_in, c_out, keep=PAPER_KEEP, patterns=8, dense=False, depthwise=False, stride=1, pad=1):
    """A layer with He-scale weights over the taps that pruning leaves, and its bias on the GPU."""
    kpf = 1 if depthwise else c_in
    kept = c_out * kpf if dense or depthwise else _kept(c_in, c_out, keep)
    fan_in = (9 if dense else 4) * kept / c_out
    weights = torch.randn((c_out, kpf, 3, 3), generator=gen) * math.sqrt(2 / fan_in)
    ids = torch.randint(0, patterns, (c_out, kpf), generator=gen, dtype=torch.uint8)
    mask = torch.zeros(c_out * kpf, dtype=torch.uint8)
    mask[torch.randperm(c_out * kpf, generator=gen)[:kept]] = 1
    layer = B.Layer(weights.numpy(), ids.numpy(), mask.reshape(c_out, kpf).numpy(),
                    wl.pattern_library(wl.PATTERN_SEED, patterns), stride=stride, pad=pad, depthwise=depthwise,
                    dense=dense)
    bias = (torch.randn(c_out, generator=gen) * 0.01).cuda()
    return layer, bias


def prepare(case, seed):
    gen = torch.Generator().manual_seed(seed)
    dev = torch.Generator(device="cuda").manual_seed(seed)
    kind, n, h, w = case["kind"], case["n"], case["h"], case["w"]
    if kind == "stack":
        layers = []
        for i, (c_in, c_out, _, _, pool) in enumerate(_stack_layers(case)):
            layer, bias = _encode(gen, c_in, c_out, dense=i == 0)
            layers.append((layer, bias, True, pool))
        stack = B.Stack(layers, n, h, w)
        x = torch.randn((n, 3, h, w), generator=dev, device="cuda")
        return {"kind": kind, "stack": stack, "x": x, "out": torch.empty(stack.output_shape(), device="cuda")}
    layer, bias = _encode(gen, case["c_in"], case["c_out"], case["keep"], case["patterns"], kind == "dense",
                          kind in ("dw", "dw_f16"), case["stride"], case["pad"])
    x = torch.randn((n, case["c_in"], h, w), generator=dev, device="cuda")
    if kind != "dense":
        x.clamp_(min=0)                      # what the ReLU of the layer before leaves
    shape = layer.output_shape(n, h, w)
    if case["pool"]:
        shape = (shape[0], shape[1], shape[2] // 2, shape[3] // 2)
    half = kind in ("f16", "dw_f16")
    if half:
        x = x.half()
    need = 0 if half else layer.workspace_floats(n, h, w)
    return {"kind": kind, "layer": layer, "bias": bias, "x": x, "pool": case["pool"],
            "out": torch.empty(shape, dtype=x.dtype, device="cuda"),
            "workspace": torch.empty(need, device="cuda") if need else None}


def run(state):
    if state["kind"] == "stack":
        return state["stack"].run(state["x"], state["out"])
    layer, x, bias, out = state["layer"], state["x"], state["bias"], state["out"]
    if state["kind"] in ("f16", "dw_f16"):
        return layer.conv2d_f16(x, bias, out, relu=True)
    return layer.conv2d_ws(x, bias, out, workspace=state["workspace"], relu=True, pool=state["pool"])


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how close two correct results are
# ---------------------------------------------------------------------------

def work(case):
    """Input once, output once, compressed weights (four values and a 2-byte index per kept
    kernel) and bias; one multiply-add per kept weight and output pixel."""
    n = case["n"]
    if case["kind"] == "stack":
        flops = weights = 0
        layers = _stack_layers(case)
        for i, (c_in, c_out, h, w, pool) in enumerate(layers):
            kernels, taps = (c_in * c_out, 9) if i == 0 else (_kept(c_in, c_out, PAPER_KEEP), 4)
            flops += 2 * taps * kernels * h * w * n
            weights += kernels * (36 if i == 0 else 18) + 4 * c_out
        c_out, h, w = layers[-1][1], layers[-1][2] // 2, layers[-1][3] // 2
        return {"bytes": 4 * n * (3 * case["h"] * case["w"] + c_out * h * w) + weights, "flops": flops}
    kind = case["kind"]
    ho, wo = _out_hw(case)
    depthwise, dense = kind in ("dw", "dw_f16"), kind == "dense"
    kernels = (case["c_out"] if depthwise else case["c_in"] * case["c_out"] if dense
               else _kept(case["c_in"], case["c_out"], case["keep"]))
    taps, size = 9 if dense else 4, 2 if kind in ("f16", "dw_f16") else 4
    out_px = (ho // 2) * (wo // 2) if case["pool"] else ho * wo
    return {"bytes": size * n * (case["c_in"] * case["h"] * case["w"] + case["c_out"] * out_px)
            + kernels * (taps * size + (0 if dense else 2)) + 4 * case["c_out"],
            "flops": 2 * taps * kernels * ho * wo * n}


def tolerance(case):
    """Four times what the path differs from the same layers in 64 bits (binary16: from their
    64-bit result rounded once, where a sum near a rounding boundary may fall on either side)."""
    if case["kind"] in ("f16", "dw_f16"):
        return {"rel": 4e-5}                 # seen: up to 0.9e-5
    # seen: 0.8e-6 after the thirteen layers, up to 0.4e-6 after one
    return {"rel": 3e-6} if case["kind"] == "stack" else {"rel": 1.6e-6}

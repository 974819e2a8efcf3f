"""What this library is used for, as cases to time: single layers of convolutional networks (fp32 and int8), classifier
layers, and residual blocks run as one sequence, through the package's public entry points.

A case is a dict of plain values.  `op` names the call:

  conv    one convolution.  `post` is the element-wise chain behind it: "none", "relu", "add" (a shortcut tensor is
          added, then Relu) or "clip" (clip to [0, 6], the activation of many depthwise-separable networks, through the
          general op-list call).  `packed` (fp32): the filter's planes were made when the network was loaded.
  fc      one FullyConnected layer of m rows, `packed` as above.
  block   a residual bottleneck block (1x1 reduce to `mid` channels, 3x3, 1x1 expand + shortcut + Relu) as one
          sequence call out of one arena.  int8: an integer island with its borders, so the input is quantized first
          and the result dequantized last.

Values: activations of unit variance and filters of variance 1 / fan_in; int8 tensors are codes of such values.  The
sizes are those of 224 x 224 classification networks (the two networks whose layers bench.py times, and depthwise
ones), plus the odd maps, channel counts and batches that other networks and crops bring."""
import math
import random

import torch

import paper_1805_00907_amd as glowmi

DEV = "cuda:0"
MAX_FLOPS = 5.93e10           # the largest listed fp32 layer
MAX_BYTES = 2.4e8


def _conv(name, dtype, n, h, w, c, k, r, stride=1, depthwise=False, post="relu", packed=False):
    return {"name": name, "op": "conv", "dtype": dtype, "n": n, "h": h, "w": w, "c": c, "k": k, "r": r,
            "stride": stride, "depthwise": depthwise, "post": post, "packed": packed}


def _fc(name, dtype, m, k, n, post="relu", packed=False):
    return {"name": name, "op": "fc", "dtype": dtype, "m": m, "k": k, "n": n, "post": post, "packed": packed}


def _block(name, dtype, n, h, w, c, mid):
    return {"name": name, "op": "block", "dtype": dtype, "n": n, "h": h, "w": w, "c": c, "mid": mid}


def listed():
    return [
        # the classifier at batch 1: one image being answered, the smallest call a program makes
        _fc("fc_f32_1x2048x1000", "f32", 1, 2048, 1000, post="none"),
        # a late-stage 3x3 at batch 1: a deep reduction on few pixels, what single-image serving consists of
        _conv("conv_f32_3x3_c256_14_b1", "f32", 1, 14, 14, 256, 256, 3, packed=True),
        # the end of a first-stage block at batch 32: contraction, shortcut and Relu in one pass; moves the most bytes
        _conv("conv_f32_1x1_c64_k256_56_add_b32", "f32", 32, 56, 56, 64, 256, 1, post="add"),
        # the downsampling 3x3 between two stages
        _conv("conv_f32_3x3s2_c128_56_b16", "f32", 16, 56, 56, 128, 128, 3, stride=2, packed=True),
        # a deep 3x3 of a plain network at batch 16 with the weights cut inside the call: the most operations
        _conv("conv_f32_3x3_c512_28_b16", "f32", 16, 28, 28, 512, 512, 3),
        # the first layer of a residual network on a small batch
        _conv("conv_f32_7x7s2_c3_224_b8", "f32", 8, 224, 224, 3, 64, 7, stride=2),
        # a depthwise layer and its clipped activation at batch 32
        _conv("conv_f32_dw3x3_c128_56_clip_b32", "f32", 32, 56, 56, 128, 128, 3, depthwise=True, post="clip"),
        # a wide hidden layer, batched, weights prepared at load time
        _fc("fc_f32_256x4096x4096", "f32", 256, 4096, 4096, packed=True),
        # a whole residual block in fp32 at batch 8
        _block("block_f32_28_c512_b8", "f32", 8, 28, 28, 512, 128),
        # int8 3x3 with channel counts and a map that fit no tile, an odd batch
        _conv("conv_i8_3x3_c72_k120_33x45_b5", "i8", 5, 33, 45, 72, 120, 3),
        # a quantized first-stage block with its borders at batch 32
        _block("block_i8_56_c256_b32", "i8", 32, 56, 56, 256, 64),
        # the largest int8 contraction
        _fc("fc_i8_1024x9216x4096", "i8", 1024, 9216, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Mostly multiples of 8, as networks are made; one in ten any number."""
    c = _log_int(rng, lo, hi)
    return c if rng.random() < 0.1 else max(8, (c + 4) // 8 * 8)


def _map(rng, lo, hi):
    h = _log_int(rng, lo, hi)
    return h, (h if rng.random() < 0.6 else max(lo, int(round(h * rng.uniform(0.6, 1.6)))))


def _drawn(rng):
    dtype = rng.choice(["f32", "i8"])
    kind = rng.choices(["conv3", "conv1", "fc", "block", "depthwise", "first"], [30, 22, 20, 12, 10, 6])[0]
    packed = dtype == "f32" and rng.random() < 0.5
    n = _log_int(rng, 1, 32)
    if kind == "fc":
        return _fc("", dtype, _log_int(rng, 1, 1024), _channels(rng, 256, 9216), _channels(rng, 64, 4608),
                   post=rng.choice(["relu", "none"]), packed=packed)
    if kind == "block":
        h, w = _map(rng, 7, 64)
        mid = _log_int(rng, 4, 64) * 8
        return _block("", dtype, n, h, w, 4 * mid, mid)
    if kind == "depthwise":
        h, w = _map(rng, 7, 112)
        c = _channels(rng, 16, 1024)
        return _conv("", dtype, n, h, w, c, c, 3, stride=rng.choice([1, 1, 2]), depthwise=True,
                     post=rng.choice(["relu", "clip"]))
    if kind == "first":
        h, w = _map(rng, 96, 320)
        r, stride = rng.choice([(7, 2), (3, 1), (3, 2)])
        return _conv("", dtype, n, h, w, 3, _log_int(rng, 4, 12) * 8, r, stride=stride)
    r = 3 if kind == "conv3" else 1
    h, w = _map(rng, 7, 112)
    return _conv("", dtype, n, h, w, _channels(rng, 16, 768), _channels(rng, 16, 1024), r,
                 stride=rng.choice([1, 1, 1, 2]), post=rng.choices(["relu", "none", "add", "clip"], [6, 1, 2, 1])[0],
                 packed=packed)


def draw(rng):
    while True:
        case = _drawn(rng)
        if case.get("post") in ("add", "clip"):
            case["packed"] = case["packed"] and case["post"] == "add"     # the op-list call takes no planes
        del case["name"]
        need = work(case)
        if need["flops"] <= MAX_FLOPS and need["bytes"] <= MAX_BYTES:
            return case


# ---- the layers of a case ------------------------------------------------------------------------------

def _desc(n, h, w, c, k, r, stride=1, depthwise=False):
    pad = r // 2
    return glowmi.ConvDesc(n, h, w, c, k, r, r, stride, stride, pad, pad, pad, pad, c if depthwise else 1)


def _convs(case):
    """(descriptor fields, has a shortcut) of the convolutions of a "conv" or "block" case."""
    n, h, w = case["n"], case["h"], case["w"]
    if case["op"] == "conv":
        return [((n, h, w, case["c"], case["k"], case["r"], case["stride"], case["depthwise"]), case["post"] == "add")]
    c, mid = case["c"], case["mid"]
    return [((n, h, w, c, mid, 1), False), ((n, h, w, mid, mid, 3), False), ((n, h, w, mid, c, 1), True)]


def _out_hw(h, w, r, stride=1):
    pad = r // 2
    return (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1


def work(case):
    """Every input, filter and output once; the tensors between the layers of a block are its own business."""
    elem = 4 if case["dtype"] == "f32" else 1
    if case["op"] == "fc":
        m, k, n = case["m"], case["k"], case["n"]
        return {"bytes": (m * k + k * n + m * n) * elem + 4 * n, "flops": 2 * m * k * n}
    flops = weights = 0
    for (n, h, w, c, k, r, *rest), _ in _convs(case):
        stride, depthwise = rest if rest else (1, False)
        oh, ow = _out_hw(h, w, r, stride)
        depth = r * r * (1 if depthwise else c)
        flops += 2 * n * oh * ow * k * depth
        weights += k * depth * elem + 4 * k
        last = n * oh * ow * k
    first = case["n"] * case["h"] * case["w"] * case["c"]
    if case["op"] == "block":
        return {"bytes": (first + last) * 4 + weights, "flops": flops}       # fp32 on both sides in either form
    return {"bytes": (first + last * (2 if case["post"] == "add" else 1)) * elem + weights, "flops": flops}


def tolerance(case):
    # int8 layers are whole numbers; a block's dequantized codes differ only if a code does
    return "exact" if case["dtype"] == "i8" else {"rel": 1e-5}


# ---- inputs --------------------------------------------------------------------------------------------

class _Values:
    """Seeded tensors on the GPU and seeded quantization parameters."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)
        self.rng = random.Random(seed)

    def normal(self, shape, std=1.0):
        return torch.randn(shape, generator=self.gen, device=DEV).mul_(std)

    def codes(self, shape, mean, std):
        return self.normal(shape, std).add_(mean).round_().clamp_(-128, 127).to(torch.int8)

    def activation_q(self):
        return glowmi.QParam(self.rng.uniform(0.02, 0.05), self.rng.randint(-20, 20))

    def filter_q(self, fan_in):
        return glowmi.QParam(1.0 / (30.0 * math.sqrt(fan_in)), 0)            # codes with a deviation of 30

    def bias_q(self, k, fan_in, xq, wq):
        return self.normal((k,), 1.0 / math.sqrt(fan_in) / (xq.scale * wq.scale)).round_().to(torch.int32)


def _buffer(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None


def _prepare_fc(case, v):
    m, k, n = case["m"], case["k"], case["n"]
    s = {"act": glowmi.ACT_RELU if case["post"] == "relu" else glowmi.ACT_NONE, "mkn": (m, k, n)}
    if case["dtype"] == "i8":
        s["xq"], s["wq"], s["yq"] = v.activation_q(), v.filter_q(k), v.activation_q()
        s["x"] = v.codes((m, k), s["xq"].offset, 1.0 / s["xq"].scale)
        s["w"] = v.codes((k, n), 0, 30.0)
        s["b"] = v.bias_q(n, k, s["xq"], s["wq"])
        s["y"] = torch.empty((m, n), dtype=torch.int8, device=DEV)
        s["ws"] = _buffer(glowmi.qfc_workspace_bytes(m, k, n))
        return s
    s["x"], s["w"], s["b"] = v.normal((m, k)), v.normal((k, n), k ** -0.5), v.normal((n,), k ** -0.5)
    s["y"] = torch.empty((m, n), device=DEV)
    s["planes"] = None
    planes = glowmi.fc_filter_planes_bytes(k, n) if case["packed"] else 0
    if planes:
        s["planes"] = _buffer(planes)
        glowmi.fc_pack_filter(s["w"], k, n, s["planes"])
        s["ws"] = _buffer(glowmi.fc_packed_workspace_bytes(m, k, n))
    else:
        s["ws"] = _buffer(glowmi.fc_workspace_bytes(m, k, n))
    return s


def _prepare_conv(case, v):
    fields, shortcut = _convs(case)[0]
    d = _desc(*fields)
    oh, ow = glowmi.conv_out_shape(d)
    cg = d.c // d.groups
    fan_in = d.r * d.s * cg
    xs, ws, ys = (d.n, d.h, d.w, d.c), (d.k, d.r, d.s, cg), (d.n, oh, ow, d.k)
    s = {"desc": d, "act": glowmi.ACT_NONE if case["post"] == "none" else glowmi.ACT_RELU,
         "ops": [("clip", 0.0, 6.0)] if case["post"] == "clip" else None, "add": None}
    if case["dtype"] == "i8":
        s["xq"], s["wq"], s["yq"] = v.activation_q(), v.filter_q(fan_in), v.activation_q()
        s["x"], s["w"] = v.codes(xs, s["xq"].offset, 1.0 / s["xq"].scale), v.codes(ws, 0, 30.0)
        s["b"] = v.bias_q(d.k, fan_in, s["xq"], s["wq"])
        s["y"] = torch.empty(ys, dtype=torch.int8, device=DEV)
        if shortcut:
            s["add_q"] = v.activation_q()
            s["add"] = v.codes(ys, s["add_q"].offset, 1.0 / s["add_q"].scale)
        s["ws"] = _buffer(glowmi.qconv2d_chainv_workspace_bytes(d, s["ops"]) if s["ops"]
                          else glowmi.qconv2d_workspace_bytes(d))
        return s
    s["x"], s["w"] = v.normal(xs), v.normal(ws, fan_in ** -0.5)
    s["b"] = v.normal((d.k,), fan_in ** -0.5)
    s["y"] = torch.empty(ys, device=DEV)
    s["add"] = v.normal(ys) if shortcut else None
    s["planes"] = None
    planes = glowmi.conv2d_filter_planes_bytes(d) if case["packed"] else 0
    if planes:
        s["planes"] = _buffer(planes)
        glowmi.conv2d_pack_filter(s["w"], d, s["planes"])
        s["ws"] = _buffer(glowmi.conv2d_packed_workspace_bytes(d))
    elif s["ops"]:
        s["ws"] = _buffer(glowmi.conv2d_chainv_workspace_bytes(d, s["ops"]))
    else:
        s["ws"] = _buffer(glowmi.conv2d_workspace_bytes(d))
    return s


def _prepare_block(case, v):
    quantized = case["dtype"] == "i8"
    s = {"x": v.normal((case["n"], case["h"], case["w"], case["c"])), "tensors": []}
    q = s["xq"] = v.activation_q()
    layers = []
    for fields, shortcut in _convs(case):
        d = _desc(*fields)
        fan_in = d.r * d.s * d.c
        shape = (d.k, d.r, d.s, d.c)
        if quantized:
            wq, yq = v.filter_q(fan_in), v.activation_q()
            w, b = v.codes(shape, 0, 30.0), v.bias_q(d.k, fan_in, q, wq)
            layers.append((d, w, b, glowmi.ACT_RELU, shortcut, wq, yq))
            q = yq
        else:
            w, b = v.normal(shape, fan_in ** -0.5), v.normal((d.k,), fan_in ** -0.5)
            layers.append((d, w, b, glowmi.ACT_RELU, shortcut))
        s["tensors"] += [w, b]                                               # the layer list holds addresses only
    s["layers"] = glowmi.seq_layers(layers)
    s["arena"] = _buffer(glowmi.seq_arena_bytes(s["layers"], quantized))
    s["y"] = torch.empty_like(s["x"])
    if quantized:
        s["x_codes"] = torch.empty(s["x"].shape, dtype=torch.int8, device=DEV)
        s["y_codes"] = torch.empty(s["x"].shape, dtype=torch.int8, device=DEV)
        s["yq"] = q
    return s


def prepare(case, seed):
    s = {"fc": _prepare_fc, "conv": _prepare_conv, "block": _prepare_block}[case["op"]](case, _Values(seed))
    s["op"], s["quantized"] = case["op"], case["dtype"] == "i8"
    return s


def run(s):
    y = s["y"]
    if s["op"] == "block":
        if s["quantized"]:
            glowmi.quantize(s["x"], s["x_codes"], s["xq"])
            glowmi.seq_qconv2d(s["x_codes"], s["xq"], s["layers"], s["y_codes"], s["arena"])
            glowmi.dequantize(s["y_codes"], y, s["yq"])
        else:
            glowmi.seq_conv2d(s["x"], s["layers"], y, s["arena"])
    elif s["op"] == "fc":
        m, k, n = s["mkn"]
        if s["quantized"]:
            glowmi.qfc(s["x"], s["xq"], s["w"], s["wq"], s["b"], y, s["yq"], m, k, n, s["act"], s["ws"])
        elif s["planes"] is not None:
            glowmi.fc_packed(s["x"], s["w"], s["planes"], s["b"], y, m, k, n, s["act"], s["ws"])
        else:
            glowmi.fc(s["x"], s["w"], s["b"], y, m, k, n, s["act"], s["ws"])
    elif s["quantized"]:
        if s["ops"]:
            glowmi.qconv2d_chainv(s["x"], s["xq"], s["w"], s["wq"], s["b"], y, s["yq"], s["desc"], s["ops"], s["ws"])
        elif s["add"] is not None:
            glowmi.qconv2d_chain(s["x"], s["xq"], s["w"], s["wq"], s["b"], y, s["yq"], s["desc"], s["add"],
                                 s["add_q"], s["act"], s["ws"])
        else:
            glowmi.qconv2d(s["x"], s["xq"], s["w"], s["wq"], s["b"], y, s["yq"], s["desc"], s["act"], s["ws"])
    elif s["ops"]:
        glowmi.conv2d_chainv(s["x"], s["w"], s["b"], y, s["desc"], s["ops"], s["ws"])
    elif s["planes"] is not None:
        glowmi.conv2d_packed(s["x"], s["w"], s["planes"], s["b"], y, s["desc"], s["add"], s["act"], s["ws"])
    elif s["add"] is not None:
        glowmi.conv2d_chain(s["x"], s["w"], s["b"], y, s["desc"], s["add"], s["act"], s["ws"])
    else:
        glowmi.conv2d(s["x"], s["w"], s["b"], y, s["desc"], s["act"], s["ws"])
    return y

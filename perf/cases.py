"""Performance cases of the convolution library: what a program that runs inference on one GPU has it do.

A case is one layer (`kind` "layer") or the five-layer stack with its pools (`kind` "stack").  A layer case names the
descriptor, the storage type, the tensor formats and the way the layer is called:

* `call` "plain": conv_fwd, the entry point without a workspace;
* `call` "workspace": conv_fwd_ws with a workspace of conv_workspace_bytes();
* `tuned`: whether the program ran conv_autotune for the descriptor when it started (once per descriptor and process, as
  a program that serves one network does) or relies on the library's own selection.

`format` is "nchw" ([N][C][H][W] tensors, [K][C][R][S] filters), "nhwc" (channel-innermost tensors, filters repacked once
to [K][R][S][C]) or "nhwc_packed" (channel-innermost tensors, filters converted once to the order the matrix
instructions consume).  Inputs are half-normal like activations behind a ReLU, or uniform in [-128, 128] for the
three-channel first layers; filters are He-scaled, biases uniform in [-0.1, 0.1].
"""
import math

import torch

from paper_1611_06945_amd import binding as B
from paper_1611_06945_amd import workloads as wl
from paper_1611_06945_amd.stack import ConvStack

_CODE = {"f32": B.CONV_F32, "f16": B.CONV_F16, "bf16": B.CONV_BF16}
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

# What the largest listed case multiplies and moves; drawn cases stay below it (the fp32 ones by a factor of two, since
# not every fp32 shape has a kernel as fast as that case's).
_MOST_FLOPS = {"f32": 2.2e10, "f16": 3.0e10, "bf16": 3.0e10}
_MOST_BYTES = 2.0e8


def _layer(N, C, H, W, K, R, stride, pad, dtype, format="nchw", call="workspace", tuned=True, relu=True, name=None):
    c = {"kind": "layer", "N": N, "C": C, "H": H, "W": W, "K": K, "R": R, "S": R, "stride": stride, "pad": pad,
         "dtype": dtype, "format": format, "call": call, "tuned": tuned, "relu": relu}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # benchmark configuration 1: the smallest call anybody makes; launch and host cost
        _layer(1, 3, 32, 32, 16, 3, 1, 1, "f32", call="plain", tuned=False, name="toy3x3_n1_f32"),
        # benchmark configuration 2: a pointwise layer of a GoogLeNet at the batch of the paper's tables
        _layer(5, 256, 28, 28, 128, 1, 1, 0, "f32", name="pointwise_n5_f32"),
        # benchmark configuration 3: an AlexNet first layer in the paper's arithmetic
        _layer(20, 3, 227, 227, 96, 11, 4, 0, "f32", name="first11x11_n20_f32"),
        # benchmark configuration 4: the mid-network layer for one image (latency of an interactive request) in fp16
        _layer(1, 256, 13, 13, 384, 3, 1, 1, "f16", name="mid3x3_n1_f16"),
        # ... and at batch 20 in fp32: the headline workload of bench.py
        _layer(20, 256, 13, 13, 384, 3, 1, 1, "f32", name="mid3x3_n20_f32"),
        # a fully-connected layer written as a convolution (Appendix A), at the batch of the stack: weights streamed once
        _layer(20, 256, 6, 6, 4096, 6, 1, 0, "f16", name="fc6x6_n20_f16"),
        # channel counts and image sizes that fit no tile, by the library's own selection and without an activation
        _layer(8, 100, 33, 35, 130, 3, 1, 1, "f16", tuned=False, relu=False, name="odd3x3_n8_f16"),
        # a pointwise layer at serving batch through the entry point that needs nothing but the tensors
        _layer(64, 256, 28, 28, 128, 1, 1, 0, "f16", call="plain", tuned=False, name="pointwise_n64_f16"),
        # a downsampling layer between two stages of a network kept channel-innermost throughout
        _layer(32, 128, 56, 56, 128, 3, 2, 1, "bf16", format="nhwc", name="down3x3_n32_bf16_nhwc"),
        # the largest 3x3 layer of Appendix A at throughput batch, bf16 storage on the plain formats
        _layer(64, 64, 56, 56, 192, 3, 1, 1, "bf16", name="wide3x3_n64_bf16"),
        # ... and in fp32: the largest case
        _layer(64, 64, 56, 56, 192, 3, 1, 1, "f32", name="wide3x3_n64_f32"),
        # benchmark configuration 5: five layers and two pools, formats chosen by the planner
        {"kind": "stack", "N": 20, "dtype": "f16", "name": "stack5_n20_f16"},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Mostly what networks use (multiples of 16 or 8), sometimes any number."""
    c = _logint(rng, lo, hi)
    step = rng.choice((16, 16, 16, 8, 1))
    return max(lo, (c + step // 2) // step * step)


def draw(rng):
    if rng.random() < 0.06:
        return {"kind": "stack", "N": rng.randint(1, 20), "dtype": rng.choice(("f16", "bf16"))}
    dtype = rng.choice(("f32", "f16", "bf16"))
    kind = rng.choice(("3x3", "3x3", "3x3", "1x1", "1x1", "5x5", "first", "down", "fc"))
    N = _logint(rng, 1, 64)
    if kind == "first":
        R, stride, pad, K = rng.choice(((11, 4, 0, 96), (7, 2, 3, 64), (3, 1, 1, 64), (3, 2, 1, 32)))
        H = rng.randint(96, 256)
        C, W, K = 3, max(96, H + rng.choice((0, 0, -5, 8))), K + rng.choice((0, 0, 0, -7))
    elif kind == "fc":
        R = rng.choice((1, 1, 6, 7))
        C = _channels(rng, 1024, 4096) if R == 1 else _channels(rng, 128, 512)
        H = W = R
        K, stride, pad = rng.choice((1000, 2048, 4096)), 1, 0
    else:
        R, stride, pad = {"3x3": (3, 1, 1), "1x1": (1, 1, 0), "5x5": (5, 1, 2), "down": (3, 2, 1)}[kind]
        H = _logint(rng, 6, 64)
        W = max(6, H + rng.choice((0, 0, 0, 3, -2)))
        C, K = _channels(rng, 16, 512), _channels(rng, 16, 512)
    fmt = "nchw"
    if dtype != "f32" and C % 8 == 0 and K % 8 == 0 and rng.random() < 0.4:
        fmt = "nhwc"
        if stride == 1 and R in (3, 5) and C % 16 == 0 and W <= 56 and rng.random() < 0.5:
            fmt = "nhwc_packed"
    call = rng.choice(("workspace", "workspace", "plain"))
    case = _layer(N, C, H, W, K, R, stride, pad, dtype, fmt, call, rng.random() < 0.5, rng.random() < 0.85)
    while case["N"] > 1:
        w = work(case)
        if w["flops"] <= _MOST_FLOPS[dtype] and w["bytes"] <= _MOST_BYTES:
            break
        case["N"] -= max(1, case["N"] // 8)
    return case


def _shape(case):
    return wl.ConvShape(*(case[k] for k in ("N", "C", "H", "W", "K", "R", "S", "stride", "pad")))


def _stack_shapes(case):
    return [w.shape for w in wl.config5_layers(case["N"], _CODE[case["dtype"]])]


def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _input(shape, dtype, g):
    if shape.C == 3:
        x = torch.rand(shape.in_shape(), generator=g, device="cuda").mul_(256.0).sub_(128.0)
    else:
        x = torch.randn(shape.in_shape(), generator=g, device="cuda").abs_()
    return x.to(_TORCH[dtype])


def _weights(shape, dtype, g):
    f = torch.randn(shape.filt_shape(), generator=g, device="cuda").mul_(wl.he_sigma(shape)).to(_TORCH[dtype])
    b = torch.rand(shape.K, generator=g, device="cuda").mul_(0.2).sub_(0.1)
    return f, b


_tuned = set()   # descriptors this process has autotuned
_stacks = {}     # (batch, storage type) -> the network this process serves: its tuned stack and its weights


def _prepare_stack(case, seed):
    key = (case["N"], case["dtype"])
    shapes = _stack_shapes(case)
    x = _input(shapes[0], case["dtype"], _rng(seed))
    if key not in _stacks:
        g = _rng(1)
        weights = [_weights(s, case["dtype"], g) for s in shapes]
        filts, biases = [w[0] for w in weights], [w[1] for w in weights]
        stack = ConvStack(shapes, _CODE[case["dtype"]], pool_after=wl.STACK_POOL_AFTER, formats="auto")
        stack.autotune(x, filts, biases)
        _stacks[key] = (stack, filts, biases)
    stack, filts, biases = _stacks[key]
    return {"kind": "stack", "stack": stack, "x": x, "filts": filts, "biases": biases}


def prepare(case, seed):
    """The tensors of one layer (or the tuned network and one batch of images), in the formats the calls take."""
    if case["kind"] == "stack":
        return _prepare_stack(case, seed)
    s, dtype, fmt = _shape(case), case["dtype"], case["format"]
    g = _rng(seed)
    x = _input(s, dtype, g)
    f, b = _weights(s, dtype, g)
    nhwc = fmt != "nchw"
    d = B.desc_of(s, _CODE[dtype], relu=case["relu"], in_nhwc=nhwc, out_nhwc=nhwc, filt_krsc=fmt == "nhwc",
                  filt_packed=fmt == "nhwc_packed")
    if nhwc:
        x = x.permute(0, 2, 3, 1).contiguous()
        if fmt == "nhwc":
            f = f.permute(0, 2, 3, 1).contiguous()
        else:
            packed = torch.empty(B.conv_transformed_filter_bytes(d), dtype=torch.uint8, device="cuda")
            B.conv_transform_filters(d, f, packed)
            f = packed
    n, k, oh, ow = s.out_shape()
    out = torch.empty((n, oh, ow, k) if nhwc else (n, k, oh, ow), dtype=_TORCH[dtype], device="cuda")
    ws = None
    if case["call"] == "workspace":
        ws = torch.empty(max(256, B.conv_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
    if case["tuned"] and bytes(d) not in _tuned:
        B.conv_autotune(d, x, f, b, out, ws, 0 if ws is None else ws.numel())
        _tuned.add(bytes(d))
    return {"kind": "layer", "desc": d, "x": x, "filt": f, "bias": b, "out": out, "ws": ws,
            "ws_bytes": 0 if ws is None else ws.numel()}


def run(state):
    if state["kind"] == "stack":
        return state["stack"].run(state["x"], state["filts"], state["biases"])
    if state["ws"] is None:
        B.conv_fwd(state["desc"], state["x"], state["filt"], state["bias"], state["out"])
    else:
        B.conv_fwd_ws(state["desc"], state["x"], state["filt"], state["bias"], state["out"], state["ws"], state["ws_bytes"])
    return state["out"]


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "stack":
        shapes = _stack_shapes(case)
        last = shapes[-1]
        moved = math.prod(shapes[0].in_shape()) + math.prod(last.out_shape()) + sum(math.prod(s.filt_shape()) for s in shapes)
        return {"bytes": moved * e + sum(4 * s.K for s in shapes), "flops": sum(s.flops for s in shapes)}
    s = _shape(case)
    return {"bytes": s.algorithmic_bytes(_CODE[case["dtype"]]), "flops": s.flops}


def tolerance(case):
    """About four times the largest error seen against the same layer in 64 bits: 3.9e-7 for sums in fp32, 2.1e-4 / 1.7e-3
    for the one rounding of the result to fp16 / bf16, 4.7e-4 for the five such roundings of the fp16 stack (in bf16 eight
    times that)."""
    if case["kind"] == "stack":
        return {"rel": 2e-3} if case["dtype"] == "f16" else {"rel": 1.5e-2}
    return {"f32": {"rel": 2e-6}, "f16": {"rel": 8e-4}, "bf16": {"rel": 6.6e-3}}[case["dtype"]]

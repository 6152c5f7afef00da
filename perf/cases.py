"""The work that users of this library have it do, as measurable cases over the public entry points.

Four kinds of case, each with the ranges that `draw` samples:

* ``matmul``  one matrix product: the classifier of a batch-1 network (one row), a few rows against a large weight matrix, ordinary and
              large square products, reductions and row counts that are no multiple of anything; all five operand types.
* ``conv``    one convolution call: weights packed beforehand (``wpacked``, the per-layer call of an inference loop, raw sums or
              requantised to int8) or both operands plain (``plain``), 2-D and 3-D, odd channel counts and image sizes, strides 1 and 2.
* ``layers``  the 53 convolutions of a ResNet-50-shaped network, one call per layer on buffers of its own: int8 at batch 1 is the
              benchmark's headline, fp16 at batch 16 its throughput form.
* ``chain``   chained int8 inference of a ResNet-18-shaped network, image to logits.

``graph`` cases replay the calls from a captured HIP graph, as a serving loop with fixed buffers does; the others call eagerly.
"""
import math

import numpy as np
import torch

from paper_2101_08458_amd import resnet18_int8, unit
from paper_2101_08458_amd import workloads as wl

DEV = "cuda:0"

# dtype -> (public constant, operand bytes, matmul, plain conv, packed-weight conv or None, integer sums)
TYPES = {
    "i8": (unit.UNIT_I8, 1, unit.unit_matmul_i8, unit.unit_conv2d_i8, unit.unit_conv2d_wpacked_i8, True),
    "f16": (unit.UNIT_F16, 2, unit.unit_matmul_f16, unit.unit_conv2d_f16, unit.unit_conv2d_wpacked_f16, False),
    "bf16": (unit.UNIT_BF16, 2, unit.unit_matmul_bf16, unit.unit_conv2d_bf16, None, False),
    "u8i8": (unit.UNIT_U8I8, 1, unit.unit_matmul_u8i8, unit.unit_conv2d_u8i8, None, True),
    "fp8": (unit.UNIT_FP8, 1, unit.unit_matmul_fp8, unit.unit_conv2d_fp8, None, False),
}


def listed():
    return [
        # the classifier of a batch-1 network: the smallest call there is, latency only
        {"name": "fc_i8_b1", "kind": "matmul", "dtype": "i8", "m": 1, "n": 1000, "k": 2048, "pitch": 0},
        # a small batch of vectors through one large weight matrix: the weights' bytes are the work
        {"name": "rows32_bf16", "kind": "matmul", "dtype": "bf16", "m": 32, "n": 4096, "k": 4096, "pitch": 0},
        # no dimension a multiple of anything: features with their own width, row pitch not a multiple of 16 bytes
        {"name": "ragged_f16", "kind": "matmul", "dtype": "f16", "m": 1533, "n": 2001, "k": 1777, "pitch": 0},
        # ordinary fp8 product
        {"name": "gemm_fp8", "kind": "matmul", "dtype": "fp8", "m": 2048, "n": 2048, "k": 4096, "pitch": 0},
        # the benchmark's square products, the fp16 one the largest case here
        {"name": "gemm_i8_4096", "kind": "matmul", "dtype": "i8", "m": 4096, "n": 4096, "k": 4096, "pitch": 0},
        {"name": "gemm_f16_8192", "kind": "matmul", "dtype": "f16", "m": 8192, "n": 8192, "k": 8192, "pitch": 0},
        # quantised layer of a large batch: int8 image in, requantised int8 image out
        {"name": "conv_i8_b32_requant", "kind": "conv", "dtype": "i8", "call": "wpacked", "requant": True, "n": 32, "c": 256,
         "d": 1, "h": 56, "w": 56, "k": 256, "t": 1, "r": 3, "stride": 1, "pad": 1},
        # unsigned activations (after a ReLU), both operands as the framework holds them, ordinary size
        {"name": "conv_u8i8_b8", "kind": "conv", "dtype": "u8i8", "call": "plain", "requant": False, "n": 8, "c": 128,
         "d": 1, "h": 28, "w": 28, "k": 128, "t": 1, "r": 3, "stride": 1, "pad": 1},
        # one layer of the 3-D network: a ResNet-18 layer lifted to depth 8
        {"name": "conv3d_f16", "kind": "conv", "dtype": "f16", "call": "plain", "requant": False, "n": 1, "c": 128,
         "d": 4, "h": 28, "w": 28, "k": 128, "t": 3, "r": 3, "stride": 1, "pad": 1},
        # the headline: all 53 layers, batch 1, int8
        {"name": "resnet50_i8_b1", "kind": "layers", "dtype": "i8", "batch": 1, "graph": True},
        # the same layers for throughput
        {"name": "resnet50_f16_b16", "kind": "layers", "dtype": "f16", "batch": 16, "graph": False},
        # a whole quantised network, one call after another from Python
        {"name": "resnet18_i8_b8", "kind": "chain", "dtype": "i8", "batch": 8, "graph": False},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi, step):
    """Log-uniform; two in three on a multiple of `step`, the others anything (odd ones among them)."""
    v = _log(rng, lo, hi)
    return v if rng.random() < 1 / 3 else max(step, (v + step // 2) // step * step)


def draw(rng):
    while True:
        kind = rng.choices(["matmul", "conv", "layers", "chain"], [5, 5, 1, 1])[0]
        if kind == "layers":
            c = {"kind": kind, "dtype": rng.choice(["i8", "f16"]), "batch": _log(rng, 1, 16), "graph": rng.random() < 0.5}
        elif kind == "chain":
            c = {"kind": kind, "dtype": "i8", "batch": _log(rng, 1, 32), "graph": rng.random() < 0.5}
        elif kind == "matmul":
            c = {"kind": kind, "dtype": rng.choice(sorted(TYPES)), "m": _size(rng, 1, 8192, 16), "n": _size(rng, 64, 8192, 64),
                 "k": _size(rng, 64, 8192, 64), "pitch": rng.choice([0, 0, 0, 64])}
        else:
            dtype, d3 = rng.choice(sorted(TYPES)), rng.random() < 0.2
            if d3:
                dtype = rng.choice(["i8", "f16"])
            call = "wpacked" if TYPES[dtype][4] is not None and not d3 and rng.random() < 0.7 else "plain"
            r = rng.choice([1, 3, 3, 5, 7]) if not d3 else rng.choice([1, 3])
            hw = rng.choice([7, 14, 28, 56, 112]) if rng.random() < 0.6 else rng.randint(9, 75)
            cin = _size(rng, 16, 512, 32)
            if r == 7:                               # the first layer of a network reads an image
                cin, hw = rng.choice([1, 3, 3, 4]), rng.choice([64, 112, 224, 224, rng.randint(65, 231)])
            c = {"kind": kind, "dtype": dtype, "call": call, "requant": dtype == "i8" and not d3 and rng.random() < 0.5,
                 "n": _log(rng, 1, 32) if not d3 else rng.choice([1, 2]), "c": cin, "d": rng.choice([4, 8]) if d3 else 1,
                 "h": hw, "w": hw, "k": _size(rng, 32, 512, 32), "t": r if d3 else 1, "r": r,
                 "stride": rng.choice([1, 1, 2]), "pad": rng.choice([r // 2, r // 2, 0])}
        w = work(c)
        # no dearer than the largest listed case, and its tensors small enough to be held three times over with ease
        if w["flops"] <= 4e11 and w["bytes"] <= 1.2e9:
            return c


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _operand(g, dtype, shape, weights, fan_in):
    """Quantised activations and weights fill their byte ranges; the float types get N(0,1) activations and He-initialised weights."""
    if dtype == "u8i8" and not weights:
        return torch.randint(0, 256, shape, generator=g, device=DEV, dtype=torch.uint8)
    if dtype in ("i8", "u8i8"):
        lo, hi = (-128, 128) if weights else (-64, 64)
        return torch.randint(lo, hi, shape, generator=g, device=DEV, dtype=torch.int8)
    x = torch.randn(shape, generator=g, device=DEV)
    if weights:
        x *= math.sqrt(2.0 / fan_in)
    return x.to({"f16": torch.float16, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dtype])


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _out(dtype, shape):
    return torch.empty(shape, dtype=torch.int32 if TYPES[dtype][5] else torch.float32, device=DEV)


def _conv_dims(c):
    def o(size, window):
        return (size + 2 * c["pad"] - window) // c["stride"] + 1
    depth = o(c["d"], c["t"]) if c["t"] > 1 or c["d"] > 1 else 1
    return depth, o(c["h"], c["r"]), o(c["w"], c["r"])


def _layer(g, dtype, batch, sh):
    """One layer of the ResNet-50-shaped set, as an inference loop holds it: weights packed, buffers allocated."""
    ut = TYPES[dtype][0]
    d = unit.conv_desc(batch, sh.c, sh.h, sh.w, sh.k, sh.r, sh.s, sh.stride, sh.pad)
    p, q = unit.unit_conv2d_out_dims(d)
    w = _operand(g, dtype, (sh.k, sh.c, sh.r, sh.s), True, sh.c * sh.r * sh.s)
    wp = _bytes(unit.unit_packed_weights_bytes(d, ut))
    (unit.unit_pack_weights_i8 if dtype == "i8" else unit.unit_pack_weights_f16)(d, w, wp)
    return {"d": d, "x": _operand(g, dtype, (batch, sh.c, sh.h, sh.w), False, 1), "wp": wp, "y": _out(dtype, (batch, sh.k, p, q))}


def _capture(fn):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fn()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


def prepare(case, seed):
    g, c, dtype = _gen(seed), case, case["dtype"]
    ut, es = TYPES[dtype][:2]
    s = {"case": c}
    if c["kind"] == "matmul":
        m, n, k, ld = c["m"], c["n"], c["k"], c["k"] + c["pitch"]
        s["A"] = _operand(g, dtype, (m, ld), False, 1)
        s["B"] = _operand(g, dtype, (n, ld), True, k)
        s["C"] = _out(dtype, (m, n))
        s["ws"] = _bytes(unit.unit_matmul_workspace(m, n, k, ld, ld, ut))
        s["fn"], s["args"] = TYPES[dtype][2], (m, n, k, s["A"], ld, s["B"], ld, s["C"], n, s["ws"])
    elif c["kind"] == "conv":
        o, p, q = _conv_dims(c)
        fan_in = c["c"] * c["t"] * c["r"] * c["r"]
        d3 = c["d"] > 1
        dims = (c["d"], c["h"], c["w"]) if d3 else (c["h"], c["w"])
        win = (c["t"], c["r"], c["r"]) if d3 else (c["r"], c["r"])
        x = _operand(g, dtype, (c["n"], c["c"]) + dims, False, 1)
        w = _operand(g, dtype, (c["k"], c["c"]) + win, True, fan_in)
        shape = (c["n"], c["k"]) + ((o, p, q) if d3 else (p, q))
        rq = y8 = None
        if c["requant"]:
            # a calibrated layer: three standard deviations of the sums fill the byte range
            sigma = math.sqrt(fan_in) * 37.0 * 74.0
            s["scale"] = torch.full((c["k"],), 127.0 / (3.0 * sigma), device=DEV)
            s["bias"] = torch.randint(-20000, 20000, (c["k"],), generator=g, device=DEV, dtype=torch.int32)
            rq = s["rq"] = unit.make_requant(s["scale"], s["bias"], relu=True)
            y8 = torch.empty(shape, dtype=torch.int8, device=DEV)
        y = None if rq is not None else _out(dtype, shape)
        s["out"] = y if rq is None else y8
        if d3:
            d = unit.conv3d_desc(c["n"], c["c"], *dims, c["k"], *win, (c["stride"],) * 3, (c["pad"],) * 3)
            ws = _bytes(unit.unit_conv3d_workspace(d, ut))
            s["fn"], s["args"] = (unit.unit_conv3d_i8 if dtype == "i8" else unit.unit_conv3d_f16), (d, x, w, y, ws)
        else:
            d = unit.conv_desc(c["n"], c["c"], c["h"], c["w"], c["k"], c["r"], c["r"], c["stride"], c["pad"])
            if c["call"] == "wpacked":
                wp = _bytes(unit.unit_packed_weights_bytes(d, ut))
                (unit.unit_pack_weights_i8 if dtype == "i8" else unit.unit_pack_weights_f16)(d, w, wp)
                w, ws, s["fn"] = wp, _bytes(unit.unit_conv2d_wpacked_workspace(d, ut)), TYPES[dtype][4]
            else:
                ws, s["fn"] = _bytes(unit.unit_conv2d_workspace(d, ut)), TYPES[dtype][3]
            s["args"] = (d, x, w, y, rq, y8, ws) if dtype == "i8" else (d, x, w, y, ws)
    elif c["kind"] == "layers":
        shapes = wl.resnet50_convs()
        s["layers"] = [_layer(g, dtype, c["batch"], sh) for sh in shapes]
        s["fn"] = TYPES[dtype][4]
        # one scratch buffer for the whole network: the layers run one after another
        s["ws"] = _bytes(max(unit.unit_conv2d_wpacked_workspace(L["d"], ut) for L in s["layers"]))
        s["graph"] = _capture(lambda: _run_layers(s)) if c["graph"] else None
    else:
        params = resnet18_int8.random_params(np.random.Generator(np.random.PCG64(seed)))
        # scales as a calibration would leave them: every layer's activations at about 45 rms after the ReLU, whose clamp takes
        # what lies beyond two standard deviations of the sums; half of a block's input is added back to its output
        for name, sh in resnet18_int8.layer_list():
            params[name]["scale"][:] = 127.0 / (2.0 * math.sqrt(sh.c * sh.r * sh.s) * 74.0 * 45.0)
        for i in params["res_mult"]:
            params["res_mult"][i] = round(0.5 / float(params[f"b{i}.c2"]["scale"][0]))
        s["net"] = resnet18_int8.ResNet18Int8(c["batch"], params, DEV)
        s["x"] = _operand(g, "i8", (c["batch"], 3, 224, 224), False, 1)
        s["graph"] = _capture(lambda: s["net"].forward(s["x"])) if c["graph"] else None
    return s


def _run_layers(s):
    fn, ws = s["fn"], s["ws"]
    if s["case"]["dtype"] == "i8":
        for L in s["layers"]:
            fn(L["d"], L["x"], L["wp"], L["y"], None, None, ws)
    else:
        for L in s["layers"]:
            fn(L["d"], L["x"], L["wp"], L["y"], ws)


def run(state):
    kind = state["case"]["kind"]
    if kind == "matmul":
        state["fn"](*state["args"])
        return state["C"]
    if kind == "conv":
        state["fn"](*state["args"])
        return state["out"]
    if kind == "layers":
        if state["graph"] is not None:
            state["graph"].replay()
        else:
            _run_layers(state)
        return [L["y"] for L in state["layers"]]
    net = state["net"]
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        net.forward(state["x"])
    return [net.logits] + net.act_y          # logits and the eight blocks' packed activations


def work(case):
    c, es = case, TYPES[case["dtype"]][1]
    if c["kind"] == "matmul":
        m, n, k = c["m"], c["n"], c["k"]
        return {"bytes": (m + n) * k * es + m * n * 4, "flops": 2 * m * n * k}
    if c["kind"] == "conv":
        o, p, q = _conv_dims(c)
        if min(o, p, q) < 1:
            return {"bytes": float("inf"), "flops": float("inf")}
        fan_in = c["c"] * c["t"] * c["r"] * c["r"]
        outs = c["n"] * c["k"] * o * p * q
        return {"bytes": (c["n"] * c["c"] * c["d"] * c["h"] * c["w"] + c["k"] * fan_in) * es + outs * (1 if c["requant"] else 4),
                "flops": 2 * outs * fan_in}
    if c["kind"] == "layers":
        b, byts, flops = c["batch"], 0, 0
        for sh in wl.resnet50_convs():
            p, q = wl.out_hw(sh)
            byts += (b * sh.c * sh.h * sh.w + sh.k * sh.c * sh.r * sh.s) * es + b * sh.k * p * q * 4
            flops += 2 * wl.macs(sh, b)
        return {"bytes": byts, "flops": flops}
    b, byts, flops = c["batch"], c["batch"] * (3 * 224 * 224 + 1000 * 4) + 512 * 1000, 2 * c["batch"] * 512 * 1000
    for name, sh in resnet18_int8.layer_list():
        p, q = wl.out_hw(sh)
        byts += sh.k * sh.c * sh.r * sh.s + (b * sh.k * p * q if name.endswith("c2") else 0)
        flops += 2 * wl.macs(sh, b)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # integer sums are exact whatever their order, and so is the requantise rule on them
    if case["dtype"] in ("i8", "u8i8"):
        return "exact"
    # products of 16-bit floats are exact in fp32; what differs is the order of the fp32 sums (against fp64 sums: up to 4.1e-7 in
    # the 2-norm and 3.6e-6 of the largest element over the shapes above and a few more, the same for fp16 and bf16)
    if case["dtype"] != "fp8":
        return {"rel": 2e-6, "max": 1.5e-5}
    # the fp8 matrix instruction adds its products with fewer bits than fp32 holds (1.1e-5 and 1.3e-4)
    return {"rel": 4.5e-5, "max": 5e-4}


def _patches(x, win, stride, pad):
    """One image [c][d][h][w] in 64 bits -> [c * taps][output positions], taps in the order of the weights."""
    x = torch.nn.functional.pad(x, (pad[2], pad[2], pad[1], pad[1], pad[0], pad[0]))
    for i, r in enumerate(win):
        x = x.unfold(1 + i, r, stride)
    c, o = x.shape[0], x.shape[1:4]
    return x.permute(0, 4, 5, 6, 1, 2, 3).reshape(c * win[0] * win[1] * win[2], -1), tuple(o)


def _conv64(x, w, stride, pad):
    """x [n][c][d][h][w], w [k][c][t][r][s]: the sums in 64 bits (one image after another, so that the patches stay small)."""
    w2, out = w.double().reshape(w.shape[0], -1), []
    for img in x:
        cols, o = _patches(img.double(), w.shape[2:], stride, pad)
        out.append((w2 @ cols).reshape((w.shape[0],) + o))
    return torch.stack(out)


def exact(case, seed):
    """The same inputs, drawn in `prepare`'s order, and plain 64-bit sums; None where the rule after the sums is the result."""
    c, dtype, g = case, case["dtype"], _gen(seed)
    if c["kind"] == "matmul":
        m, n, k, ld = c["m"], c["n"], c["k"], c["k"] + c["pitch"]
        A, B = _operand(g, dtype, (m, ld), False, 1), _operand(g, dtype, (n, ld), True, k)
        return A[:, :k].double() @ B[:, :k].double().t()
    if c["kind"] == "conv" and not c["requant"]:
        d3, t, r, p = c["d"] > 1, c["t"], c["r"], c["pad"]
        x = _operand(g, dtype, (c["n"], c["c"], c["d"], c["h"], c["w"]), False, 1)
        w = _operand(g, dtype, (c["k"], c["c"], t, r, r), True, c["c"] * t * r * r)
        y = _conv64(x, w, c["stride"], (p if d3 else 0, p, p))
        return y if d3 else y[:, :, 0]
    if c["kind"] == "layers":
        out = []
        for sh in wl.resnet50_convs():
            w = _operand(g, dtype, (sh.k, sh.c, sh.r, sh.s), True, sh.c * sh.r * sh.s)
            x = _operand(g, dtype, (c["batch"], sh.c, sh.h, sh.w), False, 1)
            out.append(_conv64(x[:, :, None], w[:, :, None], sh.stride, (0, sh.pad, sh.pad))[:, :, 0])
        return out
    return None

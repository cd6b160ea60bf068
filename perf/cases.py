"""The calls whose speed counts: what a user of the library has it do, from one small image to
products that fill the chip, through the public entry points of `paper_2105_09377_amd`.

`listed()` are fixed sizes (the library's own workloads and ragged relatives of them), `draw()`
gives further ones of the same ranges.  A case is a dict of plain values; its "kind" names the call:

  pair_of_forms  the small convolution evaluated both ways, directly and as im2col + contraction
  conv           one convolution layer on weights packed beforehand
  block          a downsampling block: 3x3/2, 1x1/2 projection, sum, ReLU, 2x2 max pooling
  stack          the ResNet-18-shaped stack, one forward pass
  mlp            three dense layers
  dense          compute dotProd (cartProd a0 a1)
  program        the im2col listing as text: pad, windows, flatten, contraction, reshape, transpose
  reduce         compute reduceSum | reduceMax over rows
  depthwise      every channel convolved with its own filter
"""

from __future__ import annotations

import math

import torch

from paper_2105_09377_amd import binding as gs
from paper_2105_09377_amd.resnet import ResNet18Stack
from paper_2105_09377_amd.synth import RESNET18_CONVS

DEV = "cuda:0"
_ESZ = {"i8": 1, "fp8": 1, "bf16": 2, "f32": 4, "i32": 4}
_OUT = {"i8": torch.int32, "i32": torch.int32, "bf16": torch.bfloat16, "f32": torch.float32}

CONV2D_PADDED = """
(transpose
 (squeeze
  (compute dotProd
   (cartProd
    (windows (access (pad (pad activations 2 P P) 3 P P) 1) (shape C K K) (shape 1 S S))
    (access weights 1)))
  1)
 (list 0 3 1 2))
"""


def listed():
    return [
        # The smallest program: one 8x8 image of three channels; latency, launches and host work.
        dict(name="tiny_conv_i8", kind="pair_of_forms", n=1, c=3, h=8, w=8, o=4, k=3, stride=1, pad=0, dtype="i8"),
        # Inference of a small dense network: three short launches that depend on each other.
        dict(name="mlp_256", kind="mlp", batch=256, d0=784, d1=512, d2=512, d3=10),
        # The ordinary 3x3 layer of a convolutional network, in both element types.
        dict(name="conv3x3_bf16", kind="conv", n=32, c=64, h=56, w=56, o=64, k=3, stride=1, pad=1, dtype="bf16",
             residual=False, relu=False),
        dict(name="conv3x3_i8", kind="conv", n=32, c=64, h=56, w=56, o=64, k=3, stride=1, pad=1, dtype="i8",
             residual=False, relu=False),
        # Two convolutions of stride 2, their sum and a pooling.
        dict(name="downsample_block", kind="block", n=32, c=128, h=28, w=28, o=256),
        # The whole network: a batch that fills the chip, and a single image (serving).
        dict(name="resnet18_b64", kind="stack", batch=64, image=224, classes=1000),
        dict(name="resnet18_b1", kind="stack", batch=1, image=224, classes=1000),
        # The contraction by itself: the largest, and one with no extent a multiple of anything.
        dict(name="dense_8192_bf16", kind="dense", m=8192, n=8192, k=8192, dtype="bf16", out="f32"),
        dict(name="dense_ragged_fp8", kind="dense", m=2047, n=1531, k=1001, dtype="fp8", out="bf16"),
        # The rewritten listing, node by node: the explicit window gather and what follows it.
        dict(name="program_im2col", kind="program", n=32, c=64, h=56, w=56, o=64, k=3, stride=1, pad=1, dtype="bf16"),
        # Row sums and depth-wise windows: bound by memory.
        dict(name="reduce_f32", kind="reduce", rows=65536, cols=1024, dtype="f32", op="sum"),
        dict(name="depthwise_bf16", kind="depthwise", n=32, c=128, h=112, w=112, k=3, stride=1, pad=1, dtype="bf16",
             out="bf16", relu=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: most often a multiple of 16, now and then anything."""
    c = _log(rng, lo, hi)
    return max(16, c // 16 * 16) if rng.random() < 0.75 else c


def draw(rng):
    kind = rng.choice(["pair_of_forms", "mlp", "conv", "conv", "conv", "block", "stack", "dense", "dense", "program",
                       "reduce", "depthwise"])
    if kind == "pair_of_forms":
        return dict(kind=kind, n=rng.randint(1, 4), c=rng.randint(1, 16), h=rng.randint(7, 32), w=rng.randint(7, 32),
                    o=rng.randint(2, 48), k=rng.choice([1, 3, 5]), stride=rng.choice([1, 2]), pad=rng.choice([0, 1]),
                    dtype=rng.choice(["i8", "bf16"]))
    if kind == "mlp":
        return dict(kind=kind, batch=_log(rng, 1, 16384), d0=_log(rng, 64, 1024), d1=8 * _log(rng, 8, 128),
                    d2=8 * _log(rng, 8, 128), d3=rng.randint(2, 100))
    if kind == "conv":
        while True:
            k, stride = rng.choice([1, 3, 3, 3, 5]), rng.choice([1, 1, 2])
            c = dict(kind=kind, n=_log(rng, 1, 64), c=_channels(rng, 16, 512), h=_log(rng, 7, 112), w=_log(rng, 7, 112),
                     o=_channels(rng, 16, 512), k=k, stride=stride, pad=rng.choice([0, k // 2]),
                     dtype=rng.choice(["bf16", "bf16", "i8"]), residual=rng.random() < 0.5, relu=rng.random() < 0.5)
            # no larger than the stack's own layers; channel counts off the vector sizes smaller still
            if work(c)["flops"] <= (15e9 if c["c"] % 32 == 0 else 4e9):
                return c
    if kind == "block":
        return dict(kind=kind, n=_log(rng, 1, 64), c=rng.choice([64, 128, 256]), h=rng.randint(7, 28),
                    w=rng.randint(7, 28), o=16 * rng.randint(4, 32))
    if kind == "stack":
        return dict(kind=kind, batch=_log(rng, 1, 48), image=rng.randint(64, 224), classes=rng.randint(10, 1000))
    if kind == "dense":
        dtype = rng.choice(["bf16", "bf16", "i8", "fp8"])
        out = "i32" if dtype == "i8" else rng.choice(["f32", "bf16"])
        if rng.random() < 0.4:      # no alignment at all
            return dict(kind=kind, m=_log(rng, 64, 2048), n=_log(rng, 64, 2048), k=_log(rng, 64, 2048), dtype=dtype, out=out)
        while True:
            c = dict(kind=kind, m=_log(rng, 64, 8192), n=8 * _log(rng, 8, 1024), k=64 * _log(rng, 1, 128), dtype=dtype, out=out)
            if work(c)["flops"] <= 1.1e12:
                return c
    if kind == "program":
        return dict(kind=kind, n=_log(rng, 1, 32), c=16 * rng.randint(1, 4), h=rng.randint(14, 56), w=rng.randint(14, 56),
                    o=8 * rng.randint(2, 16), k=rng.choice([1, 3]), stride=rng.choice([1, 2]), pad=rng.choice([0, 1]),
                    dtype=rng.choice(["bf16", "i8"]))
    if kind == "reduce":
        while True:
            c = dict(kind=kind, rows=_log(rng, 16, 1 << 18), cols=_log(rng, 7, 8192),
                     dtype=rng.choice(["f32", "bf16", "i8", "i32"]), op=rng.choice(["sum", "max"]))
            if c["rows"] * c["cols"] <= 1 << 26:
                return c
    k = rng.choice([3, 3, 5])
    dtype = rng.choice(["bf16", "bf16", "i8"])
    while True:
        c = dict(kind="depthwise", n=_log(rng, 1, 32), c=_log(rng, 16, 512), h=_log(rng, 7, 112), w=_log(rng, 7, 112),
                 k=k, stride=rng.choice([1, 1, 2]), pad=k // 2, dtype=dtype,
                 out="i32" if dtype == "i8" else rng.choice(["bf16", "f32"]), relu=rng.random() < 0.5)
        if c["n"] * c["c"] * c["h"] * c["w"] <= 52e6:
            return c


class _Rand:
    """Seeded inputs made on the GPU: N(0,1) for real types, uniform on [-127, 127] for integers."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def __call__(self, shape, dtype, scale=1.0):
        if dtype == "i8":
            return torch.randint(-127, 128, shape, dtype=torch.int8, device=DEV, generator=self.g)
        if dtype == "i32":
            return torch.randint(-10000, 10001, shape, dtype=torch.int32, device=DEV, generator=self.g)
        x = torch.randn(shape, dtype=torch.float32, device=DEV, generator=self.g) * scale
        if dtype == "fp8":
            return x.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
        return x.to(torch.bfloat16) if dtype == "bf16" else x


def _out_hw(c):
    return ((c["h"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["w"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1)


def prepare(case, seed):
    rnd, kind = _Rand(seed), case["kind"]
    s = {"case": dict(case)}
    if kind == "pair_of_forms":
        s["x"] = rnd((case["n"], case["c"], case["h"], case["w"]), case["dtype"])
        s["w"] = rnd((case["o"], case["c"], case["k"], case["k"]), case["dtype"], (case["c"] * case["k"] ** 2) ** -0.5)
    elif kind == "conv":
        st, pd = (case["stride"],) * 2, (case["pad"],) * 2
        s["x"] = rnd((case["n"], case["c"], case["h"], case["w"]), case["dtype"])
        s["w"] = rnd((case["o"], case["c"], case["k"], case["k"]), case["dtype"], (case["c"] * case["k"] ** 2) ** -0.5)
        s["packed"] = gs.conv2d_pack_weights(s["w"], for_input=(s["x"], st, pd))
        shape, odt = (case["n"], case["o"], *_out_hw(case)), "i32" if case["dtype"] == "i8" else "bf16"
        s["residual"] = rnd(shape, odt) if case["residual"] else None
        s["out"] = torch.empty(shape, dtype=_OUT[odt], device=DEV)
    elif kind == "block":
        x = s["x"] = rnd((case["n"], case["c"], case["h"], case["w"]), "bf16")
        s["w3"] = rnd((case["o"], case["c"], 3, 3), "bf16", (9 * case["c"]) ** -0.5)
        s["w1"] = rnd((case["o"], case["c"], 1, 1), "bf16", case["c"] ** -0.5)
        s["packed"] = gs.conv2d_pack_weights(s["w3"], for_input=(x, (2, 2), (1, 1)))
        s["ws"] = torch.empty(gs.conv2d_workspace(x, s["w1"], (2, 2), (0, 0), form="im2col"), dtype=torch.uint8, device=DEV)
        h, w = (case["h"] - 1) // 2 + 1, (case["w"] - 1) // 2 + 1
        s["proj"] = torch.empty((case["n"], case["o"], h, w), dtype=torch.bfloat16, device=DEV)
        s["sum"] = torch.empty_like(s["proj"])
        s["pooled"] = torch.empty((case["n"], case["o"], h // 2, w // 2), dtype=torch.bfloat16, device=DEV)
    elif kind == "stack":
        weights = {name: rnd((cout, cin, k, k), "bf16", math.sqrt(2.0 / (cin * k * k)))
                   for name, cin, cout, k, _s, _p in RESNET18_CONVS}
        weights["fc"] = rnd((case["classes"], 512), "bf16", 512 ** -0.5)
        s["net"] = ResNet18Stack(weights, case["batch"], case["image"], DEV)
        s["net"].x.copy_(rnd((case["batch"], 3, case["image"], case["image"]), "bf16"))
    elif kind == "mlp":
        d = [case["d0"], case["d1"], case["d2"], case["d3"]]
        s["x"] = rnd((case["batch"], d[0]), "bf16")
        s["ws"] = [rnd((d[i + 1], d[i]), "bf16", d[i] ** -0.5) for i in range(3)]
        s["h"] = [torch.empty((case["batch"], d[i + 1]), dtype=torch.bfloat16 if i < 2 else torch.float32, device=DEV)
                  for i in range(3)]
    elif kind == "dense":
        s["a"] = rnd((case["m"], case["k"]), case["dtype"])
        s["b"] = rnd((case["n"], case["k"]), case["dtype"], case["k"] ** -0.5)
        s["out"] = torch.empty((case["m"], case["n"]), dtype=_OUT[case["out"]], device=DEV)
    elif kind == "program":
        s["tensors"] = {"activations": rnd((case["n"], case["c"], case["h"], case["w"]), case["dtype"]),
                        "weights": rnd((case["o"], case["c"], case["k"], case["k"]), case["dtype"],
                                       (case["c"] * case["k"] ** 2) ** -0.5)}
        s["ints"] = dict(C=case["c"], K=case["k"], S=case["stride"], P=case["pad"])
        meta = {k: (tuple(v.shape), v.dtype) for k, v in s["tensors"].items()}
        s["text"] = gs.program_rewrite(CONV2D_PADDED, "im2col", meta, s["ints"])
        s["out_dtype"] = _OUT["i32" if case["dtype"] == "i8" else "bf16"]
    elif kind == "reduce":
        s["x"] = rnd((case["rows"], case["cols"]), case["dtype"])
    else:
        s["x"] = rnd((case["n"], case["c"], case["h"], case["w"]), case["dtype"])
        s["w"] = rnd((case["c"], case["k"], case["k"]), case["dtype"], 1.0 / case["k"])
        s["out"] = torch.empty((case["n"], case["c"], *_out_hw(case)), dtype=_OUT[case["out"]], device=DEV)
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "pair_of_forms":
        st, pd = (c["stride"],) * 2, (c["pad"],) * 2
        return gs.conv2d_direct(s["x"], s["w"], st, pd), gs.conv2d_im2col(s["x"], s["w"], st, pd)
    if kind == "conv":
        return gs.conv2d_direct_packed(s["x"], s["w"], s["packed"], (c["stride"],) * 2, (c["pad"],) * 2,
                                       residual=s["residual"], act=gs.GS_ACT_RELU if c["relu"] else gs.GS_ACT_NONE,
                                       out=s["out"])
    if kind == "block":
        gs.conv2d_im2col(s["x"], s["w1"], (2, 2), (0, 0), out=s["proj"], workspace=s["ws"])
        gs.conv2d_direct_packed(s["x"], s["w3"], s["packed"], (2, 2), (1, 1), residual=s["proj"], act=gs.GS_ACT_RELU,
                                out=s["sum"])
        gs.windows_reduce(s["sum"], 2, (2, 2), (2, 2), None, None, gs.GS_MAX, out=s["pooled"])
        return s["sum"], s["pooled"]
    if kind == "stack":
        return s["net"].forward()
    if kind == "mlp":
        h = s["x"]
        for i, w in enumerate(s["ws"]):
            h = gs.cartesian_dot(h, w, act=gs.GS_ACT_RELU if i < 2 else gs.GS_ACT_NONE, out=s["h"][i])
        return s["h"]
    if kind == "dense":
        return gs.cartesian_dot(s["a"], s["b"], out=s["out"])
    if kind == "program":
        return gs.program_eval(s["text"], s["tensors"], s["ints"], out_dtype=s["out_dtype"])
    if kind == "reduce":
        return gs.reduce(s["x"], 1, gs.GS_SUM if c["op"] == "sum" else gs.GS_MAX)
    return gs.depthwise_conv2d(s["x"], s["w"], (c["stride"],) * 2, (c["pad"],) * 2,
                               act=gs.GS_ACT_RELU if c["relu"] else gs.GS_ACT_NONE, out=s["out"])


def _conv_work(n, c, h, w, o, k, stride, pad, esz, osz, extra=0):
    ho, wo = (h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1
    res = n * o * ho * wo
    return dict(bytes=float(n * c * h * w * esz + o * c * k * k * esz + res * (osz + extra)), flops=2.0 * res * c * k * k)


def work(case):
    kind = case["kind"]
    if kind in ("pair_of_forms", "conv", "program"):
        e, osz = _ESZ[case["dtype"]], 4 if case["dtype"] == "i8" or kind == "pair_of_forms" else 2
        w = _conv_work(case["n"], case["c"], case["h"], case["w"], case["o"], case["k"], case["stride"], case["pad"], e, osz,
                       osz if case.get("residual") else 0)
        if kind == "pair_of_forms":         # two results
            w = {k: 2 * v for k, v in w.items()}
        return w
    if kind == "block":
        n, c, h, w, o = (case[k] for k in ("n", "c", "h", "w", "o"))
        a, b = _conv_work(n, c, h, w, o, 3, 2, 1, 2, 2), _conv_work(n, c, h, w, o, 1, 2, 0, 2, 2)
        ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
        return dict(bytes=float(2 * (n * c * h * w + 10 * o * c + n * o * (ho * wo + (ho // 2) * (wo // 2)))),
                    flops=a["flops"] + b["flops"])
    if kind == "stack":
        hw, hin, flops, weights = case["image"], 0, 0.0, 0
        for name, cin, cout, k, st, p in RESNET18_CONVS:
            weights += cin * cout * k * k
            if name == "conv1":
                ho = (hw + 2 * p - k) // st + 1
                hw = (ho - 1) // 2 + 1
            elif name.endswith("c1"):
                ho = hw = (hw + 2 * p - k) // st + 1
            else:
                ho = hw
            flops += 2.0 * case["batch"] * ho * ho * cout * cin * k * k
        flops += 2.0 * case["batch"] * 512 * case["classes"]
        return dict(bytes=2.0 * (case["batch"] * 3 * case["image"] ** 2 + weights + 512 * case["classes"]) +
                    4.0 * case["batch"] * case["classes"], flops=flops)
    if kind == "mlp":
        d, b = [case["d0"], case["d1"], case["d2"], case["d3"]], case["batch"]
        macs = sum(d[i] * d[i + 1] for i in range(3))
        return dict(bytes=2.0 * (b * d[0] + macs) + 4.0 * b * d[3], flops=2.0 * b * macs)
    if kind == "dense":
        e, osz = _ESZ[case["dtype"]], 2 if case["out"] == "bf16" else 4
        return dict(bytes=float((case["m"] + case["n"]) * case["k"] * e + case["m"] * case["n"] * osz),
                    flops=2.0 * case["m"] * case["n"] * case["k"])
    if kind == "reduce":
        e = _ESZ[case["dtype"]]
        osz = 4 if case["dtype"] == "i8" and case["op"] == "sum" else e
        return dict(bytes=float(case["rows"] * (case["cols"] * e + osz)), flops=float(case["rows"] * case["cols"]))
    ho, wo = _out_hw(case)
    osz = 2 if case["out"] == "bf16" else 4
    planes = case["n"] * case["c"]
    return dict(bytes=float(planes * (case["h"] * case["w"] * _ESZ[case["dtype"]] + ho * wo * osz) +
                            case["c"] * case["k"] ** 2 * _ESZ[case["dtype"]]),
                flops=2.0 * planes * ho * wo * case["k"] ** 2)


def tolerance(case):
    """About four times what a pass differs by from itself with sums in 64 bits (measured)."""
    kind, dtype = case["kind"], case.get("dtype", "bf16")
    if dtype in ("i8", "i32") or (kind == "reduce" and case["op"] == "max"):
        return "exact"
    if kind == "stack":             # twenty layers, each stored as bfloat16: 2.0e-3 .. 3.3e-3, 8.9e-3
        return {"rel": 1.3e-2, "max": 3.6e-2}
    if kind == "mlp":               # a hidden value stored one bfloat16 step off now and then: 5.1e-5, 7.3e-3
        return {"rel": 3e-4, "max": 3e-2}
    if kind == "dense" and case["out"] == "f32":
        # 8-bit floats: the matrix unit aligns the products of a step before it adds them (7.4e-6, 8.8e-5)
        return {"rel": 3e-5, "max": 4e-4} if dtype == "fp8" else {"rel": 1e-5, "max": 1e-4}
    if kind == "pair_of_forms" or (kind == "reduce" and dtype == "f32") or (kind == "depthwise" and case["out"] == "f32"):
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "block":             # the projection is rounded before it is added: 1.7e-3, 7.9e-3
        return {"rel": 7e-3, "max": 3.2e-2}
    return {"rel": 7e-3, "max": 1.6e-2}     # one rounding to bfloat16: 1.7e-3, 3.9e-3

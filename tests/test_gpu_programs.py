"""GPU parity of programs given as text: the same s-expression goes to the CPU oracle's interpreter
and to `glenside_program_eval`; integer results bit-exact, bfloat16 within 1e-2 relative."""

import numpy as np
import pytest
import torch

from oracle import sexpr
from paper_2105_09377_amd import binding as gs, synth
from helpers import assert_parity, fp8_slack, to_oracle
import listings

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_both(text, tensors, ints=None, out_dtype=None):
    ints = ints or {}
    want = sexpr.evaluate(text, {k: to_oracle(v) for k, v in tensors.items()}, ints)
    got = gs.program_eval(text, {k: v.to(DEV) for k, v in tensors.items()}, ints, out_dtype=out_dtype)
    assert tuple(got.shape) == want.shape
    return got, want


@pytest.mark.parametrize("dtype,odt", [("i8", None), ("bf16", None), ("bf16", torch.bfloat16)])
@pytest.mark.parametrize("shape", [(2, 3, 9, 8, 5, 3, 2, 2, 1), (3, 64, 20, 20, 70, 3, 3, 1, 1), (2, 16, 12, 12, 8, 1, 1, 2, 2)])
def test_conv2d_listing(dtype, odt, shape):
    n, c, h, w, o, kh, kw, sh, sw = shape
    cfg = synth.conv_layer(n, c, h, w, o, kh, 1, 0, dtype, 9300 + c + o)
    wt = cfg["w"][:, :, :, :kw].contiguous()
    ints = dict(C=c, Kh=kh, Kw=kw, Sh=sh, Sw=sw)
    tensors = {"activations": cfg["x"], "weights": wt}
    got, want = run_both(listings.CONV2D, tensors, ints, odt)
    assert_parity(got, want.materialize(), what=f"Fig. 2a {dtype} {shape}")
    # the program the im2col rules derive from it (Fig. 5), dispatched like Fig. 2a or node by node
    meta = {k: (tuple(v.shape), v.dtype) for k, v in tensors.items()}
    im2col = gs.program_rewrite(listings.CONV2D, "im2col", meta, ints)
    got2 = gs.program_eval(im2col, {k: v.to(DEV) for k, v in tensors.items()}, ints, out_dtype=odt)
    assert_parity(got2, want.materialize(), what=f"Fig. 5 {dtype} {shape}")
    # the same surely node by node (explicit windows -> flatten -> contraction -> reshape -> squeeze -> transpose):
    # a reshape of the flattened weights to their own shape is no part of the listing
    by_node = im2col.replace("(flatten (access weights 1))", f"(reshape (flatten (access weights 1)) (shape {o}) (shape {c * kh * kw}))")
    assert by_node != im2col
    got3 = gs.program_eval(by_node, {k: v.to(DEV) for k, v in tensors.items()}, ints, out_dtype=odt)
    assert_parity(got3, want.materialize(), what=f"Fig. 5 by node {dtype} {shape}")
    if dtype == "i8":
        assert torch.equal(got, got2) and torch.equal(got, got3)


def test_conv2d_listing_on_padded_tensor():
    cfg = synth.conv_layer(2, 32, 14, 14, 40, 3, 1, 1, "i8", 9400)
    ints = dict(C=32, Kh=3, Kw=3, Sh=1, Sw=1, Ph=1, Pw=1)
    got, want = run_both(listings.CONV2D_PADDED, {"activations": cfg["x"], "weights": cfg["w"]}, ints)
    assert_parity(got, want.materialize(), what="padded Fig. 2a")
    assert torch.equal(got, gs.conv2d_direct(cfg["x"].to(DEV), cfg["w"].to(DEV), (1, 1), (1, 1)))


# Zero padding that a consumer can take over (convolution, windows, sums of windows), padding that it
# cannot (one side only, other dimensions, a maximum), and the flat form of the convolution listing.
@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("pads", [((2, 1, 1), (3, 2, 2)), ((2, 1, 0), (3, 0, 2)), ((1, 0, 2), (2, 1, 1)), ((0, 1, 0), (3, 1, 1))])
def test_padding_in_front_of_windows(pads, dtype):
    x = {"i8": synth.uniform_int8, "bf16": lambda s, lo, hi, st: synth.normal_bf16(s, 1.0, st)}[dtype]((2, 6, 9, 8), -9, 9, 9450)
    grown = [2, 6, 9, 8]
    act = "activations"
    for dim, lo, hi in pads:
        act = f"(pad {act} {dim} {lo} {hi})"
        grown[dim] += lo + hi
    c = grown[1]
    w = {"i8": synth.uniform_int8, "bf16": lambda s, lo, hi, st: synth.normal_bf16(s, 0.2, st)}[dtype]((5, c, 3, 2), -9, 9, 9451)
    ints = dict(C=c, Kh=3, Kw=2, Sh=1, Sw=2)
    tensors = {"activations": x, "weights": w}
    conv = listings.CONV2D.replace("activations", act, 1)
    meta = {k: (tuple(v.shape), v.dtype) for k, v in tensors.items()}
    for text in (conv, gs.program_rewrite(conv, "im2col", meta, ints)):
        got, want = run_both(text, tensors, ints)
        assert_parity(got, want.materialize(), what=text)
    for text in (f"(windows (access {act} 2) (shape Kh Kw) (shape Sh Sw))",
                 f"(compute reduceSum (windows (access {act} 2) (shape Kh Kw) (shape Sh Sw)))",
                 f"(compute reduceMax (windows (access {act} 2) (shape Kh Kw) (shape Sh Sw)))"):
        got, want = run_both(text, {"activations": x}, ints)
        assert_parity(got, want.materialize(), what=text)


# Convolutions that the direct kernels refuse (a stride above 64, rows or windows too large for the LDS, many
# images in one tile), the next ones that they take, and the sides of the line to where they are faster: the
# flat form evaluates all of them.
@pytest.mark.parametrize("dtype,odt", [("i8", None), ("bf16", None), ("bf16", torch.bfloat16)])
@pytest.mark.parametrize("shape", [(1, 2, 70, 9, 3, 3, 1, 65, 1), (1, 16, 4, 1300, 8, 3, 3, 1, 1), (1, 16, 4, 900, 8, 3, 3, 1, 1),
                                   (40, 32, 3, 3, 8, 3, 3, 1, 1), (16, 32, 3, 3, 8, 3, 3, 1, 1), (1, 32, 12, 12, 4, 11, 11, 1, 1),
                                   (2, 64, 9, 10, 24, 3, 3, 1, 1), (9, 48, 33, 31, 9, 3, 3, 1, 1), (8, 48, 33, 31, 9, 3, 3, 1, 1),
                                   (1, 16, 6, 5, 20, 1, 1, 1, 1), (8, 3, 36, 37, 129, 5, 5, 1, 1), (2, 512, 9, 9, 4, 1, 1, 4, 4),
                                   (2, 16, 9, 11, 5, 3, 3, 2, 2), (2, 17, 9, 11, 5, 3, 3, 2, 2), (2, 32, 9, 10, 5, 3, 3, 2, 2)])
def test_flat_form_of_every_route(shape, dtype, odt):
    n, c, h, w, o, kh, kw, sh, sw = shape
    tensors = {"activations": gen_small(dtype, (n, c, h, w), 9470), "weights": gen_small(dtype, (o, c, kh, kw), 9471)}
    ints = dict(C=c, Kh=kh, Kw=kw, Sh=sh, Sw=sw)
    meta = {k: (tuple(v.shape), v.dtype) for k, v in tensors.items()}
    got, want = run_both(gs.program_rewrite(listings.CONV2D, "im2col", meta, ints), tensors, ints, odt)
    assert_parity(got, want.materialize(), what=str(shape))


# Both sides of the lines between the ways that the flat form goes: padded 1x1 windows on few and many channels by results and
# positions, few short windows and longer ones, few 5x5 windows.
@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("shape", [(32, 32, 30, 30, 64, 1, 1, 1), (32, 32, 30, 29, 64, 1, 1, 1), (32, 32, 30, 30, 65, 1, 1, 1), (32, 35, 61, 61, 5, 1, 2, 1),
                                   (32, 9, 30, 30, 64, 1, 1, 1), (32, 9, 31, 30, 64, 1, 1, 1), (16, 11, 30, 30, 128, 1, 1, 1), (16, 11, 30, 30, 129, 1, 1, 1),
                                   (96, 32, 30, 30, 65, 1, 1, 1),
                                   (2, 28, 9, 11, 20, 3, 1, 1), (2, 29, 9, 11, 20, 3, 1, 1), (2, 56, 9, 11, 20, 3, 1, 1), (2, 57, 9, 11, 20, 3, 1, 1),
                                   (2, 40, 9, 14, 20, 5, 1, 0), (8, 40, 14, 14, 20, 5, 1, 2), (1, 102, 13, 63, 70, 3, 2, 1), (1, 101, 7, 39, 70, 5, 2, 0)])
def test_flat_form_on_both_sides_of_its_lines(shape, dtype):
    n, c, h, w, o, k, s, p = shape
    tensors = {"activations": gen_small(dtype, (n, c, h, w), 9476), "weights": gen_small(dtype, (o, c, k, k), 9477)}
    ints = dict(C=c, Kh=k, Kw=k, Sh=s, Sw=s, Ph=p, Pw=p)
    meta = {name: (tuple(v.shape), v.dtype) for name, v in tensors.items()}
    want = torch.nn.functional.conv2d(tensors["activations"].double(), tensors["weights"].double(), stride=s, padding=p).numpy()
    got = gs.program_eval(gs.program_rewrite(listings.CONV2D_PADDED, "im2col", meta, ints), {name: v.to(DEV) for name, v in tensors.items()}, ints)
    assert_parity(got, want.astype(np.int64) if dtype == "i8" else want, what=str(shape))


# Padded rows around the LDS limit of the direct kernels: with padding of its own a patch row is two pixels longer
# than a row of the padded tensor, so at 748 columns the padding is materialised; and a few-channel image that
# only the few-channel kernel takes.
@pytest.mark.parametrize("shape", [(1, 40, 3, 746, 8, 3, 1), (1, 40, 3, 747, 8, 3, 1), (1, 40, 3, 748, 8, 3, 1), (1, 3, 9, 1100, 8, 7, 3)])
def test_padded_rows_at_the_lds_limit(shape):
    n, c, h, w, o, k, p = shape
    tensors = {"activations": synth.uniform_int8((n, c, h, w), -9, 9, 9480), "weights": synth.uniform_int8((o, c, k, k), -9, 9, 9481)}
    ints = dict(C=c, Kh=k, Kw=k, Sh=1, Sw=1, Ph=p, Pw=p)
    meta = {name: (tuple(v.shape), v.dtype) for name, v in tensors.items()}
    xp = torch.nn.functional.pad(tensors["activations"].double(), (p, p, p, p))
    want = torch.nn.functional.conv2d(xp, tensors["weights"].double()).to(torch.int32)
    for text in (listings.CONV2D_PADDED, gs.program_rewrite(listings.CONV2D_PADDED, "im2col", meta, ints)):
        got = gs.program_eval(text, {name: v.to(DEV) for name, v in tensors.items()}, ints)
        assert torch.equal(got.cpu(), want)


# Padding of at least the window in front of convolutions that the pipelined kernels take (whole chunks of
# channels; rows of whole vectors and not; several images in a tile): whole patch rows are padding.
@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("shape", [(3, 64, 12, 16, 70, 3, 3, 1), (3, 64, 12, 16, 64, 3, 7, 1), (2, 128, 9, 13, 40, 3, 5, 2), (9, 64, 4, 4, 64, 3, 4, 1),
                                   (2, 64, 10, 10, 32, 1, 3, 1), (2, 64, 8, 8, 33, 5, 9, 1), (1, 64, 6, 40, 32, 3, 64, 1)])
def test_padding_wider_than_the_window(shape, dtype):
    n, c, h, w, o, k, p, s = shape
    x = gen_small(dtype, (n, c, h, w), 9490)
    wt = gen_small(dtype, (o, c, k, k), 9491)
    ints = dict(C=c, Kh=k, Kw=k, Sh=s, Sw=s, Ph=p, Pw=p)
    want = torch.nn.functional.conv2d(torch.nn.functional.pad(x.double(), (p, p, p, p)), wt.double(), stride=s).numpy()
    want = want.astype(np.int64) if dtype == "i8" else want
    got = gs.program_eval(listings.CONV2D_PADDED, {"activations": x.to(DEV), "weights": wt.to(DEV)}, ints)
    assert_parity(got, want, what=str(shape))
    assert torch.equal(got, gs.conv2d_direct(x.to(DEV), wt.to(DEV), (s, s), (p, p)))


def gen_small(dtype, shape, stream):
    return synth.uniform_int8(shape, -9, 9, stream) if dtype == "i8" else synth.normal_bf16(shape, 0.3, stream)


@pytest.mark.parametrize("dtype", ["i8", "bf16", "fp8"])
@pytest.mark.parametrize("dims", [(32, 32, 32), (70, 96, 200)])
def test_matmul_listing_and_its_rewrites(dtype, dims):
    m, n, k = dims
    if dtype == "i8":
        a, w = synth.uniform_int8((m, k), -127, 127, 9500), synth.uniform_int8((k, n), -127, 127, 9501)
    elif dtype == "bf16":
        a, w = synth.normal_bf16((m, k), 1.0, 9500), synth.normal_bf16((k, n), k ** -0.5, 9501)
    else:
        a, w = synth.normal_fp8((m, k), 1.0, 9500), synth.normal_fp8((k, n), k ** -0.5, 9501)
    tensors = {"activations": a, "weights": w}
    got, want = run_both(listings.MATMUL, tensors)
    ref = want.materialize()
    slack = fp8_slack(to_oracle(a), to_oracle(w).T) if dtype == "fp8" else None
    assert_parity(got, ref, what="Fig. 2b", slack=slack)
    meta = {k_: (tuple(v.shape), v.dtype) for k_, v in tensors.items()}
    dev = {k_: v.to(DEV) for k_, v in tensors.items()}
    blocked = gs.program_rewrite(listings.MATMUL, "block", meta, params=(16, 32, 16))
    assert_parity(gs.program_eval(blocked, dev), ref, what="blocked program (Fig. 7)", slack=slack)
    systolic = gs.program_rewrite(listings.MATMUL, "systolic", meta)
    assert_parity(gs.program_eval(systolic, dev), ref, what="systolicArray (Fig. 3)", slack=slack)


# Both listings where one launch or the im2col entry point evaluates them: 1x1 windows with and without padding, whole
# and broken steps of channels, small images, few windows just below and above the line, strides that no direct kernel takes.
@pytest.mark.parametrize("dtype,odt", [("i8", torch.int32), ("bf16", torch.bfloat16), ("bf16", torch.float32)])
@pytest.mark.parametrize("n,c,h,w,o,k,s,p", [
    (2, 64, 14, 15, 40, 1, 1, 0), (3, 48, 17, 22, 33, 1, 2, 0), (9, 16, 41, 34, 20, 1, 1, 1), (1, 33, 9, 7, 65, 1, 2, 1), (1, 24, 60, 70, 10, 1, 1, 0),
    (5, 32, 14, 18, 48, 3, 1, 0), (1, 48, 31, 43, 50, 3, 2, 0), (2, 64, 23, 44, 30, 3, 1, 1), (4, 48, 18, 25, 17, 3, 1, 1), (2, 7, 20, 20, 9, 3, 4, 1), (1, 40, 9, 9, 5, 4, 1, 0)])
def test_convolution_listings_in_one_launch_and_as_im2col(n, c, h, w, o, k, s, p, dtype, odt):
    cfg = synth.conv_layer(n, c, h, w, o, k, s, p, dtype, 9650 + c + o)
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p).numpy()
    want = want.astype(np.int64) if dtype == "i8" else want
    dev = {"activations": cfg["x"].to(DEV), "weights": cfg["w"].to(DEV)}
    ints = dict(C=c, Kh=k, Kw=k, Sh=s, Sw=s, Ph=p, Pw=p)
    meta = {name: (tuple(v.shape), v.dtype) for name, v in dev.items()}
    for text in (listings.CONV2D_PADDED, gs.program_rewrite(listings.CONV2D_PADDED, "im2col", meta, ints)):
        assert_parity(gs.program_eval(text, dev, ints, out_dtype=odt), want, what=text)


@pytest.mark.parametrize("dtype", ["i8", "bf16", "f32"])
def test_maxpool_listing(dtype):
    x = {"i8": synth.uniform_int8((3, 5, 17, 18), -127, 127, 9600), "bf16": synth.normal_bf16((3, 5, 17, 18), 1.0, 9600),
         "f32": synth.normal_f32((3, 5, 17, 18), 1.0, 9600)}[dtype]
    got, want = run_both(listings.MAXPOOL, {"activations": x}, dict(Kh=3, Kw=2, Sh=2, Sw=2))
    np.testing.assert_array_equal(to_oracle(got), want.materialize())


def test_transformer_compositions():
    a = synth.normal_f32((6, 10), 1.0, 9700)
    b = synth.normal_f32((6, 10), 1.0, 9701)
    t = {"a": a, "b": b}
    for text in [
        "(compute reduceSum (pair (access a 2) (access b 2)))",                       # element-wise sum (Sec. 5.4)
        "(compute reduceMax (pair (access a 2) (access b 2)))",
        "(compute reduceSum (access a 1))",
        "(compute reduceSum (pair (access a 1) (access b 1)))",                       # folds the rows as well
        "(concat (slice (access a 1) 1 0 4) (slice (access b 1) 1 4 10) 1)",
        "(transpose (concat (access a 1) (access b 1) 0) (list 1 0))",
        "(slice (access a 1) 0 2 5)",                                                 # a view, copied out
        "(access a 1)",
        "(flatten (pair (access a 1) (access b 1)))",
        "(compute relu (compute reduceSum (pair (access a 2) (access b 2))))",
        "(reshape (compute reduceSum (windows (access a 1) (shape 4) (shape 3))) (shape 3 6) (shape))",
    ]:
        got, want = run_both(text, t)
        assert_parity(got, want.materialize(), float_tol=1e-5, what=text)


def test_unsupported_and_workspace_errors():
    a = synth.normal_bf16((8, 16), 1.0, 9800).to(DEV)
    with pytest.raises(gs.GlensideError) as e:
        gs.program_eval("(cartProd (access a 1) (access a 1))", {"a": a})            # a bare Cartesian product
    assert e.value.status == gs.GS_ERR_UNSUPPORTED
    out = torch.empty((8, 8), dtype=torch.float32, device=DEV)
    with pytest.raises(gs.GlensideError) as e:
        gs.program_eval("(compute dotProd (cartProd (access a 1) (slice (access a 1) 1 0 16)))", {"a": a}, out=out,
                        workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
    assert e.value.status == gs.GS_ERR_WORKSPACE


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
def test_random_programs(dtype):
    """Two hundred seeded random programs (Table 1 transformers, dotProd / reduceSum / reduceMax) on small
    tensors: whatever the library accepts must equal the oracle -- bit for bit on int8 inputs -- and it must
    accept most of them; what it refuses, it must refuse with a status, launching nothing."""
    import random_programs
    rng = np.random.default_rng(20210509 + (0 if dtype == "i8" else 1))
    shapes = {"a": (3, 4, 6, 5), "b": (6, 8), "c": (2, 1, 7)}
    def make(shape, stream):
        return synth.uniform_int8(shape, -5, 5, stream) if dtype == "i8" else synth.normal_bf16(shape, 1.0, stream)
    tensors = {k: make(s, 9900 + i) for i, (k, s) in enumerate(shapes.items())}
    tensors.update({k + "2": make(s, 9950 + i) for i, (k, s) in enumerate(shapes.items())})
    same = {k: (k[:-1] if k.endswith("2") else k + "2") for k in tensors}
    host = {k: to_oracle(v) for k, v in tensors.items()}
    dev = {k: v.to(DEV) for k, v in tensors.items()}
    ran = refused = 0
    for i in range(200):
        text = random_programs.grow(rng, host, same, depth=int(rng.integers(1, 6)))
        want = sexpr.evaluate(text, host)
        try:
            got = gs.program_eval(text, dev)
        except gs.GlensideError as e:
            # rank: a cartProd inside a dotProd may exceed the eight dimensions of the boundary
            assert e.status in (gs.GS_ERR_UNSUPPORTED, gs.GS_ERR_DTYPE) or \
                (e.status == gs.GS_ERR_RANK and "cartProd" in text), (text, e.status)
            refused += 1
            continue
        ran += 1
        assert tuple(got.shape) == want.shape, text
        ref = want.materialize()
        if not np.isfinite(ref.astype(np.float64)).all():        # reduceMax over a padded window of -inf etc.
            np.testing.assert_array_equal(np.isfinite(to_oracle(got)), np.isfinite(ref), err_msg=text)
            continue
        # a chain of computes stores its intermediate results in bfloat16 (one more rounding of
        # 2^-9 per link, which a later cancellation can amplify); the oracle keeps fp64 throughout
        chained = dtype == "bf16" and text.count("compute") > 1
        assert_parity(got, ref, float_tol=5e-2 if chained else 1e-2, what=text)
    assert ran >= 150, (ran, refused)

"""GPU parity: every entry point of the C ABI against the CPU oracle on the same seeded inputs.

Integer results must be bit-exact; bf16-in / fp32-accumulate results must be within 1e-2 maximum
relative error (floor 1e-3 * max|ref| on the denominator).  Sizes span several tiles and ragged
tails of the kernels' 32/64/128-wide tiles.
"""

import math

import numpy as np
import pytest
import torch

from oracle import access_pattern as ap
from oracle import brute
from oracle import programs as pg
from paper_2105_09377_amd import binding as gs
from paper_2105_09377_amd import synth
import tile_instances
from helpers import assert_parity, fp8_slack, to_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def gen(dtype, shape, stream, scale=1.0):
    if dtype == "i8":
        return synth.uniform_int8(shape, -127, 127, stream)
    if dtype == "i32":
        return synth.uniform_int32(shape, -100000, 100000, stream)
    if dtype == "bf16":
        return synth.normal_bf16(shape, scale, stream)
    if dtype == "fp8":
        return synth.normal_fp8(shape, scale, stream)
    return synth.normal_f32(shape, scale, stream)


def oracle_windows(x, n_access, window, stride, pad_lo, pad_hi, fill):
    node = ap.tensor(to_oracle(x))
    nc = x.dim() - n_access
    for d in range(nc):
        lo = pad_lo[d] if pad_lo else 0
        hi = pad_hi[d] if pad_hi else 0
        if lo or hi:
            node = ap.pad(node, n_access + d, lo, hi, fill)
    return ap.windows(ap.access(node, n_access), window, stride)


LOWEST = {"i8": -128, "i32": -2 ** 31, "bf16": -np.inf, "f32": -np.inf}

# ---------------------------------------------------------------------------------------------
# windows
# ---------------------------------------------------------------------------------------------

WINDOW_CASES = [
    # dtype, shape, n_access, window, stride, pad_lo, pad_hi, pad_mode
    ("f32", (5, 37), 1, (4,), (3,), None, None, gs.GS_PAD_ZERO),
    ("bf16", (2, 3, 9, 11), 2, (3, 2), (2, 3), (1, 0), (1, 1), gs.GS_PAD_LOWEST),
    ("i8", (1, 3, 8, 8), 1, (3, 3, 3), (1, 1, 1), None, None, gs.GS_PAD_ZERO),
    ("i8", (2, 5, 13, 10), 1, (5, 3, 3), (1, 2, 2), (0, 1, 1), (0, 1, 1), gs.GS_PAD_ZERO),
    ("bf16", (3, 16, 20, 20), 1, (16, 3, 3), (1, 1, 1), (0, 1, 1), (0, 1, 1), gs.GS_PAD_ZERO),
    ("i32", (2, 2, 6, 7), 2, (2, 2), (2, 2), None, None, gs.GS_PAD_LOWEST),
    ("bf16", (2, 3, 15, 15), 1, (3, 7, 7), (1, 2, 2), (0, 3, 3), (0, 3, 3), gs.GS_PAD_ZERO),
    # convolution-shaped windows through LDS: 16-byte rows, several channel passes, strides,
    # asymmetric padding, every element size
    ("bf16", (2, 8, 24, 32), 1, (8, 3, 3), (1, 1, 1), (0, 1, 1), (0, 1, 1), gs.GS_PAD_ZERO),
    ("bf16", (1, 320, 6, 40), 1, (320, 3, 3), (1, 1, 1), (0, 1, 1), (0, 1, 1), gs.GS_PAD_ZERO),
    ("i8", (2, 48, 10, 48), 1, (48, 3, 3), (1, 2, 2), (0, 1, 1), (0, 1, 1), gs.GS_PAD_LOWEST),
    ("i8", (1, 16, 9, 21), 1, (16, 2, 4), (1, 1, 3), (0, 0, 2), (0, 1, 0), gs.GS_PAD_ZERO),
    ("f32", (3, 4, 11, 12), 1, (4, 5, 3), (1, 2, 1), (0, 2, 1), (0, 2, 1), gs.GS_PAD_LOWEST),
    ("i32", (1, 8, 7, 9), 1, (8, 1, 1), (1, 2, 2), None, None, gs.GS_PAD_ZERO),
]


@pytest.mark.parametrize("case", WINDOW_CASES)
def test_access_windows(case):
    dtype, shape, na, window, stride, lo, hi, mode = case
    x = gen(dtype, shape, 1000 + len(shape) + shape[-1])
    got = gs.access_windows(x.to(DEV), na, window, stride, lo, hi, mode)
    fill = LOWEST[dtype] if mode == gs.GS_PAD_LOWEST else 0
    want = oracle_windows(x, na, window, stride, lo, hi, fill).materialize()
    got_np = to_oracle(got)
    assert got_np.shape == want.shape
    np.testing.assert_array_equal(got_np, want)          # a gather is exact in every dtype


def test_access_windows_is_the_im2col_matrix():
    """flatten(windows ...) of Fig. 5 is the same memory as the windows result."""
    x = gen("i8", (2, 4, 9, 9), 1100)
    got = gs.access_windows(x.to(DEV), 1, (4, 3, 3), (1, 2, 2), (0, 1, 1), (0, 1, 1))
    want = pg.im2col_matrix(ap.tensor(to_oracle(x)), (4, 3, 3), (2, 2), (1, 1)).materialize()
    np.testing.assert_array_equal(to_oracle(got).reshape(want.shape), want)


# ---------------------------------------------------------------------------------------------
# compute dotProd (cartProd a0 a1)
# ---------------------------------------------------------------------------------------------

DOT_CASES = [
    # dtype, a0 shape, n0, a1 shape, n1, out dtype, relu
    ("i8", (36, 27), 1, (4, 27), 1, torch.int32, False),          # the tiny conv's im2col product
    ("i8", (300, 328), 1, (200, 328), 1, torch.int32, False),     # ragged tiles, K not a slab multiple
    ("i8", (130, 1000), 1, (70, 1000), 1, torch.int32, True),
    ("bf16", (256, 784), 1, (512, 784), 1, torch.float32, True),  # MLP layer 1
    ("bf16", (256, 512), 1, (10, 512), 1, torch.float32, False),  # MLP layer 3
    ("bf16", (100, 147), 1, (64, 147), 1, torch.bfloat16, False), # K = 147: unaligned rows
    ("bf16", (2, 3, 4, 5), 2, (7, 4, 5), 1, torch.float32, False),  # multi-dim access and compute shapes
    ("bf16", (513, 64), 1, (129, 64), 1, torch.bfloat16, True),
    ("i8", (1, 5), 1, (1, 5), 1, torch.int32, False),
    # K a whole number of 32-byte steps but not of 128-byte slabs: short last slab
    ("bf16", (70, 80), 1, (300, 80), 1, torch.float32, False),
    ("bf16", (33, 16), 1, (65, 16), 1, torch.bfloat16, True),
    ("i8", (129, 96), 1, (140, 96), 1, torch.int32, False),
    ("bf16", (300, 784), 1, (512, 784), 1, torch.bfloat16, True),
    # result rows written 8 and 4 columns per lane, in every result type
    ("i8", (64, 128), 1, (72, 128), 1, torch.int32, True),
    ("bf16", (40, 64), 1, (76, 64), 1, torch.bfloat16, False),
    ("bf16", (200, 256), 1, (264, 256), 1, torch.float32, False),
    # 8-bit floats: 64-byte K steps; K not a multiple of 64 takes the loader for rows of any alignment
    ("fp8", (300, 328), 1, (200, 328), 1, torch.float32, False),
    ("fp8", (130, 1000), 1, (70, 1000), 1, torch.bfloat16, True),
    ("fp8", (64, 128), 1, (72, 128), 1, torch.float32, True),
    ("fp8", (129, 192), 1, (140, 192), 1, torch.bfloat16, False),   # short last slab
    ("fp8", (2, 3, 4, 8), 2, (7, 4, 8), 1, torch.float32, False),
    ("fp8", (1, 5), 1, (1, 5), 1, torch.float32, False),
    ("fp8", (256, 832), 1, (512, 832), 1, torch.float32, True),
]


@pytest.mark.parametrize("case", DOT_CASES)
def test_cartesian_dot(case):
    dtype, s0, n0, s1, n1, odt, relu = case
    k = int(np.prod(s0[n0:]))
    a0 = gen(dtype, s0, 1200 + s0[0], 1.0)
    a1 = gen(dtype, s1, 1300 + s1[0], 1.0 / np.sqrt(k) if dtype in ("bf16", "fp8") else 1.0)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), n0, n1, odt, gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE)
    prog = pg.cartesian_dot(ap.access(ap.tensor(to_oracle(a0)), n0), ap.access(ap.tensor(to_oracle(a1)), n1))
    if relu:
        prog = ap.compute(ap.relu, prog)
    assert tuple(got.shape) == prog.access_shape
    slack = None
    if dtype == "fp8":
        slack = fp8_slack(to_oracle(a0).reshape(-1, k), to_oracle(a1).reshape(-1, k)).reshape(prog.access_shape)
    assert_parity(got, prog.materialize(), what=str(case), slack=slack)


# Edges of the contraction's tile rules: rows of any byte alignment and length (fewer than 16 bytes, one
# byte more than a 16-byte piece or a 128-byte slab), one tile, the last few-tile shape and the first
# beyond it, 64x64 and 128x128 tiles of both loaders, results cut inside a group of eight columns.
DOT_EDGE_CASES = [
    # m, n, k
    (1, 1, 1), (31, 33, 15), (33, 31, 16), (32, 32, 17), (65, 10, 129), (1, 75, 648), (512, 1023, 130),
    (513, 1025, 257), (700, 1001, 385), (1281, 2047, 255), (2050, 40, 64), (544, 1024, 192), (1700, 2048, 128),
    (49153, 40, 64), (96, 65, 1984),
]


@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32), ("fp8", torch.bfloat16)])
@pytest.mark.parametrize("mnk", DOT_EDGE_CASES)
def test_cartesian_dot_tile_edges(mnk, dtype, odt):
    m, n, k = mnk
    a0, a1 = gen(dtype, (m, k), 1400 + m, 1.0), gen(dtype, (n, k), 1500 + n, 1.0 if dtype == "i8" else k ** -0.5)
    # the result sits between guard values: nothing outside it may be written
    buf = torch.full((m * n + 512,), 77, dtype=odt, device=DEV)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), out=buf[256:256 + m * n].view(m, n))
    x, y = to_oracle(a0), to_oracle(a1)
    assert_parity(got, brute.matmul(x, y.T), what=str(mnk), slack=fp8_slack(x, y) if dtype == "fp8" else None)
    assert (buf[:256] == 77).all() and (buf[256 + m * n:] == 77).all()


# The tile shapes between one and two rounds of the chip, cut by both ends of the result: 64x128 (short K, and long K of few
# columns), 128x128 with two and three slab buffers, 256x256 that do not fill the chip, and unaligned rows in 128x64 and in
# 128x128 tiles of sixteen waves; K of one slab, a broken one and several.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("i8", torch.int32), ("fp8", torch.float32)])
@pytest.mark.parametrize("mnk", [(1500, 2101, 64), (1499, 2104, 448), (1501, 2100, 4160), (2201, 2310, 192), (4610, 262, 4608), (3601, 3590, 2112),
                                 (1103, 1073, 189), (1105, 1071, 1021), (1700, 2045, 131), (1701, 2047, 643)])
def test_cartesian_dot_tile_shapes(mnk, dtype, odt):
    m, n, k = mnk
    a0, a1 = gen(dtype, (m, k), 1410 + m, 1.0), gen(dtype, (n, k), 1510 + n, 1.0 if dtype == "i8" else k ** -0.5)
    buf = torch.full((m * n + 512,), 77, dtype=odt, device=DEV)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), out=buf[256:256 + m * n].view(m, n)).cpu().double()
    x, y = torch.from_numpy(np.asarray(to_oracle(a0), dtype=np.float64)), torch.from_numpy(np.asarray(to_oracle(a1), dtype=np.float64))
    want = x @ y.T
    if dtype == "i8":
        assert torch.equal(got, want)
    else:       # fp32 sums of k products, pairwise in parts, and one rounding to bfloat16; 8-bit floats: see fp8_slack
        slack = k * 2.0 ** -24 * (x.abs() @ y.abs().T) + (2.0 ** -8 * want.abs() if odt == torch.bfloat16 else 0)
        if dtype == "fp8":
            slack = slack + torch.from_numpy(fp8_slack(x.numpy(), y.numpy()))
        assert ((got - want).abs() <= slack).all()
    assert (buf[:256] == 77).all() and (buf[256 + m * n:] == 77).all()


# Many 128x128 tiles that a narrow result would leave half empty, and the first width at which it does not.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("i8", torch.int32)])
@pytest.mark.parametrize("mnk", [(20600, 64, 65), (64, 20600, 33), (20600, 65, 33), (65, 20600, 65), (1, 20600, 129), (20600, 1, 129)])
def test_cartesian_dot_narrow_results(mnk, dtype, odt):
    m, n, k = mnk
    a0, a1 = gen(dtype, (m, k), 1450 + m), gen(dtype, (n, k), 1550 + n)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), out_dtype=odt)
    assert_parity(got, brute.matmul(to_oracle(a0), to_oracle(a1).T), what=str(mnk))


def test_blocked_dot_of_narrow_blocks():
    a0, a1 = gen("bf16", (1300, 77), 1460), gen("bf16", (900, 77), 1560)
    for tile in ((40, 50), (64, 300), (300, 64), (65, 65)):
        got = gs.cartesian_dot_blocked(a0.to(DEV), a1.to(DEV), *tile, 77)
        assert_parity(got, brute.matmul(to_oracle(a0), to_oracle(a1).T), what=str(tile))


# Rows of fewer than 16 bytes (and of none) at any size: one tile, cut tiles, 64x64 and 128x128 ones, narrow results.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32), ("fp8", torch.bfloat16)])
@pytest.mark.parametrize("mnk", [(1, 1, 0), (130, 70, 0), (33, 65, 1), (129, 64, 7), (700, 333, 3), (1281, 2047, 5), (1664, 1280, 7), (30000, 3, 2),
                                 (2, 30001, 7)])
def test_cartesian_dot_short_rows(mnk, dtype, odt):
    m, n, k = mnk
    if dtype in ("i8", "fp8"):
        k = 2 * k + (1 if k > 1 else 0)
    a0, a1 = gen(dtype, (m, k), 1420 + m), gen(dtype, (n, k), 1520 + n)
    buf = torch.full((m * n + 512,), 77, dtype=odt, device=DEV)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), act=gs.GS_ACT_RELU, out=buf[256:256 + m * n].view(m, n))
    x, y = to_oracle(a0), to_oracle(a1)
    assert_parity(got, np.maximum(brute.matmul(x, y.T), 0), what=str(mnk), slack=fp8_slack(x, y) if dtype == "fp8" else None)
    assert (buf[:256] == 77).all() and (buf[256 + m * n:] == 77).all()


@pytest.mark.parametrize("dtype", ["bf16", "i8", "fp8"])
def test_blocked_dot_of_short_slices(dtype):
    """K slices of fewer than 16 bytes at every alignment, each added to the result of those in front."""
    m, n, k = 150, 139, 17
    a0, a1 = gen(dtype, (m, k), 1440), gen(dtype, (n, k), 1540)
    x, y = to_oracle(a0), to_oracle(a1)
    for tile_k in (3, 5, 7):
        got = gs.cartesian_dot_blocked(a0.to(DEV), a1.to(DEV), 70, 65, tile_k)
        assert_parity(got, brute.matmul(x, y.T), what=str(tile_k), slack=fp8_slack(x, y) if dtype == "fp8" else None)


def test_results_that_do_not_fit_the_memory():
    """4 TB of result: torch's own exception, as from any allocation."""
    a = torch.zeros((1 << 20, 16), dtype=torch.int8, device=DEV)
    with pytest.raises(torch.OutOfMemoryError):
        gs.cartesian_dot(a, a)
    assert gs.cartesian_dot(a[:1], a[:1]).item() == 0


def test_cartesian_dot_extreme_int8_values():
    """-128 * -128 * K stays exact in int32."""
    a0 = torch.full((40, 512), -128, dtype=torch.int8)
    a1 = torch.full((33, 512), -128, dtype=torch.int8)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV))
    assert (got.cpu() == 128 * 128 * 512).all()


def test_cartesian_dot_fp8_every_code():
    """All 254 finite e4m3 codes (subnormals, -0, +-448) as operands: the hardware must read the
    OCP encoding (bias 7, no infinities), not a variant with another bias or NaN placement."""
    codes = np.arange(256, dtype=np.uint8)
    codes[codes == 0x7F] = 0
    codes[codes == 0xFF] = 0x80
    a0 = torch.from_numpy(np.stack([np.roll(codes, r) for r in range(64)])).view(torch.float8_e4m3fn)
    a1 = gen("fp8", (40, 256), 1777, 0.5)
    for odt in (torch.float32, torch.bfloat16):
        got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), 1, 1, odt)
        assert_parity(got, brute.matmul(to_oracle(a0), to_oracle(a1).T), float_tol=1e-2, what=str(odt),
                      slack=fp8_slack(to_oracle(a0), to_oracle(a1)))
    # one code at a time against 1.0: the products are the decoded values themselves
    eye = torch.from_numpy(np.where(np.eye(256, dtype=bool), 0x38, 0).astype(np.uint8)).view(torch.float8_e4m3fn)
    row = torch.from_numpy(np.tile(codes, (3, 1))).view(torch.float8_e4m3fn)
    got = gs.cartesian_dot(row.to(DEV), eye.to(DEV), 1, 1, torch.float32).cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(got, np.tile(to_oracle(row)[0], (3, 1)))


def test_cartesian_dot_empty():
    a0 = torch.zeros((0, 16), dtype=torch.bfloat16, device=DEV)
    a1 = torch.zeros((8, 16), dtype=torch.bfloat16, device=DEV)
    assert gs.cartesian_dot(a0, a1).shape == (0, 8)

# Products large enough for the 256x256 (8 waves) and 128x128 tiles of the direct-to-LDS kernel,
# with ragged last tiles in both directions and results written 8, 4 and 1 columns per lane.
# Sampled rows of a0 (first, last, and both sides of tile boundaries) against every row of a1.
BIG_DOT_CASES = [
    # dtype, I, J, K, out dtype, relu
    ("bf16", 4100, 4104, 512, torch.bfloat16, True),     # 256x256, 8 columns per lane
    ("bf16", 4100, 4100, 512, torch.float32, False),     # 256x256, 4 columns per lane
    ("bf16", 4099, 4099, 144, torch.bfloat16, False),    # 256x256, one column per lane, short last slab
    ("i8", 4100, 4104, 512, torch.int32, True),          # 256x256 int8
    ("i8", 4100, 4099, 96, torch.int32, False),
    ("bf16", 1800, 1808, 264 * 2, torch.bfloat16, True), # 128x128, 8 columns per lane
    ("bf16", 1800, 1804, 264 * 2, torch.float32, False), # 128x128, 4 columns per lane
    ("i8", 1801, 1803, 160, torch.int32, False),         # 128x128, one column per lane
    ("i8", 1800, 1808, 512, torch.int32, True),
    ("fp8", 4100, 4104, 512, torch.bfloat16, True),      # 256x256, 8-bit floats
    ("fp8", 4100, 4099, 192, torch.float32, False),      # short last slab
    ("fp8", 1800, 1804, 576, torch.float32, False),      # 128x128
]


@pytest.mark.parametrize("case", BIG_DOT_CASES)
def test_cartesian_dot_large_tiles(case):
    dtype, I, J, K, odt, relu = case
    a0 = gen(dtype, (I, K), 1400 + I + K, 1.0)
    a1 = gen(dtype, (J, K), 1500 + J + K, 1.0 / np.sqrt(K) if dtype in ("bf16", "fp8") else 1.0)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), 1, 1, odt, gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE)
    rows = sorted({0, 1, 31, 32, 63, 64, 127, 128, 129, 255, 256, 257, 1023, 1024, I // 2, I - 130, I - 5, I - 2, I - 1}
                  | set(int(v) for v in np.random.default_rng(I + J).integers(0, I, 40)))
    idx = torch.tensor(rows)
    want = brute.matmul(to_oracle(a0[idx]), to_oracle(a1).T)
    if relu:
        want = np.maximum(want, 0)
    slack = fp8_slack(to_oracle(a0[idx]), to_oracle(a1)) if dtype == "fp8" else None
    assert_parity(got[idx.to(DEV)], want, what=str(case), slack=slack)


@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("o,n", [(256, 21), (128, 8), (192, 24)])
def test_conv2d_im2col_large_tiles_residual_relu(dtype, odt, o, n):
    """1x1 convolutions whose im2col product takes the 256x256 (O = 256, 65856 positions; O = 192
    with a ragged channel tile) and 128x128 (O = 128, 25088 positions) tiles, with the fused
    residual and ReLU and the (N,O,H',W') addressing of the stores; whole images."""
    cfg = synth.conv_layer(n, 64, 56, 56, o, 1, 1, 0, dtype, 8100 + o + n, gain=1.0)
    res = gen("i32" if dtype == "i8" else ("bf16" if odt == torch.bfloat16 else "f32"), (n, o, 56, 56), 8200 + o)
    got = gs.conv2d_im2col(cfg["x"].to(DEV), cfg["w"].to(DEV), (1, 1), (0, 0), residual=res.to(DEV),
                           act=gs.GS_ACT_RELU, out_dtype=odt)
    idx = torch.tensor([0, n // 2, n - 1])
    want = brute.conv2d(to_oracle(cfg["x"][idx]), to_oracle(cfg["w"]), (1, 1), (0, 0)) + to_oracle(res[idx])
    assert_parity(got[idx.to(DEV)], np.maximum(want, 0), what=f"{dtype} O={o} N={n}")


@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("c,k,o,h,w", [(32, 3, 300, 93, 95), (32, 1, 200, 211, 213), (16, 3, 64, 181, 183), (3, 1, 130, 121, 123)])
def test_conv2d_im2col_of_one_image_with_residual(c, k, o, h, w, dtype, odt):
    """One image of an odd plane: rows of the product are as long as the plane, of any alignment, and the residual
    is read eight values at a time wherever they lie (more than 512 tiles of 32x32, all loaders)."""
    cfg = synth.conv_layer(1, c, h, w, o, k, 1, k // 2, dtype, 8300 + o + h, gain=1.0)
    shape = (1, o, h, w)
    res = gen("i32" if dtype == "i8" else ("bf16" if odt == torch.bfloat16 else "f32"), shape, 8400 + o)
    got = gs.conv2d_im2col(cfg["x"].to(DEV), cfg["w"].to(DEV), (1, 1), (k // 2, k // 2), residual=res.to(DEV), act=gs.GS_ACT_RELU, out_dtype=odt)
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), padding=k // 2) + res.double()
    want = want.clamp_min(0).numpy()
    assert_parity(got, want.astype(np.int64) if dtype == "i8" else want, what=f"{dtype} {c} {k} {o}")


@pytest.mark.parametrize("mnk,dtype,odt", [((8191, 8201, 33), "bf16", torch.bfloat16), ((6001, 7003, 7), "bf16", torch.float32),
                                           ((7003, 6001, 64), "i8", torch.int32), ((6007, 6009, 65), "fp8", torch.bfloat16)])
def test_cartesian_dot_streams_odd_rows(mnk, dtype, odt):
    """Results above 128 MB in 32-bit values, whose stores pass the cache by, with rows of odd length."""
    m, n, k = mnk
    a0, a1 = gen(dtype, (m, k), 1470 + m), gen(dtype, (n, k), 1570 + n, k ** -0.5 if dtype != "i8" else 1.0)
    buf = torch.full((m * n + 512,), 77, dtype=odt, device=DEV)
    got = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), out=buf[256:256 + m * n].view(m, n))
    rows = torch.tensor(sorted({0, 1, 2, 127, 128, m // 2, m - 129, m - 2, m - 1}))
    x, y = to_oracle(a0[rows]), to_oracle(a1)
    assert_parity(got[rows.to(DEV)], brute.matmul(x, y.T), what=str(mnk), slack=fp8_slack(x, y) if dtype == "fp8" else None)
    assert (buf[:256] == 77).all() and (buf[256 + m * n:] == 77).all()
    # every row was written: a second product into the same buffer, cleared, is the same
    again = gs.cartesian_dot(a0.to(DEV), a1.to(DEV), out=torch.zeros((m, n), dtype=odt, device=DEV))
    assert torch.equal(got, again)



# ---------------------------------------------------------------------------------------------
# conv2d, both forms
# ---------------------------------------------------------------------------------------------

CONV_CASES = [
    # dtype, N, C, H, W, O, Kh, Kw, stride, pad, out dtype
    ("i8", 1, 3, 8, 8, 4, 3, 3, (1, 1), (0, 0), torch.int32),          # tiny configuration
    ("i8", 3, 40, 13, 13, 70, 3, 3, (1, 1), (1, 1), torch.int32),       # odd W, ragged C / O / M tails
    ("i8", 2, 64, 20, 18, 33, 3, 3, (2, 2), (1, 1), torch.int32),
    ("bf16", 2, 16, 20, 20, 24, 3, 3, (1, 1), (1, 1), torch.float32),
    ("bf16", 5, 32, 7, 7, 130, 3, 3, (1, 1), (1, 1), torch.bfloat16),   # 49-position planes: tiles span images
    ("bf16", 3, 24, 14, 14, 48, 1, 1, (2, 2), (0, 0), torch.float32),   # 1x1 stride-2 projection
    ("bf16", 2, 3, 30, 30, 16, 7, 7, (2, 2), (3, 3), torch.bfloat16),   # 7x7/2 pad 3, C = 3
    ("bf16", 1, 48, 9, 11, 20, 3, 2, (1, 2), (0, 1), torch.float32),    # non-square everything
    ("bf16", 2, 128, 12, 12, 64, 3, 3, (1, 1), (1, 1), torch.float32),  # several channel chunks
    # fewer channels than a 32-byte chunk: im2col rows formed in LDS (conv_smallc)
    ("bf16", 2, 1, 19, 23, 5, 3, 3, (1, 1), (1, 1), torch.float32),      # odd width: scalar staging
    ("bf16", 1, 3, 40, 272, 70, 5, 3, (2, 1), (2, 1), torch.bfloat16),   # two channel tiles, Wo > 128
    ("bf16", 2, 8, 16, 16, 64, 3, 3, (1, 1), (1, 1), torch.bfloat16),
    ("i8", 2, 16, 12, 32, 33, 3, 3, (1, 2), (1, 1), torch.int32),
    ("i8", 1, 3, 9, 9, 4, 1, 1, (1, 1), (0, 0), torch.int32),
    # few channels, windows a whole number of dwords apart: fragments read straight from the staged rows
    ("bf16", 2, 3, 33, 37, 20, 5, 8, (1, 2), (2, 3), torch.float32),     # 8-wide kernel rows
    ("bf16", 1, 2, 20, 300, 70, 3, 3, (2, 2), (1, 1), torch.bfloat16),   # Wo = 150, two channel tiles
    ("i8", 2, 4, 16, 40, 33, 3, 5, (1, 4), (1, 2), torch.int32),
    ("bf16", 3, 1, 9, 9, 4, 1, 1, (2, 2), (0, 0), torch.float32),
    # few output tiles, many chunks: the channel sum is split among workgroups (2 and 4 ways)
    ("bf16", 2, 256, 7, 7, 128, 3, 3, (1, 1), (1, 1), torch.bfloat16),
    ("bf16", 3, 128, 8, 8, 96, 3, 3, (1, 1), (1, 1), torch.float32),
    ("i8", 2, 512, 7, 7, 64, 3, 3, (1, 1), (1, 1), torch.int32),
    ("bf16", 2, 256, 14, 14, 64, 1, 1, (2, 2), (0, 0), torch.bfloat16),
    # odd widths: rows moved as runs of four pixels that cross row ends, unaligned loads
    ("bf16", 3, 64, 9, 7, 70, 3, 3, (1, 1), (1, 1), torch.bfloat16),
    ("bf16", 2, 64, 15, 13, 64, 3, 3, (2, 2), (1, 1), torch.float32),
    ("bf16", 7, 64, 7, 7, 32, 5, 5, (1, 1), (2, 2), torch.float32),
    ("bf16", 1, 64, 33, 45, 48, 3, 3, (1, 1), (0, 0), torch.bfloat16),
    ("i8", 2, 128, 7, 9, 33, 3, 3, (1, 1), (1, 1), torch.int32),
]


def conv_inputs(case):
    dtype, n, c, h, w, o, kh, kw, stride, pad, odt = case
    x = gen(dtype, (n, c, h, w), 1400 + c + h)
    wt = gen(dtype, (o, c, kh, kw), 1500 + o, 1.0 / np.sqrt(c * kh * kw) if dtype == "bf16" else 1.0)
    return x, wt


def conv_oracle(x, wt, stride, pad):
    xo, wo = to_oracle(x), to_oracle(wt)
    macs = x.shape[0] * wt.shape[0] * x.shape[2] * x.shape[3] * wt[0].numel()
    if macs <= 4_000_000:
        return pg.conv2d(ap.tensor(xo), ap.tensor(wo), stride, pad).materialize()
    return brute.conv2d(xo, wo, stride, pad)


@pytest.mark.parametrize("form", ["direct", "im2col"])
@pytest.mark.parametrize("case", CONV_CASES)
def test_conv2d(case, form):
    x, wt = conv_inputs(case)
    stride, pad, odt = case[8], case[9], case[10]
    fn = gs.conv2d_direct if form == "direct" else gs.conv2d_im2col
    got = fn(x.to(DEV), wt.to(DEV), stride, pad, out_dtype=odt)
    assert_parity(got, conv_oracle(x, wt, stride, pad), what=f"{form} {case}")


def _random_conv_cases(seed, count):
    """Seeded shapes across the kernels' branches: channel counts on and off the 16 / 32 multiples,
    widths that are and are not multiples of the producers' vectors, planes of 7..40, strides,
    paddings up to half the window, rectangular windows, few and many output channels."""
    r = np.random.default_rng(seed)
    cases = []
    while len(cases) < count:
        dtype = ("bf16", "i8")[int(r.integers(2))]
        n = int(r.integers(1, 6))
        c = int(r.choice([3, 8, 16, 24, 32, 48, 64, 96, 128, 160, 256]))
        h, w = int(r.integers(5, 41)), int(r.integers(5, 41))
        o = int(r.choice([1, 5, 32, 64, 70, 128, 200, 256]))
        kh, kw = [(1, 1), (3, 3), (3, 3), (3, 3), (5, 5), (3, 2), (2, 3)][int(r.integers(7))]
        stride = (int(r.integers(1, 3)), int(r.integers(1, 3)))
        pad = (int(r.integers(0, kh // 2 + 1)), int(r.integers(0, kw // 2 + 1)))
        if h + 2 * pad[0] < kh or w + 2 * pad[1] < kw or n * c * h * w * o * kh * kw > 3e9:
            continue
        odt = torch.int32 if dtype == "i8" else (torch.bfloat16, torch.float32)[int(r.integers(2))]
        cases.append((dtype, n, c, h, w, o, kh, kw, stride, pad, odt, bool(r.integers(2)), bool(r.integers(2))))
    return cases


@pytest.mark.parametrize("case", _random_conv_cases(20210905, 48))
def test_conv2d_random_shapes(case):
    """Both forms on seeded random shapes, with and without the fused residual and ReLU."""
    dtype, n, c, h, w, o, kh, kw, stride, pad, odt, with_res, relu = case
    x, wt = conv_inputs(case[:11])
    ho, wo_ = (h + 2 * pad[0] - kh) // stride[0] + 1, (w + 2 * pad[1] - kw) // stride[1] + 1
    res = None
    if with_res:
        res = (synth.uniform_int32((n, o, ho, wo_), -50000, 50000, 1701) if odt == torch.int32 else
               synth.normal_bf16((n, o, ho, wo_), 1.0, 1702) if odt == torch.bfloat16 else
               synth.normal_f32((n, o, ho, wo_), 1.0, 1703))
    want = brute.conv2d(to_oracle(x), to_oracle(wt), stride, pad)
    if res is not None:
        want = want + to_oracle(res)
    if relu:
        want = np.maximum(want, 0)
    act = gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE
    outs = []
    for fn in (gs.conv2d_direct, gs.conv2d_im2col):
        got = fn(x.to(DEV), wt.to(DEV), stride, pad, residual=None if res is None else res.to(DEV), act=act, out_dtype=odt)
        assert_parity(got, want, what=f"{fn.__name__} {case}")
        outs.append(got)
    if dtype == "i8":
        assert torch.equal(outs[0], outs[1])


def test_conv2d_direct_equals_im2col_bitwise_int8():
    """The rewrite of Sec. 5.3 preserves the result: both forms agree bit for bit on integers."""
    case = ("i8", 4, 32, 17, 19, 40, 3, 3, (1, 1), (1, 1), torch.int32)
    x, wt = conv_inputs(case)
    a = gs.conv2d_direct(x.to(DEV), wt.to(DEV), (1, 1), (1, 1))
    b = gs.conv2d_im2col(x.to(DEV), wt.to(DEV), (1, 1), (1, 1))
    assert torch.equal(a, b)
    assert_parity(a, conv_oracle(x, wt, (1, 1), (1, 1)))


@pytest.mark.parametrize("form", ["direct", "im2col"])
@pytest.mark.parametrize("hw", [10, 12, 9])    # planes of 100, 144, 81 positions: 4, 8, 1 results per store
@pytest.mark.parametrize("c", [32, 128])     # 128 channels: enough chunks for the producer / consumer kernel
@pytest.mark.parametrize("dtype,odt", [("i8", torch.int32), ("bf16", torch.bfloat16), ("bf16", torch.float32)])
def test_conv2d_residual_relu(form, dtype, odt, hw, c):
    case = (dtype, 2, c, hw, hw, 40, 3, 3, (1, 1), (1, 1), odt)
    x, wt = conv_inputs(case)
    if odt == torch.int32:
        res = synth.uniform_int32((2, 40, hw, hw), -50000, 50000, 1601)
    elif odt == torch.bfloat16:
        res = synth.normal_bf16((2, 40, hw, hw), 1.0, 1602)
    else:
        res = synth.normal_f32((2, 40, hw, hw), 1.0, 1603)
    fn = gs.conv2d_direct if form == "direct" else gs.conv2d_im2col
    got = fn(x.to(DEV), wt.to(DEV), (1, 1), (1, 1), residual=res.to(DEV), act=gs.GS_ACT_RELU, out_dtype=odt)
    conv = pg.conv2d(ap.tensor(to_oracle(x)), ap.tensor(to_oracle(wt)), (1, 1), (1, 1))
    prog = ap.compute(ap.relu, pg.add(conv, ap.access(ap.tensor(to_oracle(res)), 4)))
    assert_parity(got, prog.materialize(), what=f"{form} {dtype} residual+relu")


@pytest.mark.parametrize("dtype,odt,hw", [("bf16", torch.bfloat16, 7), ("bf16", torch.float32, 8), ("i8", torch.int32, 8)])
def test_conv2d_split_channel_sum_residual_relu(dtype, odt, hw):
    """Split channel sums are combined with the residual and ReLU in a second kernel; and the
    packed entry point gives the same result with and without the scratch that enables the split."""
    c = 512 if dtype == "i8" else 256
    case = (dtype, 2, c, hw, hw, 128, 3, 3, (1, 1), (1, 1), odt)
    x, wt = conv_inputs(case)
    shape = (2, 128, hw, hw)
    res = {torch.int32: lambda: synth.uniform_int32(shape, -50000, 50000, 1611),
           torch.bfloat16: lambda: synth.normal_bf16(shape, 1.0, 1612),
           torch.float32: lambda: synth.normal_f32(shape, 1.0, 1613)}[odt]()
    xd, wd, rd = x.to(DEV), wt.to(DEV), res.to(DEV)
    assert gs.conv2d_workspace(xd, wd, (1, 1), (1, 1)) > gs.conv2d_pack_weights(wd).numel()   # scratch is asked for
    got = gs.conv2d_direct(xd, wd, (1, 1), (1, 1), residual=rd, act=gs.GS_ACT_RELU, out_dtype=odt)
    want = np.maximum(brute.conv2d(to_oracle(x), to_oracle(wt), (1, 1), (1, 1)) + to_oracle(res), 0)
    assert_parity(got, want, what="split")
    plain = gs.conv2d_direct_packed(xd, wd, gs.conv2d_pack_weights(wd), (1, 1), (1, 1), residual=rd,
                                    act=gs.GS_ACT_RELU, out_dtype=odt)
    assert_parity(plain, want, what="unsplit")


@pytest.mark.parametrize("odt", [torch.bfloat16, torch.float32])
def test_conv2d_few_channels_residual_relu(odt):
    case = ("bf16", 2, 3, 20, 24, 40, 7, 7, (2, 2), (3, 3), odt)
    x, wt = conv_inputs(case)
    shape = (2, 40, 10, 12)
    res = synth.normal_bf16(shape, 1.0, 1621) if odt == torch.bfloat16 else synth.normal_f32(shape, 1.0, 1622)
    got = gs.conv2d_direct(x.to(DEV), wt.to(DEV), (2, 2), (3, 3), residual=res.to(DEV), act=gs.GS_ACT_RELU, out_dtype=odt)
    want = np.maximum(brute.conv2d(to_oracle(x), to_oracle(wt), (2, 2), (3, 3)) + to_oracle(res), 0)
    assert_parity(got, want, what="few channels, residual + relu")


def _random_few_channel_cases(seed, count):
    """Seeded shapes for the few-channel kernel: 1..4 channels (8 for int8), windows of 3..7, rows
    that are and are not whole 16-byte vectors, output heights on and off the multiples of four
    (a task is four output rows), output widths on and off the multiples of 4 and 8 and past 128."""
    r = np.random.default_rng(seed)
    cases = []
    while len(cases) < count:
        dtype = ("bf16", "bf16", "i8")[int(r.integers(3))]
        n = int(r.integers(1, 4))
        c = int(r.integers(1, 5)) if dtype == "bf16" else int(r.choice([1, 3, 4, 8]))
        h = int(r.integers(7, 60))
        w = int(r.choice([8, 16, 24, 31, 32, 40, 50, 56, 64, 100, 160, 272]))
        o = int(r.choice([5, 32, 64, 70]))
        k = int(r.choice([3, 5, 7]))
        stride = (int(r.integers(1, 3)), int(r.integers(1, 3)))
        pad = (int(r.integers(0, k // 2 + 1)), int(r.integers(0, k // 2 + 1)))
        if h + 2 * pad[0] < k or w + 2 * pad[1] < k:
            continue
        odt = torch.int32 if dtype == "i8" else (torch.bfloat16, torch.float32)[int(r.integers(2))]
        cases.append((dtype, n, c, h, w, o, k, k, stride, pad, odt, bool(r.integers(2)), bool(r.integers(2))))
    return cases


@pytest.mark.parametrize("case", _random_few_channel_cases(20210908, 40))
def test_conv2d_few_channels_random_shapes(case):
    dtype, n, c, h, w, o, kh, kw, stride, pad, odt, with_res, relu = case
    x, wt = conv_inputs(case[:11])
    ho, wo_ = (h + 2 * pad[0] - kh) // stride[0] + 1, (w + 2 * pad[1] - kw) // stride[1] + 1
    res = None
    if with_res:
        res = (synth.uniform_int32((n, o, ho, wo_), -50000, 50000, 1711) if odt == torch.int32 else
               synth.normal_bf16((n, o, ho, wo_), 1.0, 1712) if odt == torch.bfloat16 else
               synth.normal_f32((n, o, ho, wo_), 1.0, 1713))
    want = brute.conv2d(to_oracle(x), to_oracle(wt), stride, pad)
    if res is not None:
        want = want + to_oracle(res)
    if relu:
        want = np.maximum(want, 0)
    got = gs.conv2d_direct(x.to(DEV), wt.to(DEV), stride, pad, residual=None if res is None else res.to(DEV),
                           act=gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE, out_dtype=odt)
    assert_parity(got, want, what=str(case))


# Edges of conv_tile_kernel in the instances that the cost model picks: planes of which a tile holds several or
# none, whose ends cut a 16-byte store; channel counts whose chunks the groups of a channel sum divide, do not
# divide, or do not all get; channel tiles cut short; rows too short for it, which take another kernel.
# test_conv_tile_instances takes every instance.
CONV_TILE_CASES = [
    # k, n, c (32-byte chunks), h, w, o, stride, pad
    (3, 1, 1, 1, 4, 1, 1, 1), (3, 3, 2, 4, 5, 31, 1, 1), (3, 70, 3, 2, 4, 33, 1, 1), (3, 1, 4, 56, 56, 64, 1, 1), (3, 2, 5, 9, 11, 65, 2, 0),
    (3, 5, 9, 7, 7, 96, 1, 1), (3, 1, 33, 7, 7, 40, 1, 1), (3, 21, 8, 7, 7, 130, 1, 1), (3, 2, 7, 14, 14, 64, 2, 1), (3, 9, 4, 28, 28, 128, 1, 1),
    (3, 6, 4, 28, 28, 72, 2, 1), (3, 33, 2, 31, 29, 17, 1, 0), (3, 16, 4, 56, 56, 64, 1, 1), (3, 13, 3, 41, 52, 100, 1, 1), (3, 40, 2, 40, 44, 128, 2, 1),
    (3, 2, 6, 3, 112, 16, 1, 1), (3, 1, 2, 112, 3, 48, 1, 1), (3, 3, 2, 20, 18, 32, 1, 3), (3, 2, 2, 60, 62, 200, 2, 2), (3, 64, 1, 16, 16, 65, 1, 1),
    (5, 1, 1, 5, 5, 1, 1, 0), (5, 2, 3, 4, 6, 33, 1, 2), (5, 30, 2, 7, 7, 70, 1, 2), (5, 12, 4, 28, 30, 128, 1, 2), (5, 9, 2, 31, 33, 40, 2, 2),
    (5, 1, 9, 14, 14, 65, 1, 2), (5, 3, 1, 112, 4, 16, 2, 1),
    (1, 1, 4, 1, 4, 1, 1, 0), (1, 3, 4, 5, 5, 33, 2, 0), (1, 50, 8, 7, 7, 64, 1, 0), (1, 2, 12, 14, 15, 130, 2, 0), (1, 64, 4, 28, 28, 128, 2, 0),
    (1, 1, 4, 9, 94, 16, 1, 0), (1, 2, 4, 7, 101, 33, 1, 0), (1, 2, 8, 13, 83, 40, 2, 0), (1, 8, 4, 56, 56, 64, 1, 0), (1, 5, 20, 29, 31, 31, 1, 0), (1, 32, 8, 28, 28, 256, 2, 0), (1, 1, 64, 7, 7, 512, 2, 0),
]


@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("case", CONV_TILE_CASES)
def test_conv2d_tiles(case, dtype, odt):
    k, n, chunks, h, w, o, s, p = case
    c = chunks * (32 if dtype == "i8" else 16)
    cfg = synth.conv_layer(n, c, h, w, o, k, s, p, dtype, 8500 + h + 3 * o)
    x, wt = cfg["x"].to(DEV), cfg["w"].to(DEV)
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p)
    res = gen("i32" if dtype == "i8" else ("bf16" if odt == torch.bfloat16 else "f32"), tuple(want.shape), 8600 + o)
    packed = gs.conv2d_pack_weights(wt, for_input=(x, (s, s), (p, p)))
    # results sit between guard values: nothing outside them may be written
    buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
    out = buf[256:256 + want.numel()].view(want.shape)
    for residual, act in ((None, gs.GS_ACT_NONE), (res, gs.GS_ACT_RELU)):
        ref = want if residual is None else (want + res.double()).clamp_min(0)
        ref = ref.numpy().astype(np.int64) if dtype == "i8" else ref.numpy()
        how = dict(act=act, out=out, residual=None if residual is None else residual.to(DEV))
        gs.conv2d_direct_packed(x, wt, packed, (s, s), (p, p), **how)
        assert_parity(out, ref, what=f"{dtype} {case}")
        if k == 1:      # the listing's own weights
            out.fill_(55)
            gs.conv2d_im2col(x, wt, (s, s), (p, p), **how)
            assert_parity(out, ref, what=f"{dtype} {case} im2col")
        assert (buf[:256] == 77).all() and (buf[256 + want.numel():] == 77).all()


# Every built instance of conv_tile_kernel, on the smallest layer that the planner puts there: workgroup shape,
# window, stride, interleaved blocks (widths that are multiples of four, two, or neither), patch items per thread (up
# to rows of some 2000 pixels), one chunk per group or several, packed weights or the listing's own.
@pytest.mark.parametrize("shape", tile_instances.SHAPES)
@pytest.mark.parametrize("k,natural", [(1, False), (1, True), (3, False), (5, False)])
@pytest.mark.parametrize("dtype", ["bf16", "i8"])
def test_conv_tile_instances(dtype, k, natural, shape):
    layers = tile_instances.layers(dtype, k, natural, shape)
    assert set(layers) == tile_instances.built(dtype, k, shape)
    for (s, *instance), (way, (n, c, h, w, o, p)) in layers.items():
        cfg = synth.conv_layer(n, c, h, w, o, k, s, p, dtype, 9100 + h + w)
        x, wt = cfg["x"].to(DEV), cfg["w"].to(DEV)
        want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p)
        packed = gs.conv2d_pack_weights(wt, for_input=(x, (s, s), (p, p)))
        for odt, with_res in ((torch.int32, False), (torch.int32, True)) if dtype == "i8" else ((torch.bfloat16, False), (torch.float32, True)):
            res = gen("i32" if dtype == "i8" else "f32", tuple(want.shape), 9200 + w) if with_res else None
            buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
            out = buf[256:256 + want.numel()].view(want.shape)
            rd = None if res is None else res.to(DEV)
            st, plan = tile_instances.call(gs.make_ap(x, 1), gs.make_ap(wt, 1), s, p, None if rd is None else gs.make_ap(rd, 4),
                                           gs.GS_ACT_RELU if with_res else gs.GS_ACT_NONE, gs.make_ap(out, 4),
                                           None if natural else packed.data_ptr(), way, gs._stream(x))
            assert (st, plan[:4]) == (gs.GS_OK, (shape, *instance))
            ref = want if res is None else (want + res.double()).clamp_min(0)
            assert_parity(out, ref.numpy().astype(np.int64) if dtype == "i8" else ref.numpy(), what=f"{plan} {(n, c, h, w)} stride {s}")
            assert (buf[:256] == 77).all() and (buf[256 + want.numel():] == 77).all()


# Depth-wise windows on the matrix units: tiles beside and above each other, cut at both ends, one and several planes to a task, rows
# that end inside a piece, padding and none; infinities and NaN, which reach only the results whose windows hold them.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("n,c,h,w,k,p", [(3, 100, 63, 62, 3, 1), (40, 90, 15, 31, 3, 1), (9, 130, 31, 29, 3, 0), (2, 50, 95, 111, 5, 2), (25, 80, 27, 16, 5, 2),
                                         (7, 64, 29, 32, 5, 0), (3, 64, 44, 100, 5, 1), (4, 33, 112, 112, 5, 2), (20, 90, 33, 62, 5, 2), (1, 40, 93, 125, 3, 1)])
def test_depthwise_tiles(n, c, h, w, k, p, dtype, odt):
    x, wt = gen(dtype, (n, c, h, w), 9900 + h), gen(dtype, (c, k, k), 9950 + w, 1.0 / k)
    if dtype == "bf16":
        x[0, 0, 0, 0], x[-1, -1, -1, -1], x[0, 1, h // 2, w // 2], x[n // 2, 2, h - 1, 7] = float("inf"), float("-inf"), float("nan"), float("inf")
    want = torch.nn.functional.conv2d(x.double(), wt.double()[:, None], padding=p, groups=c)
    buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
    out = buf[256:256 + want.numel()].view(want.shape)
    for act in (gs.GS_ACT_NONE, gs.GS_ACT_RELU):
        gs.depthwise_conv2d(x.to(DEV), wt.to(DEV), (1, 1), (p, p), act=act, out=out)
        got, ref = out.cpu().double(), want if act == gs.GS_ACT_NONE else torch.where(want > 0, want, torch.zeros_like(want))
        if dtype == "i8":
            assert torch.equal(got, ref)
        else:
            # k k products and sums in fp32 (2^-24 each), one rounding to bfloat16
            mag = torch.nn.functional.conv2d(torch.nan_to_num(x.double(), posinf=0, neginf=0).abs(), wt.double().abs()[:, None], padding=p, groups=c)
            slack = k * k * 2.0 ** -24 * mag + (2.0 ** -8 * torch.nan_to_num(ref, posinf=0, neginf=0).abs() if odt == torch.bfloat16 else 0)
            fine = torch.isfinite(ref)
            assert torch.equal(torch.nan_to_num(got[~fine], nan=7.0), torch.nan_to_num(ref[~fine], nan=7.0))
            assert torch.isfinite(got[fine]).all() and ((got - ref).abs()[fine] <= slack[fine]).all()
        assert (buf[:256] == 77).all() and (buf[256 + want.numel():] == 77).all()


# What a window does not hold does not change its result by a bit, infinities and NaN included (the matrix units multiply
# them with zeros; finite values round as they do without them).
@pytest.mark.parametrize("odt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n,c,h,w,k,p", [(3, 100, 63, 62, 3, 1), (2, 50, 95, 111, 5, 2), (25, 80, 27, 16, 5, 2), (7, 64, 29, 32, 5, 0)])
def test_depthwise_tiles_windows_stay_apart(n, c, h, w, k, p, odt):
    x, wt = gen("bf16", (n, c, h, w), 9910 + h), gen("bf16", (c, k, k), 9955 + w, 1.0 / k)
    odd = torch.zeros(x.shape, dtype=torch.bool)
    odd[:, :, ::9, ::17] = True
    y = torch.where(odd, torch.tensor([float("inf"), float("-inf"), float("nan")], dtype=x.dtype)[torch.arange(x.numel()).view(x.shape) % 3], x)
    held = torch.nn.functional.conv2d(odd.float(), torch.ones(c, 1, k, k), padding=p, groups=c) > 0
    a, b = (gs.depthwise_conv2d(t.to(DEV), wt.to(DEV), (1, 1), (p, p), out_dtype=odt).cpu() for t in (x, y))
    assert torch.isfinite(a).all() and torch.equal(a[~held], b[~held])
    assert not torch.isfinite(b[held]).any()


# 5x5 windows at stride 2: strips cut by the row's end, odd planes, several planes to a task and bands of one.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("n,c,h,w,p", [(1, 1, 5, 5, 0), (3, 17, 12, 17, 2), (2, 9, 31, 46, 1), (20, 24, 8, 16, 2), (1, 3, 203, 301, 2)])
def test_depthwise_5x5_stride_2(n, c, h, w, p, dtype, odt):
    x, wt = gen(dtype, (n, c, h, w), 9960 + h), gen(dtype, (c, 5, 5), 9970 + w, 0.2)
    want = torch.nn.functional.conv2d(x.double(), wt.double()[:, None], padding=p, stride=2, groups=c).numpy()
    got = gs.depthwise_conv2d(x.to(DEV), wt.to(DEV), (2, 2), (p, p), out_dtype=odt)
    assert_parity(got, want.astype(np.int64) if dtype == "i8" else want, what=str((n, c, h, w, p)))


# Rows of any length in 16-byte vectors (reduce_rows_any_kernel): the rows' first and last vectors shared in every phase,
# each lane group, a workgroup per row (and the numbers of rows from which it is a wavefront), several rounds of rows, the tensor
# ending inside a vector; lowest values at the rows' ends, which a neighbour's value must not replace.
@pytest.mark.parametrize("op", [gs.GS_SUM, gs.GS_MAX])
@pytest.mark.parametrize("dtype,odt", [("f32", None), ("i32", None), ("i8", None), ("bf16", torch.bfloat16), ("bf16", torch.float32)])
@pytest.mark.parametrize("rows,cols", [(16411, 67), (8193, 129), (4099, 259), (2053, 517), (1031, 1029), (130, 2403), (17, 9001), (3, 40003), (40011, 131),
                                       (999, 1125), (1000, 1125), (999, 4497), (1000, 4497), (1999, 6689), (2000, 6689), (5, 2049), (430, 2399),
                                       (1599, 2301), (1600, 2301), (1599, 2305), (12337, 85), (34999, 87), (35000, 87)])
def test_reduce_rows_of_any_length(rows, cols, dtype, odt, op):
    x = gen(dtype, (rows, cols), 9800 + cols)
    if op == gs.GS_MAX:
        x[1::3] = LOWEST[dtype] if dtype in ("i8", "i32") else float("-inf")
    got = gs.reduce(x.to(DEV), 1, op, out_dtype=odt)
    if op == gs.GS_MAX:
        assert torch.equal(got.cpu().double(), x.double().amax(1))
    elif dtype in ("i8", "i32"):
        assert torch.equal(got.cpu().long(), x.long().sum(1))
    else:       # pairwise sums: 2^-24 per level of some log2(cols) + 3 of the magnitudes, then the store's rounding
        want = x.double().sum(1)
        slack = (math.log2(cols) + 3) * 2.0 ** -24 * x.double().abs().sum(1) + (2.0 ** -8 if odt == torch.bfloat16 else 0) * want.abs()
        assert ((got.cpu().double() - want).abs() <= slack).all()


# Small images in one launch (conv_images_kernel), both forms: images and weight rows shorter than a 16-byte piece, several images
# in a tile, tiles cut by the end, windows that reach past the image on all sides, the longest contraction.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("n,c,h,w,o,kh,kw,s,p", [
    (1, 1, 1, 1, 1, 1, 1, 1, 0), (1, 1, 2, 3, 33, 1, 1, 1, 0), (3, 1, 1, 1, 5, 1, 1, 1, 1), (1, 3, 8, 8, 4, 3, 3, 1, 0), (40, 2, 3, 5, 7, 2, 3, 1, 1), (2, 7, 9, 4, 32, 5, 5, 2, 2),
    (1, 13, 31, 32, 48, 3, 3, 1, 1), (4, 14, 32, 20, 26, 1, 1, 1, 1), (1, 2, 190, 11, 9, 7, 3, 3, 3), (2, 15, 12, 12, 64, 5, 5, 1, 2), (1, 5, 4, 192, 40, 4, 9, 2, 4),
    (3, 12, 6, 6, 31, 6, 6, 1, 0), (64, 1, 4, 4, 65, 4, 4, 1, 3), (2, 4, 7, 7, 16, 9, 9, 1, 1), (1, 1, 40, 40, 8, 22, 23, 1, 5)])
def test_conv2d_small_images(n, c, h, w, o, kh, kw, s, p, dtype, odt):
    x, wt = gen(dtype, (n, c, h, w), 9500 + h), gen(dtype, (o, c, kh, kw), 9600 + o, (c * kh * kw) ** -0.5)
    want = torch.nn.functional.conv2d(x.double(), wt.double(), stride=s, padding=p)
    res = gen("i32" if dtype == "i8" else ("bf16" if odt == torch.bfloat16 else "f32"), tuple(want.shape), 9700 + o)
    xd, wd = x.to(DEV), wt.to(DEV)
    buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
    out = buf[256:256 + want.numel()].view(want.shape)
    for fn in (gs.conv2d_direct, gs.conv2d_im2col):
        for residual, act in ((None, gs.GS_ACT_NONE), (res, gs.GS_ACT_RELU)):
            ref = want if residual is None else (want + res.double()).clamp_min(0)
            ref = ref.numpy().astype(np.int64) if dtype == "i8" else ref.numpy()
            fn(xd, wd, (s, s), (p, p), act=act, out=out, residual=None if residual is None else residual.to(DEV))
            assert_parity(out, ref, what=fn.__name__)
            assert (buf[:256] == 77).all() and (buf[256 + want.numel():] == 77).all()


# The same instances with channels that do not fill the last chunk: one short, one more than the chunk before, and 1x1
# steps that lack whole chunks.  Infinities in the last channel and in the channels that follow it in memory.
@pytest.mark.parametrize("shape", tile_instances.SHAPES[1:])
@pytest.mark.parametrize("k,natural", [(1, False), (1, True), (3, False), (5, False)])
@pytest.mark.parametrize("dtype", ["bf16", "i8"])
def test_conv_tile_instances_odd_channels(dtype, k, natural, shape):
    unit = 32 if dtype == "i8" else 16
    reached = set()
    for (s, *_rest), (way, (n, c, h, w, o, p)) in tile_instances.layers(dtype, k, natural, shape).items():
        for less in ((unit // 2, 5 * unit // 2, 3 * unit) if natural else (1, unit - 1, unit + 3)):
            cfg = synth.conv_layer(n, c - less, h, w, o, k, s, p, dtype, 9300 + h + w)
            if dtype == "bf16":
                cfg["x"][0, -1, 0, 0] = float("inf")
                cfg["x"][n - 1, 0, h - 1, w - 1] = float("-inf")
            x, wt = cfg["x"].to(DEV), cfg["w"].to(DEV)
            want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p)
            packed = gs.conv2d_pack_weights(wt, for_input=(x, (s, s), (p, p)))
            odt = torch.int32 if dtype == "i8" else torch.bfloat16
            buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
            out = buf[256:256 + want.numel()].view(want.shape)
            st, plan = tile_instances.call(gs.make_ap(x, 1), gs.make_ap(wt, 1), s, p, None, gs.GS_ACT_NONE, gs.make_ap(out, 4),
                                           None if natural else packed.data_ptr(), way, gs._stream(x))
            if _rest[2] and st == gs.GS_ERR_UNSUPPORTED:
                continue                # built for several chunks only, whose three patch buffers do not fit
            assert (st, plan[0], plan[3]) == (gs.GS_OK, shape, 0)
            reached.add((s, *plan[1:4]))
            got = out.double().cpu()
            same = torch.isfinite(want)
            assert torch.equal(torch.nan_to_num(got[~same], nan=7.0), torch.nan_to_num(want[~same], nan=7.0))
            assert torch.isfinite(got[same]).all()
            got, want = torch.where(same, got, 0.0).numpy(), torch.where(same, want, 0.0).numpy()
            if dtype == "i8":
                assert np.array_equal(got, want), f"{plan} {(n, c - less, h, w)} stride {s}"
            else:       # one rounding to bfloat16
                assert np.abs(got - want).max() <= 2.0 ** -8 * np.abs(want).max(), f"{plan} {(n, c - less, h, w)} stride {s}"
            assert (buf[:256] == 77).all() and (buf[256 + want.size:] == 77).all()
    assert reached == {i for i in tile_instances.built(dtype, k, shape) if not i[3]}


# A 3x3 convolution and a 1x1 projection of the same input, both at stride 2, in one launch: every instance, and through the
# entry point also what no instance takes (odd channels, bytes, other windows).
@pytest.mark.parametrize("shape", tile_instances.SHAPES)
def test_conv_tile_instances_with_projection(shape):
    reached = set()
    for (s, *_rest), (way, (n, c, h, w, o, p)) in tile_instances.layers("bf16", 3, False, shape).items():
        if s == 1:
            continue
        cfg, proj = (synth.conv_layer(n, c, h, w, o, k, s, p, "bf16", 9380 + h + w) for k in (3, 1))
        x, w3, w1 = cfg["x"].to(DEV), cfg["w"].to(DEV), proj["w"].to(DEV)
        wants = [torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p).clamp_min(0),
                 torch.nn.functional.conv2d(cfg["x"].double(), proj["w"].double(), stride=s)]
        packed, packed1 = gs.conv2d_pack_weights(w3), gs.conv2d_pack_weights(w1)
        numel = wants[0].numel()
        buf = torch.full((2, numel + 512), 77, dtype=torch.bfloat16, device=DEV)
        outs = [b[256:256 + numel].view(wants[0].shape) for b in buf]
        st, plan = tile_instances.call_with_projection(gs.make_ap(x, 1), gs.make_ap(w3, 1), s, p, gs.GS_ACT_RELU, gs.make_ap(outs[0], 4),
                                                       packed.data_ptr(), gs.make_ap(w1, 1), gs.make_ap(outs[1], 4), packed1.data_ptr(),
                                                       way, gs._stream(x))
        assert (st, plan[0]) == (gs.GS_OK, shape)
        reached.add((s, *plan[1:4]))
        for out, want in zip(outs, wants):      # one rounding to bfloat16
            assert (out.double().cpu() - want).abs().max() <= 2.0 ** -8 * want.abs().max(), f"{plan} {(n, c, h, w)}"
        assert (buf[:, :256] == 77).all() and (buf[:, 256 + numel:] == 77).all()
    assert reached == {i for i in tile_instances.built("bf16", 3, shape) if i[0] == 2}


@pytest.mark.parametrize("n,c,h,w,o,k,s,dtype,odt", [
    (1, 64, 57, 56, 128, 3, 2, "bf16", torch.bfloat16), (5, 32, 14, 15, 33, 3, 2, "bf16", torch.float32), (2, 24, 9, 9, 40, 3, 2, "bf16", torch.bfloat16),
    (3, 64, 28, 28, 64, 3, 2, "i8", torch.int32), (2, 32, 12, 12, 32, 3, 1, "bf16", torch.bfloat16), (2, 32, 12, 12, 32, 5, 2, "bf16", torch.bfloat16)])
def test_conv2d_with_projection(n, c, h, w, o, k, s, dtype, odt):
    cfg, proj = (synth.conv_layer(n, c, h, w, o, k_, s, k_ // 2, dtype, 9390 + c + o) for k_ in (k, 1))
    x, wk, w1 = cfg["x"].to(DEV), cfg["w"].to(DEV), proj["w"].to(DEV)
    wants = [torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=k // 2).clamp_min(0).numpy(),
             torch.nn.functional.conv2d(cfg["x"].double(), proj["w"].double(), stride=s).numpy()]
    outs = [torch.full(want.shape, 77, dtype=odt, device=DEV) for want in wants]
    packed, packed1 = gs.conv2d_pack_weights(wk, for_input=(x, (s, s), (k // 2, k // 2))), gs.conv2d_pack_weights(w1, for_input=(x, (s, s), (0, 0)))
    gs.conv2d_direct_packed_with_projection(x, wk, packed, w1, packed1, (s, s), (k // 2, k // 2), gs.GS_ACT_RELU, *outs)
    for out, want in zip(outs, wants):
        assert_parity(out, want.astype(np.int64) if dtype == "i8" else want)
    with pytest.raises(gs.GlensideError):
        gs.conv2d_direct_packed_with_projection(x, wk, packed, w1[:, 1:].contiguous(), packed1, (s, s), (k // 2, k // 2), gs.GS_ACT_RELU, *outs)


# Half a chunk of channels and more: conv_tile_kernel, or im2col rows where results are few; packed and with weights that come
# with the call.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("i8", torch.int32)])
@pytest.mark.parametrize("c,n,h,w,o,k,s,p", [(8, 3, 21, 40, 33, 3, 1, 1), (15, 40, 14, 30, 65, 3, 2, 1), (9, 2, 60, 71, 70, 5, 1, 2), (11, 30, 12, 53, 16, 1, 1, 0), (13, 9, 25, 70, 96, 1, 2, 0),
                                             (15, 1, 3, 4, 1, 3, 1, 1), (12, 5, 90, 91, 40, 5, 2, 0), (7, 4, 30, 30, 40, 3, 1, 1)])
def test_conv2d_half_a_chunk_of_channels(c, n, h, w, o, k, s, p, dtype, odt):
    cfg = synth.conv_layer(n, 2 * c if dtype == "i8" else c, h, w, o, k, s, p, dtype, 9350 + c + o)
    x, wt = cfg["x"].to(DEV), cfg["w"].to(DEV)
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), stride=s, padding=p).numpy()
    want = want.astype(np.int64) if dtype == "i8" else want
    ws, packed = (torch.full((gs.conv2d_workspace(x, wt, (s, s), (p, p)),), 0x5a, dtype=torch.uint8, device=DEV) for _ in range(2))
    gs.conv2d_pack_weights(wt, packed)
    assert_parity(gs.conv2d_direct_packed(x, wt, packed, (s, s), (p, p), out_dtype=odt), want, what="packed")
    assert_parity(gs.conv2d_direct(x, wt, (s, s), (p, p), out_dtype=odt, workspace=ws), want, what="packed by the call")
    assert torch.equal(ws, packed)              # (no scratch: their channel sums are not split)


@pytest.mark.parametrize("k,c,dtype", [(3, 33, "bf16"), (5, 50, "i8"), (1, 40, "bf16")])
def test_conv2d_odd_channels_in_the_least_workspace(k, c, dtype):
    """The blocked copy of the weights is optional where channels do not fill a chunk: a workspace without room for it
    is taken, and gives the same result."""
    cfg = synth.conv_layer(2, c, 9, 11, 40, k, 1, k // 2, dtype, 9400 + c)
    x, wt, pad = cfg["x"].to(DEV), cfg["w"].to(DEV), (k // 2, k // 2)
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), padding=k // 2).numpy()
    want = want.astype(np.int64) if dtype == "i8" else want
    step = 32 if dtype == "i8" else 16
    front = 40 * k * k * -(-c // step) * 32
    least = -(-front // 256) * 256 + 256
    full = gs.conv2d_pack_weights(wt).numel()
    assert least < full
    for size in (least, full - 1, full):
        packed = gs.conv2d_pack_weights(wt, packed=torch.empty(size, dtype=torch.uint8, device=DEV))
        assert_parity(gs.conv2d_direct_packed(x, wt, packed, (1, 1), pad), want, what=f"packed in {size} bytes")
    with pytest.raises(Exception):
        gs.conv2d_pack_weights(wt, packed=torch.empty(least - 1, dtype=torch.uint8, device=DEV))


# Packing and convolving may be told of buffers of different sizes, each large enough, in either order; what lies in a
# buffer from before is never taken for a copy of the weights.
@pytest.mark.parametrize("k,c,dtype", [(3, 33, "bf16"), (5, 50, "i8"), (1, 40, "bf16"), (1, 200, "i8"), (3, 11, "bf16"), (5, 20, "i8"), (1, 12, "bf16")])
def test_conv2d_packed_and_read_in_other_sizes(k, c, dtype):
    cfg, other = (synth.conv_layer(3, c, 13, 18, 72, k, 1, k // 2, dtype, 9420 + c + i) for i in (0, 1))
    x, wt, pad = cfg["x"].to(DEV), cfg["w"].to(DEV), (k // 2 if k > 1 else 0,) * 2
    want = torch.nn.functional.conv2d(cfg["x"].double(), cfg["w"].double(), padding=pad).numpy()
    want = want.astype(np.int64) if dtype == "i8" else want
    full = gs.conv2d_workspace(x, wt, (1, 1), pad)

    def takes(size):
        try:
            gs.conv2d_pack_weights(wt, packed=torch.empty(size, dtype=torch.uint8, device=DEV))
        except gs.GlensideError:
            return False
        return True
    least = next(size for size in range(256, full + 256, 256) if takes(size))
    assert least < full
    for before in (0x5A, None):         # a buffer of anything, and one that held other weights in all copies
        for packs, reads in ((least, full), (least, full + 4096), (full, least), (full, full + 4096)):
            buf = torch.full((full + 4096,), before or 0, dtype=torch.uint8, device=DEV)
            if before is None:
                gs.conv2d_pack_weights(other["w"].to(DEV), packed=buf)
            gs.conv2d_pack_weights(wt, packed=buf[:packs])
            assert_parity(gs.conv2d_direct_packed(x, wt, buf[:reads], (1, 1), pad), want, what=f"packed in {packs}, read in {reads} bytes")


# Few channels and many output rows: tasks of two rows (conv_rows_kernel).  Odd row counts, rows cut inside a
# 16-byte store, several position and channel tiles, windows of one row, 16-byte loads and element by element.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("n,c,h,w,o,kh,kw,pad", [(41, 3, 77, 80, 64, 7, 7, 3), (42, 3, 79, 83, 33, 7, 7, 3), (11, 1, 300, 300, 40, 3, 5, 1),
                                                 (30, 9, 64, 64, 100, 3, 3, 1), (40, 5, 90, 48, 65, 1, 8, 0), (50, 2, 66, 66, 8, 2, 4, 1)])
def test_conv2d_few_channels_many_rows(n, c, h, w, o, kh, kw, pad, dtype, odt):
    s = 4 if dtype == "i8" else 2
    if dtype == "i8":
        n *= 4
    x, wt = gen(dtype, (n, c, h, w), 8700 + h), gen(dtype, (o, c, kh, kw), 8800 + o, (c * kh * kw) ** -0.5)
    want = torch.nn.functional.conv2d(x.double(), wt.double(), stride=s, padding=pad)
    res = gen("i32" if dtype == "i8" else ("bf16" if odt == torch.bfloat16 else "f32"), tuple(want.shape), 8900 + o)
    buf = torch.full((want.numel() + 512,), 77, dtype=odt, device=DEV)
    out = buf[256:256 + want.numel()].view(want.shape)
    packed = gs.conv2d_pack_weights(wt.to(DEV), for_input=(x.to(DEV), (s, s), (pad, pad)))
    for residual, act in ((None, gs.GS_ACT_NONE), (res, gs.GS_ACT_RELU)):
        ref = want if residual is None else (want + res.double()).clamp_min(0)
        ref = ref.numpy().astype(np.int64) if dtype == "i8" else ref.numpy()
        how = dict(act=act, residual=None if residual is None else residual.to(DEV))
        gs.conv2d_direct_packed(x.to(DEV), wt.to(DEV), packed, (s, s), (pad, pad), out=out, **how)
        assert_parity(out, ref, what=f"{dtype} packed")
        assert (buf[:256] == 77).all() and (buf[256 + want.numel():] == 77).all()
        got = gs.conv2d_direct(x.to(DEV), wt.to(DEV), (s, s), (pad, pad), out_dtype=odt, **how)
        assert_parity(got, ref, what=f"{dtype} weights as they are")


# conv2d_direct(.., ws) == conv2d_pack_weights(w, ws), then conv2d_direct_packed(.., ws): the workspace holds the same
# bytes afterwards and goes on serving other batches.  Few channels in both forms and with tasks of two rows, a chunk
# filled in part, whole chunks, 1x1, output channels past a block of 32 and of 64, an empty batch.
@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("n,c,h,w,o,k,s,p", [(1, 3, 8, 8, 4, 3, 1, 0), (2, 3, 40, 44, 70, 7, 2, 3), (41, 3, 77, 80, 64, 7, 4, 3), (3, 9, 12, 11, 130, 5, 1, 2),
                                             (2, 1, 9, 9, 5, 1, 1, 0), (1, 40, 9, 10, 33, 3, 1, 1), (2, 64, 14, 14, 65, 3, 2, 1), (1, 32, 7, 9, 31, 5, 1, 2),
                                             (2, 128, 7, 7, 40, 1, 1, 0), (0, 3, 8, 8, 4, 3, 1, 0), (0, 64, 8, 8, 4, 3, 1, 0)])
def test_conv2d_direct_leaves_packed_weights(n, c, h, w, o, k, s, p, dtype):
    x, wt = gen(dtype, (n, c, h, w), 8950 + h).to(DEV), gen(dtype, (o, c, k, k), 8960 + o, (c * k * k) ** -0.5).to(DEV)
    x2 = gen(dtype, (n + 3, c, h, w), 8970 + h)
    size = gs.conv2d_workspace(x2.to(DEV), wt, (s, s), (p, p))
    size = max(size, gs.conv2d_workspace(x, wt, (s, s), (p, p)))
    ws, packed = (torch.full((size,), 0x5a, dtype=torch.uint8, device=DEV) for _ in range(2))
    gs.conv2d_direct(x, wt, (s, s), (p, p), workspace=ws)
    gs.conv2d_pack_weights(wt, packed)
    weights = gs.conv2d_pack_weights(wt).numel()          # without scratch for a split channel sum
    assert torch.equal(ws[:weights], packed[:weights])
    got = gs.conv2d_direct_packed(x2.to(DEV), wt, ws, (s, s), (p, p))
    want = torch.nn.functional.conv2d(x2.double(), wt.cpu().double(), stride=s, padding=p).numpy()
    assert_parity(got, want.astype(np.int64) if dtype == "i8" else want, what="packed by the call")


def test_conv2d_minus_128_and_empty_batch():
    x = torch.full((1, 32, 6, 6), -128, dtype=torch.int8)
    w = torch.full((8, 32, 3, 3), -128, dtype=torch.int8)
    got = gs.conv2d_direct(x.to(DEV), w.to(DEV), (1, 1), (1, 1))
    assert_parity(got, conv_oracle(x, w, (1, 1), (1, 1)))
    empty = torch.zeros((0, 32, 6, 6), dtype=torch.int8, device=DEV)
    assert gs.conv2d_direct(empty, w.to(DEV), (1, 1), (1, 1)).shape == (0, 8, 6, 6)
    assert gs.conv2d_im2col(empty, w.to(DEV), (1, 1), (1, 1)).shape == (0, 8, 6, 6)


# ---------------------------------------------------------------------------------------------
# reduce, pooling, pair
# ---------------------------------------------------------------------------------------------

REDUCE_CASES = [
    ("i8", (7, 13), 1), ("i8", (3, 5, 4), 1), ("i32", (10, 49), 1), ("bf16", (6, 5, 7, 7), 2),
    ("f32", (33, 100), 1), ("bf16", (3, 5000), 1), ("f32", (1000, 1), 1), ("i32", (2, 9000), 1),
    ("bf16", (513, 4), 1), ("f32", (5,), 0),
    # many short rows: staged through LDS, 128 rows per workgroup, ragged last workgroup
    ("bf16", (600, 49), 1), ("i8", (777, 33), 1), ("f32", (515, 9), 1), ("i32", (1030, 13), 1),
    ("bf16", (9, 64, 7, 7), 2),
]


@pytest.mark.parametrize("op", [gs.GS_SUM, gs.GS_MAX])
@pytest.mark.parametrize("case", REDUCE_CASES)
def test_reduce(case, op):
    dtype, shape, na = case
    x = gen(dtype, shape, 1700 + len(shape) + shape[0])
    got = gs.reduce(x.to(DEV), na, op)
    oper = ap.reduceSum if op == gs.GS_SUM else ap.reduceMax
    want = ap.compute(oper, ap.access(ap.tensor(to_oracle(x)), na)).materialize()
    if op == gs.GS_MAX:
        np.testing.assert_array_equal(to_oracle(got), want)      # max is exact in every dtype
    else:
        assert_parity(got, want, float_tol=1e-2 if dtype == "bf16" else 1e-4, what=str(case))


def test_reduce_scaled_mean_is_global_average_pool():
    x = gen("bf16", (4, 24, 7, 7), 1801)
    got = gs.reduce(x.to(DEV), 2, gs.GS_SUM, scale=1.0 / 49.0)
    prog = ap.compute(ap.scale(1.0 / 49.0), ap.compute(ap.reduceSum, ap.access(ap.tensor(to_oracle(x)), 2)))
    assert_parity(got, prog.materialize())


POOL_CASES = [
    ("bf16", (2, 5, 14, 14), (2, 2), (2, 2), None),
    ("bf16", (2, 3, 17, 16), (3, 3), (2, 2), (1, 1)),
    ("i8", (1, 4, 9, 12), (3, 2), (1, 2), (1, 0)),
    ("f32", (2, 2, 8, 8), (8, 8), (1, 1), None),
    ("i32", (3, 3, 10, 10), (2, 2), (2, 2), None),
    ("bf16", (3, 4, 112, 112), (3, 3), (2, 2), (1, 1)),     # the ResNet stem pooling plane
    ("bf16", (1, 2, 150, 136), (3, 3), (2, 2), (1, 1)),     # several bands of rows per plane
    ("f32", (1, 3, 70, 200), (5, 3), (3, 2), (2, 1)),       # run-time window, several bands
    ("i8", (2, 3, 33, 64), (2, 2), (2, 2), None),
    ("i8", (1, 2, 31, 35), (3, 3), (1, 1), (1, 1)),
]


@pytest.mark.parametrize("case", POOL_CASES)
def test_max_pool_fused_and_unfused(case):
    dtype, shape, window, stride, pad = case
    x = gen(dtype, shape, 1900 + shape[-1])
    xd = x.to(DEV)
    fused = gs.windows_reduce(xd, 2, window, stride, pad, pad, gs.GS_MAX)
    win = gs.access_windows(xd, 2, window, stride, pad, pad, gs.GS_PAD_LOWEST)
    unfused = gs.reduce(win, 4, gs.GS_MAX)
    want = pg.max_pool2d(ap.tensor(to_oracle(x)), window, stride, pad or (0, 0), LOWEST[dtype]).materialize()
    np.testing.assert_array_equal(to_oracle(fused), want)
    assert torch.equal(fused, unfused)


# Planes pooled several to a workgroup: a last workgroup with fewer planes, runs that start off a 16-byte
# boundary, planes just below and above the size of one workgroup's share, and few planes cut into bands.
@pytest.mark.parametrize("dtype", ["bf16", "i8", "f32"])
@pytest.mark.parametrize("shape,win,stride,pad", [((3, 5, 7, 7), 2, 2, 0), ((7, 3, 13, 11), 3, 2, 1), ((2, 3, 63, 65), 3, 1, 1),
                                                  ((1, 3, 64, 64), 2, 2, 0), ((1, 2, 1, 1), 1, 1, 0), ((37, 9, 5, 3), 3, 3, 2),
                                                  ((1, 5, 155, 157), 3, 2, 1), ((1, 7, 96, 112), 3, 2, 1)])
def test_pool_of_whole_planes(shape, win, stride, pad, dtype):
    x = gen(dtype, shape, 2300 + shape[2], 3.0)
    for op, fill in ((gs.GS_MAX, -np.inf), (gs.GS_SUM, 0)):
        got = gs.windows_reduce(x.to(DEV), 2, (win, win), (stride, stride), (pad, pad), (pad, pad), op)
        cells = np.pad(to_oracle(x).astype(np.float64), ((0, 0), (0, 0), (pad, pad), (pad, pad)), constant_values=fill)
        want = np.lib.stride_tricks.sliding_window_view(cells, (win, win), axis=(2, 3))[:, :, ::stride, ::stride]
        want = want.max(axis=(4, 5)) if op == gs.GS_MAX else want.sum(axis=(4, 5))
        if dtype == "i8":
            np.testing.assert_array_equal(to_oracle(got), want.astype(np.int64))
        else:
            assert_parity(got, want, what=f"{shape} {op}")


# Padding of at least the window: some windows hold no element at all.  One case per kernel and window form:
# planes pooled several to a workgroup, vectors, bands, and windows of one and three dimensions.
@pytest.mark.parametrize("dtype", ["bf16", "i8", "i32", "f32"])
@pytest.mark.parametrize("shape,window,stride,pad", [
    ((3, 5, 4, 6), (1, 1), (1, 1), (1, 1)), ((3, 5, 4, 6), (2, 2), (1, 2), (2, 3)), ((2, 3, 7, 5), (3, 3), (1, 1), (4, 3)),
    ((2, 3, 7, 5), (5, 4), (2, 1), (6, 5)), ((1, 2, 96, 112), (3, 3), (1, 1), (4, 1)), ((1, 1, 220, 300), (4, 4), (2, 2), (5, 6)),
    ((3, 10), (2,), (1,), (3,)), ((2, 3, 4, 5), (1, 2, 2), (1, 1, 1), (1, 2, 2))])
def test_windows_wholly_in_padding(shape, window, stride, pad, dtype):
    x = gen(dtype, shape, 2400 + shape[-1])
    if dtype == "i8":
        x = x.clamp(max=-100)           # nothing above what padding holds by much
    n_access = len(shape) - len(window)
    got = gs.windows_reduce(x.to(DEV), n_access, window, stride, pad, pad, gs.GS_MAX)
    want = ap.compute(ap.reduceMax, oracle_windows(x, n_access, window, stride, pad, pad, LOWEST[dtype])).materialize()
    np.testing.assert_array_equal(to_oracle(got), want)
    unfused = gs.reduce(gs.access_windows(x.to(DEV), n_access, window, stride, pad, pad, gs.GS_PAD_LOWEST), len(shape), gs.GS_MAX)
    assert torch.equal(got, unfused)
    total = gs.windows_reduce(x.to(DEV), n_access, window, stride, pad, pad, gs.GS_SUM)
    want = ap.compute(ap.reduceSum, oracle_windows(x, n_access, window, stride, pad, pad, 0)).materialize()
    assert_parity(total, want, what=f"{shape} {window}")


# Both sides of the lines between whole planes and bands: results per plane (a workgroup's threads, 1 KB where rows
# are vectors), planes per compute unit, folds per element, bytes per plane.
@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("planes,h,w,win,stride,pad", [
    (5, 16, 16, 3, 1, 1), (5, 17, 16, 3, 1, 1), (5, 16, 17, 3, 1, 1), (3, 47, 32, 3, 1, 1), (3, 63, 64, 2, 2, 0), (2, 65, 64, 2, 2, 0),
    (127, 35, 33, 2, 2, 0), (128, 35, 33, 2, 2, 0), (255, 35, 33, 3, 1, 1), (256, 35, 33, 3, 1, 1), (256, 35, 33, 5, 1, 2),
    (256, 35, 33, 4, 1, 1), (256, 111, 111, 3, 2, 1), (257, 156, 157, 3, 2, 1), (130, 156, 157, 2, 2, 0), (1, 220, 223, 2, 2, 0)])
def test_pool_whole_planes_or_bands(planes, h, w, win, stride, pad, dtype):
    x = gen(dtype, (planes, h, w), 2500 + planes + h)
    got = gs.windows_reduce(x.to(DEV), 1, (win, win), (stride, stride), (pad, pad), (pad, pad), gs.GS_MAX)
    want = torch.nn.functional.max_pool2d(torch.nn.functional.pad(x.float()[:, None], (pad,) * 4, value=-float("inf")), win, stride)
    assert torch.equal(got.cpu().float(), want[:, 0])


# Padding that makes many results of few elements: small planes whose workgroup's results would pass 2^31 if
# planes were counted by their elements only (the first), and ones that leave a workgroup a few planes.
@pytest.mark.parametrize("planes,size,pad", [(4100, 1, 363), (300, 2, 60), (33, 3, 130)])
def test_pool_of_small_planes_under_wide_padding(planes, size, pad):
    x = torch.randint(-127, 0, (planes, size, size), dtype=torch.int8)
    got = gs.windows_reduce(x.to(DEV), 1, (size, size), (1, 1), (pad, pad), (pad, pad), gs.GS_MAX)
    out = 2 * pad + 1
    assert tuple(got.shape) == (planes, out, out)
    # only the windows within size - 1 of the middle one hold an element
    lo, hi = pad - size + 1, pad + size
    want = torch.nn.functional.max_pool2d(torch.nn.functional.pad(x.float(), (size - 1,) * 4, value=-128.0)[:, None], size, 1)[:, 0]
    assert torch.equal(got[:, lo:hi, lo:hi].cpu(), want.to(torch.int8))
    got[:, lo:hi, lo:hi] = -128
    assert int(got.max()) == -128 and int(got.min()) == -128


def test_sum_pool_and_1d_windows_reduce():
    x = gen("f32", (3, 40), 1950)
    got = gs.windows_reduce(x.to(DEV), 1, (5,), (3,), (2,), (2,), gs.GS_SUM, scale=0.2)
    node = ap.windows(ap.access(ap.pad(ap.tensor(to_oracle(x)), 1, 2, 2, 0.0), 1), (5,), (3,))
    want = ap.compute(ap.scale(0.2), ap.compute(ap.reduceSum, node)).materialize()
    assert_parity(got, want, float_tol=1e-5)


SUM_POOL_CASES = [
    ("bf16", (2, 6, 7, 7), (7, 7), (1, 1), None, 1.0 / 49.0, torch.float32),
    ("bf16", (2, 3, 40, 48), (3, 3), (2, 2), (1, 1), 1.0 / 9.0, torch.bfloat16),
    ("i8", (2, 3, 12, 16), (2, 2), (2, 2), None, 1.0, torch.int32),
    ("f32", (1, 2, 90, 100), (4, 4), (4, 4), None, 0.0625, torch.float32),
]


@pytest.mark.parametrize("case", SUM_POOL_CASES)
def test_sum_pool_2d(case):
    dtype, shape, window, stride, pad, scale, odt = case
    x = gen(dtype, shape, 1960 + shape[-1])
    got = gs.windows_reduce(x.to(DEV), 2, window, stride, pad, pad, gs.GS_SUM, scale=scale, out_dtype=odt)
    node = ap.tensor(to_oracle(x))
    if pad:
        node = ap.pad(ap.pad(node, 2, pad[0], pad[0], 0), 3, pad[1], pad[1], 0)
    prog = ap.compute(ap.reduceSum, ap.windows(ap.access(node, 2), window, stride))
    if scale != 1.0:
        prog = ap.compute(ap.scale(scale), prog)
    # fp32 accumulation of up to 49 terms against an fp64 sum: error <= 49 * 2^-24 * sum|x|, and the
    # result may be 1e-3 of that sum after cancellation (the floor in rel_error) -> 1e-4 covers it.
    assert_parity(got, prog.materialize(), float_tol=1e-2 if odt == torch.bfloat16 else 1e-4)


@pytest.mark.parametrize("dtype", ["i32", "bf16", "f32"])
@pytest.mark.parametrize("op", [gs.GS_SUM, gs.GS_MAX])
def test_pair_reduce(dtype, op):
    a, b = gen(dtype, (3, 5, 7, 11), 2001), gen(dtype, (3, 5, 7, 11), 2002)
    got = gs.pair_reduce(a.to(DEV), b.to(DEV), op, gs.GS_ACT_RELU)
    oper = ap.reduceSum if op == gs.GS_SUM else ap.reduceMax
    pr = ap.pair(ap.access(ap.tensor(to_oracle(a)), 4), ap.access(ap.tensor(to_oracle(b)), 4))
    want = ap.compute(ap.relu, ap.compute(oper, pr)).materialize()
    assert_parity(got, want, float_tol=1e-2 if dtype == "bf16" else 1e-6)


# ---------------------------------------------------------------------------------------------
# transformers that move data: transpose, slice, concat, pair, pad
# ---------------------------------------------------------------------------------------------

def assert_same_values(got, node, what):
    """A transformer only moves elements: the stored values must be the oracle's, exactly."""
    want = node.materialize()
    assert tuple(got.shape) == tuple(want.shape), what
    np.testing.assert_array_equal(to_oracle(got), want, err_msg=what)


TRANSPOSE_CASES = [
    # dtype, shape, n_access, perm
    ("bf16", (3, 20, 20, 24), 1, (0, 3, 1, 2)),      # the (N,H',W',O) -> (N,O,H',W') tail of Fig. 5
    ("f32", (70, 130), 1, (1, 0)),                   # ((N),(O)) -> ((O),(N)), ragged 64 x 64 tiles
    ("i8", (5, 67, 33), 2, (0, 2, 1)),
    ("i32", (4, 3, 5, 6), 2, (3, 1, 0, 2)),          # no dimension keeps its place
    ("bf16", (6, 7, 64), 1, (1, 0, 2)),              # the contiguous dimension stays: rows are copied
    ("bf16", (2, 3, 4, 5, 6), 3, (4, 3, 2, 1, 0)),
    ("f32", (9,), 1, (0,)),
    ("i8", (2, 64, 136), 1, (0, 2, 1)),              # 8 elements per lane
    ("bf16", (3, 7, 9), 1, (0, 2, 1)),               # odd extents: one element per lane
]


@pytest.mark.parametrize("case", TRANSPOSE_CASES)
def test_transpose(case):
    dtype, shape, na, perm = case
    x = gen(dtype, shape, 2100 + len(shape) + shape[0])
    got = gs.transpose(x.to(DEV), na, perm)
    assert_same_values(got, ap.transpose(ap.access(ap.tensor(to_oracle(x)), na), perm), str(case))


SLICE_CASES = [
    ("bf16", (4, 64, 40), 1, 1, 8, 56), ("i8", (37, 19), 1, 1, 3, 17), ("f32", (10, 6, 8), 2, 0, 2, 9),
    ("i32", (5, 12), 1, 1, 4, 4), ("bf16", (3, 5, 7, 16), 2, 2, 1, 6),
]


@pytest.mark.parametrize("case", SLICE_CASES)
def test_slice(case):
    dtype, shape, na, dim, lo, hi = case
    x = gen(dtype, shape, 2200 + shape[0])
    got = gs.slice_(x.to(DEV), na, dim, lo, hi)
    assert_same_values(got, ap.slice_(ap.access(ap.tensor(to_oracle(x)), na), dim, lo, hi), str(case))


CONCAT_CASES = [
    ("bf16", (4, 24, 32), (4, 40, 32), 1, 1), ("i8", (3, 5), (3, 9), 1, 1), ("f32", (2, 6, 8), (5, 6, 8), 1, 0),
    ("i32", (4, 3, 0), (4, 3, 5), 2, 2), ("bf16", (2, 3, 4, 8), (2, 3, 4, 24), 2, 3),
]


@pytest.mark.parametrize("case", CONCAT_CASES)
def test_concat(case):
    dtype, sa, sb, na, dim = case
    a, b = gen(dtype, sa, 2300 + sa[0]), gen(dtype, sb, 2310 + sb[0])
    got = gs.concat(a.to(DEV), b.to(DEV), na, dim)
    node = ap.concat(ap.access(ap.tensor(to_oracle(a)), na), ap.access(ap.tensor(to_oracle(b)), na), dim)
    assert_same_values(got, node, str(case))


@pytest.mark.parametrize("case", [("bf16", (6, 5, 16), 1), ("i8", (7, 3), 1), ("f32", (4, 9, 2), 2),
                                  ("i32", (5, 8), 2), ("bf16", (33, 64), 0)])
def test_pair(case):
    dtype, shape, na = case
    a, b = gen(dtype, shape, 2400 + shape[0]), gen(dtype, shape, 2410 + shape[0])
    got = gs.pair(a.to(DEV), b.to(DEV), na)
    node = ap.pair(ap.access(ap.tensor(to_oracle(a)), na), ap.access(ap.tensor(to_oracle(b)), na))
    assert_same_values(got, node, str(case))


@pytest.mark.parametrize("case", [("bf16", (3, 8, 16), 1, 2, 8, 8, gs.GS_PAD_ZERO), ("i8", (5, 7), 1, 1, 2, 3, gs.GS_PAD_LOWEST),
                                  ("f32", (4, 6, 5), 2, 1, 1, 0, gs.GS_PAD_LOWEST), ("i32", (2, 9), 1, 0, 0, 0, gs.GS_PAD_ZERO)])
def test_pad(case):
    dtype, shape, na, dim, lo, hi, mode = case
    x = gen(dtype, shape, 2500 + shape[0])
    got = gs.pad(x.to(DEV), na, dim, lo, hi, mode)
    fill = LOWEST[dtype] if mode == gs.GS_PAD_LOWEST else 0
    assert_same_values(got, ap.pad(ap.access(ap.tensor(to_oracle(x)), na), dim, lo, hi, fill), str(case))


@pytest.mark.parametrize("dtype,block", [("i8", 16), ("i8", 32), ("bf16", 16), ("bf16", 64)])
def test_cartesian_dot_blocked_is_the_blocked_program(dtype, block):
    """Square blocks, every dimension a multiple: the program of Fig. 7 generalised, block by block."""
    m, k, o = 2 * block, 4 * block, 3 * block
    a = gen(dtype, (m, k), 2701 + block, 1.0)
    w = gen(dtype, (k, o), 2702 + block, 1.0 / np.sqrt(k) if dtype == "bf16" else 1.0)    # (K,O) as in Fig. 2b
    wt = gs.transpose(w.to(DEV), 1, (1, 0))                                                 # ((O),(K))
    got = gs.cartesian_dot_blocked(a.to(DEV), wt, block, block, block)
    prog, count = pg.blocked_matmul(ap.tensor(to_oracle(a)), ap.tensor(to_oracle(w)), block)
    assert count == 2 * 3 * 4
    assert_parity(got, prog.materialize(), what=f"blocked {dtype} {block}")
    if dtype == "i8":
        assert torch.equal(got, gs.cartesian_dot(a.to(DEV), wt))


@pytest.mark.parametrize("tiles", [(64, 64, 128), (100, 48, 80), (1000, 1000, 1000), (17, 256, 33),
                                   (100, 48, 128), (17, 200, 64), (128, 130, 256), (150, 64, 64)])
def test_cartesian_dot_blocked_ragged_tiles(tiles):
    """Tile sizes that do not divide the matrix: last blocks and last K slices are smaller."""
    a0, a1 = gen("i8", (150, 328), 2801), gen("i8", (130, 328), 2802)
    got = gs.cartesian_dot_blocked(a0.to(DEV), a1.to(DEV), *tiles)
    assert torch.equal(got, gs.cartesian_dot(a0.to(DEV), a1.to(DEV)))
    b0, b1 = gen("bf16", (150, 320), 2803), gen("bf16", (130, 320), 2804, 1.0 / np.sqrt(320))
    gotf = gs.cartesian_dot_blocked(b0.to(DEV), b1.to(DEV), *tiles)
    prog = pg.cartesian_dot(ap.access(ap.tensor(to_oracle(b0)), 1), ap.access(ap.tensor(to_oracle(b1)), 1))
    assert_parity(gotf, prog.materialize(), what=f"ragged {tiles}")
    c0, c1 = gen("fp8", (150, 320), 2805), gen("fp8", (130, 320), 2806, 1.0 / np.sqrt(320))
    got8 = gs.cartesian_dot_blocked(c0.to(DEV), c1.to(DEV), *tiles)
    assert_parity(got8, brute.matmul(to_oracle(c0), to_oracle(c1).T), what=f"ragged fp8 {tiles}",
                  slack=fp8_slack(to_oracle(c0), to_oracle(c1)))


@pytest.mark.parametrize("dtype,tiles", [("bf16", (512, 512, 128)), ("i8", (512, 768, 256)), ("fp8", (1024, 512, 128)),
                                         ("bf16", (384, 640, 64))])
def test_cartesian_dot_blocked_one_launch_large(dtype, tiles):
    """Blocks large enough for the 256x256 and 128x128 tiles, a last block of four rows, K slices that
    are whole slabs (one launch); sampled rows on both sides of block boundaries against the oracle."""
    I, J, K = 4100, 4104, 256
    a0 = gen(dtype, (I, K), 2901, 1.0)
    a1 = gen(dtype, (J, K), 2902, 1.0 / np.sqrt(K) if dtype != "i8" else 1.0)
    got = gs.cartesian_dot_blocked(a0.to(DEV), a1.to(DEV), *tiles)
    bm = tiles[0]
    rows = sorted({0, 1, 255, 256, bm - 1, bm, bm + 1, 2 * bm - 1, 2 * bm, I - 5, I - 4, I - 3, I - 1}
                  | set(int(v) for v in np.random.default_rng(7).integers(0, I, 30)))
    idx = torch.tensor(rows)
    want = brute.matmul(to_oracle(a0[idx]), to_oracle(a1).T)
    assert_parity(got[idx.to(DEV)], want, what=f"{dtype} {tiles}",
                  slack=fp8_slack(to_oracle(a0[idx]), to_oracle(a1)) if dtype == "fp8" else None)
    if dtype == "i8":
        assert torch.equal(got, gs.cartesian_dot(a0.to(DEV), a1.to(DEV)))


def test_blocked_matmul_from_slices_and_concat():
    """Fig. 7 on the GPU: a matmul split in two along N and K with slice, cartProd/dotProd on the
    blocks, pair + reduceSum over the K halves and concat along N equals the unblocked product
    (exactly, for integers)."""
    a = gen("i8", (48, 128), 2601)
    b = gen("i8", (80, 128), 2602)
    A, B = a.to(DEV), b.to(DEV)
    whole = gs.cartesian_dot(A, B)
    cols = []
    for n0, n1 in ((0, 32), (32, 80)):
        bn = gs.slice_(B, 1, 0, n0, n1)
        halves = [gs.cartesian_dot(gs.slice_(A, 1, 1, k0, k0 + 64), gs.slice_(bn, 1, 1, k0, k0 + 64)) for k0 in (0, 64)]
        cols.append(gs.pair_reduce(halves[0], halves[1], gs.GS_SUM))
    blocked = gs.concat(cols[0], cols[1], 2, 1)
    assert torch.equal(blocked, whole)
    prog = pg.cartesian_dot(ap.access(ap.tensor(to_oracle(a)), 1), ap.access(ap.tensor(to_oracle(b)), 1))
    assert_parity(blocked, prog.materialize(), what="blocked matmul")


# ---------------------------------------------------------------------------------------------
# depth-wise windows
# ---------------------------------------------------------------------------------------------

def oracle_depthwise(x, w, stride, pad):
    """C one-channel convolutions (brute-force loops), stacked along the channel dimension."""
    xo, wo = to_oracle(x), to_oracle(w)
    return np.concatenate([brute.conv2d(np.ascontiguousarray(xo[:, c:c + 1]), np.ascontiguousarray(wo[c:c + 1, None]),
                                        stride, pad) for c in range(x.shape[1])], axis=1)


def test_depthwise_is_the_sliced_program():
    """Small case against the program itself: slice / Fig. 2a / concat, evaluated by the interpreter."""
    for dtype, odt in (("bf16", torch.float32), ("i8", torch.int32)):
        x, w = gen(dtype, (2, 5, 9, 11), 3101), gen(dtype, (5, 3, 3), 3102, 0.3)
        got = gs.depthwise_conv2d(x.to(DEV), w.to(DEV), (1, 1), (1, 1), out_dtype=odt)
        prog = pg.depthwise_conv2d(ap.tensor(to_oracle(x)), ap.tensor(to_oracle(w)[:, None]), (1, 1), (1, 1))
        assert tuple(got.shape) == prog.access_shape
        assert_parity(got, prog.materialize(), what=f"depth-wise program {dtype}")


DEPTHWISE_CASES = [
    # dtype, N, C, H, W, Kh, Kw, stride, pad, out dtype, relu
    ("bf16", 3, 24, 56, 56, 3, 3, (1, 1), (1, 1), torch.bfloat16, False),   # several planes per task, 16-byte stores
    ("bf16", 2, 16, 112, 112, 3, 3, (2, 2), (1, 1), torch.bfloat16, True),  # one plane per task, stride 2
    ("bf16", 1, 3, 300, 200, 3, 3, (1, 1), (1, 1), torch.float32, False),   # planes cut into bands of rows
    ("bf16", 1, 2, 301, 203, 3, 3, (2, 2), (1, 1), torch.bfloat16, False),  # bands, stride 2, odd sizes
    ("bf16", 4, 40, 14, 14, 3, 3, (1, 1), (1, 1), torch.bfloat16, True),    # rows that are no multiple of 16 bytes
    ("bf16", 5, 67, 7, 7, 3, 3, (1, 1), (1, 1), torch.float32, False),      # ragged last group of planes
    ("bf16", 2, 6, 28, 28, 3, 3, (2, 2), (1, 1), torch.bfloat16, False),
    ("bf16", 2, 7, 13, 17, 5, 5, (1, 1), (2, 2), torch.float32, True),      # 5x5
    ("bf16", 2, 3, 20, 19, 3, 2, (2, 1), (1, 0), torch.float32, False),     # run-time window loops
    ("bf16", 2, 3, 9, 9, 1, 1, (1, 1), (0, 0), torch.bfloat16, False),      # 1x1: a per-channel scale
    ("bf16", 1, 1, 3, 3, 3, 3, (1, 1), (0, 0), torch.float32, False),       # a single window
    ("i8", 3, 24, 56, 56, 3, 3, (1, 1), (1, 1), torch.int32, False),
    ("i8", 2, 9, 112, 112, 3, 3, (2, 2), (1, 1), torch.int32, True),
    ("i8", 4, 33, 14, 14, 3, 3, (1, 1), (1, 1), torch.int32, False),
    ("i8", 1, 2, 200, 333, 5, 5, (1, 1), (2, 2), torch.int32, False),
    ("i8", 2, 3, 20, 19, 4, 3, (3, 2), (0, 2), torch.int32, False),
]


@pytest.mark.parametrize("case", DEPTHWISE_CASES)
def test_depthwise_conv2d(case):
    dtype, n, c, h, w_, kh, kw, stride, pad, odt, relu = case
    x = gen(dtype, (n, c, h, w_), 3200 + c + h)
    w = gen(dtype, (c, kh, kw), 3300 + c + kh, 1.0 / np.sqrt(kh * kw) if dtype == "bf16" else 1.0)
    got = gs.depthwise_conv2d(x.to(DEV), w.to(DEV), stride, pad, gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE, odt)
    want = oracle_depthwise(x, w, stride, pad)
    if relu:
        want = np.maximum(want, 0)
    assert_parity(got, want, what=str(case))


# Enough planes for strips of several output rows: heights that leave each remainder, bands, columns read as
# aligned vectors (widths of a multiple of eight, "same" padding) and not; rows of NaN next to the border stay theirs.
@pytest.mark.parametrize("dtype,odt", [("bf16", torch.bfloat16), ("bf16", torch.float32), ("i8", torch.int32)])
@pytest.mark.parametrize("k,pad", [(3, 1), (3, 0), (5, 2)])
@pytest.mark.parametrize("n,c,h,w_", [(64, 520, 8, 16), (61, 560, 7, 24), (64, 523, 9, 9), (16, 509, 30, 17), (16, 130, 54, 104), (2, 100, 203, 240)])
def test_depthwise_strips_of_several_rows(n, c, h, w_, k, pad, dtype, odt):
    x = gen(dtype, (n, c, h, w_), 3400 + c + h)
    w = gen(dtype, (c, k, k), 3500 + c + k, 1.0 / k if dtype == "bf16" else 1.0)
    if dtype == "bf16":
        x[0, 0, 0] = float("nan")
        x[-1, -1, -1] = float("inf")
    got = gs.depthwise_conv2d(x.to(DEV), w.to(DEV), (1, 1), (pad, pad), gs.GS_ACT_NONE, odt).cpu()
    wide = torch.float64
    xp = torch.nn.functional.pad(x.to(wide), (pad, pad, pad, pad))
    ho, wo = h + 2 * pad - k + 1, w_ + 2 * pad - k + 1
    want = sum(xp[:, :, i:i + ho, j:j + wo] * w.to(wide)[None, :, i, j, None, None] for i in range(k) for j in range(k))
    if dtype == "i8":
        assert torch.equal(got, want.to(torch.int32))
        return
    finite = torch.isfinite(want)
    assert torch.equal(finite, torch.isfinite(got)) and torch.equal(torch.isnan(want), torch.isnan(got))
    # one rounding to the result's type, and k * k products summed in 32 bits
    mag = sum(xp[:, :, i:i + ho, j:j + wo].abs() * w.to(wide).abs()[None, :, i, j, None, None] for i in range(k) for j in range(k))
    bound = mag * (k * k * 2.0 ** -23) + (want.abs() * 2.0 ** -8 if odt == torch.bfloat16 else 0.0) + 1e-30
    assert bool(((got.to(wide) - want).abs() <= bound)[finite].all())


def test_depthwise_extremes_and_empty():
    x = torch.full((2, 3, 10, 10), -128, dtype=torch.int8)
    w = torch.full((3, 3, 3), -128, dtype=torch.int8)
    got = gs.depthwise_conv2d(x.to(DEV), w.to(DEV), (1, 1), (0, 0))
    assert (got.cpu() == 128 * 128 * 9).all()
    # an infinity next to the border must not leak into windows that do not contain it
    xf = torch.zeros((1, 1, 8, 8), dtype=torch.bfloat16)
    xf[0, 0, 0, 7] = float("inf")
    wf = torch.ones((1, 3, 3), dtype=torch.bfloat16)
    gf = gs.depthwise_conv2d(xf.to(DEV), wf.to(DEV), (1, 1), (1, 1)).cpu()
    assert torch.isinf(gf[0, 0, :2, 6:]).all() and torch.isfinite(gf[0, 0, 2:]).all() and torch.isfinite(gf[0, 0, :, :6]).all()
    empty = torch.zeros((0, 4, 8, 8), dtype=torch.bfloat16, device=DEV)
    assert gs.depthwise_conv2d(empty, torch.ones((4, 3, 3), dtype=torch.bfloat16, device=DEV), (1, 1), (1, 1)).shape == (0, 4, 8, 8)


# ---------------------------------------------------------------------------------------------
# seeded random sweeps of the window kernels
# ---------------------------------------------------------------------------------------------

def _random_window_cases(seed, count):
    r = np.random.default_rng(seed)
    cases = []
    while len(cases) < count:
        dtype = ("i8", "bf16", "f32", "i32")[int(r.integers(4))]
        n, c = int(r.integers(1, 4)), int(r.integers(1, 20))
        h, w = int(r.integers(3, 70)), int(r.integers(3, 70))
        k = (int(r.integers(1, 5)), int(r.integers(1, 5)))
        s = (int(r.integers(1, 4)), int(r.integers(1, 4)))
        p = (int(r.integers(0, k[0])), int(r.integers(0, k[1])))
        if h + 2 * p[0] < k[0] or w + 2 * p[1] < k[1]:
            continue
        cases.append((dtype, (n, c, h, w), k, s, p))
    return cases


@pytest.mark.parametrize("case", _random_window_cases(20210906, 40))
def test_windows_random_shapes(case):
    """Pooling (fused windows + reduceMax / reduceSum) and the explicit gather on seeded random planes,
    windows, strides and paddings; maxima and gathers bit-exact, sums within the accumulation bound."""
    dtype, shape, k, s, p = case
    x = gen(dtype, shape, 3500 + shape[2] + shape[3])
    xd = x.to(DEV)
    xo = to_oracle(x)
    got = gs.windows_reduce(xd, 2, k, s, p, p, gs.GS_MAX)
    np.testing.assert_array_equal(to_oracle(got), pg.max_pool2d(ap.tensor(xo), k, s, p, LOWEST[dtype]).materialize())
    win = gs.access_windows(xd, 2, k, s, p, p, gs.GS_PAD_ZERO)
    want_win = oracle_windows(x, 2, k, s, p, p, 0).materialize()
    np.testing.assert_array_equal(to_oracle(win), want_win)
    odt = {"i8": torch.int32, "i32": torch.int32, "bf16": torch.float32, "f32": torch.float32}[dtype]
    tot = gs.windows_reduce(xd, 2, k, s, p, p, gs.GS_SUM, out_dtype=odt)
    want_sum = want_win.sum(axis=(4, 5))
    if dtype in ("i8", "i32"):
        np.testing.assert_array_equal(to_oracle(tot), want_sum)
    else:
        assert_parity(tot, want_sum, float_tol=1e-4, what=str(case))


def _random_depthwise_cases(seed, count):
    r = np.random.default_rng(seed)
    cases = []
    while len(cases) < count:
        dtype = ("bf16", "i8")[int(r.integers(2))]
        n, c = int(r.integers(1, 4)), int(r.integers(1, 40))
        h, w = int(r.integers(3, 60)), int(r.integers(3, 60))
        kh, kw = [(3, 3), (3, 3), (5, 5), (1, 1), (2, 3), (4, 2)][int(r.integers(6))]
        s = (int(r.integers(1, 3)), int(r.integers(1, 3)))
        p = (int(r.integers(0, kh)), int(r.integers(0, kw)))
        if h + 2 * p[0] < kh or w + 2 * p[1] < kw:
            continue
        odt = torch.int32 if dtype == "i8" else (torch.bfloat16, torch.float32)[int(r.integers(2))]
        cases.append((dtype, n, c, h, w, kh, kw, s, p, odt, bool(r.integers(2))))
    return cases


@pytest.mark.parametrize("case", _random_depthwise_cases(20210907, 30))
def test_depthwise_random_shapes(case):
    dtype, n, c, h, w_, kh, kw, stride, pad, odt, relu = case
    x = gen(dtype, (n, c, h, w_), 3600 + c + h)
    w = gen(dtype, (c, kh, kw), 3700 + c + kh, 1.0 / np.sqrt(kh * kw) if dtype == "bf16" else 1.0)
    got = gs.depthwise_conv2d(x.to(DEV), w.to(DEV), stride, pad, gs.GS_ACT_RELU if relu else gs.GS_ACT_NONE, odt)
    want = oracle_depthwise(x, w, stride, pad)
    assert_parity(got, np.maximum(want, 0) if relu else want, what=str(case))

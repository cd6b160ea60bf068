"""Layers for every built instance of conv_tile_kernel: what the library's planner makes of a layer in a workgroup
shape is asked through `gs_test_conv_tile`, on the host."""

import ctypes
import functools

from paper_2105_09377_amd import binding as gs

SHAPES = range(5)
# Position blocks of a wave and channel-sum groups of the workgroup shapes (conv_kernels.h).
BLOCKS, GROUPS = (4, 2, 2, 2, 1), (1, 1, 1, 4, 4)


def ap(shape, n_access, dtype, data=0x10000):
    a = gs.gs_ap()
    a.data, a.dtype, a.rank, a.n_access, a.reserved = data, dtype, len(shape), n_access, 0
    for i, s in enumerate(shape):
        a.shape[i] = s
    return a


def call(x, w, stride, pad, residual, act, out, packed, way, stream):
    """(status, (shape, interleaved blocks, items per thread, a single chunk per group, positions of a tile))."""
    plan = (ctypes.c_int * 5)()
    pair = lambda v: (ctypes.c_int64 * 2)(v, v)
    ref = lambda t: ctypes.byref(t) if t is not None else None
    st = gs.lib().gs_test_conv_tile(ref(x), ref(w), pair(stride), pair(pad), ref(residual), act, ref(out),
                                    ctypes.c_void_p(packed), way, plan, ctypes.c_void_p(stream))
    return st, tuple(plan)


def call_with_projection(x, w, stride, pad, act, out, packed, w_proj, out_proj, packed_proj, way, stream):
    plan = (ctypes.c_int * 5)()
    pair = lambda v: (ctypes.c_int64 * 2)(v, v)
    st = gs.lib().gs_test_conv_tile_with_projection(ctypes.byref(x), ctypes.byref(w), pair(stride), pair(pad), act, ctypes.byref(out),
                                                    ctypes.c_void_p(packed), ctypes.byref(w_proj), ctypes.byref(out_proj),
                                                    ctypes.c_void_p(packed_proj), way, plan, ctypes.c_void_p(stream))
    return st, tuple(plan)


def built(dtype, k, shape):
    """(stride, interleaved blocks, items per thread, a single chunk) of the instances that conv_tile_inst.hip builds."""
    nj, ks = BLOCKS[shape], GROUPS[shape]
    if k == 5 and nj > 2:
        return set()
    blocks = {1: [1], 2: [1]}
    if ks == 1 and nj >= 2:
        blocks = {1: [1, 2] + ([4] if nj >= 4 else []), 2: [1, 2]}
    return {(s, il, maxi, one) for s in (1, 2) for il in blocks[s] for maxi in (1, 2, 4) for one in ((0, 1) if ks > 1 else (0,))
            if maxi < 4 or nj <= 2}


@functools.lru_cache(maxsize=None)
def layers(dtype, k, natural, shape):
    """Instance -> the way to cut it and the smallest layer (n, c, h, w, o, pad) among the candidates that lands there."""
    found = {}
    unit, code = (32, gs.GS_I8) if dtype == "i8" else (16, gs.GS_BF16)
    steps = 4 if k == 1 else 1          # chunks go to 1x1 windows four at a time
    # 3 chunks: groups of a channel sum with one and with none; 9: groups with several, unevenly
    for chunks in (3, 9):
        for n, h in ((1, 3), (2, 9), (1, 12), (3, 14), (2, 40), (40, 4)):
            for w in (4, 5, 6, 7, 8, 14, 15, 28, 29, 30, 56, 57, 58, 62, 66, 68, 75, 76, 90, 100, 101, 112, 113, 114, 130, 131, 132, 150, 151, 152, 180, 200, 201, 202, 223, 226, 300, 301, 302, 509, 512, 514, 900, 901, 902, 1300, 1301, 1302, 2050, 2051):
                if h < k or w < k or n * h * w > 40000:
                    continue
                for s in (1, 2):
                    size = n * h * w * chunks
                    x, wt = ap((n, steps * chunks * unit, h, w), 1, code), ap((40, steps * chunks * unit, k, k), 1, code)
                    for way in (shape, shape + len(SHAPES)):      # the second: tiles of whole output rows (1x1 windows)
                        st, plan = call(x, wt, s, k // 2, None, 0, None, None if natural else 0x10000, way, None)
                        key = (s, *plan[1:4])
                        if st == gs.GS_OK and (key not in found or size < found[key][0]):
                            found[key] = (size, way, (n, steps * chunks * unit, h, w, 40, k // 2))
    return {key: (way, layer) for key, (_size, way, layer) in found.items()}

"""Build the HIP library and the binding's extension module in-tree: `python -m paper_2105_09377_amd.build`."""

from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libglenside.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-inline-asm",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# (source, object, extra defines).  The pipelined convolution kernel is instantiated once per
# element type and tile shape, each in its own object so that they compile in parallel.
UNITS = [(src, os.path.splitext(src)[0] + ".o", []) for src in
         ("api.hip", "program.hip", "windows.hip", "gemm.hip", "conv.hip", "conv_smallc.hip", "conv_images.hip", "reduce.hip", "move.hip", "depthwise.hip")]
for _tr, _tag in (("Bf16Traits", "bf16"), ("I8Traits", "i8")):
    for _tile in range(3):
        UNITS.append(("conv3_inst.hip", f"conv3_{_tag}_t{_tile}.o",
                      [f"-DGS_CONV3_TRAITS={_tr}", f"-DGS_CONV3_TILE={_tile}",
                       f"-DGS_CONV3_NAME=launch_conv3_{_tag}_t{_tile}"]))
    for _k in (1, 3, 5):
        for _odd, _suffix, _shapes in ((0, "", range(5)), (1, "odd", range(1, 5))):
            for _shape in _shapes:
                _name = f"conv_tile_{_tag}_k{_k}s{_shape}{_suffix}"
                UNITS.append(("conv_tile_inst.hip", _name + ".o",
                              [f"-DGS_TILE_TRAITS={_tr}", f"-DGS_TILE_SHAPE={_shape}", f"-DGS_TILE_K={_k}",
                               f"-DGS_TILE_ODD={_odd}", f"-DGS_TILE_NAME=launch_{_name}"]))


def _compile(unit) -> str:
    src, obj, defines = unit
    obj = os.path.join(CSRC, obj)
    cmd = ["hipcc", *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed on " + src)
    noise = "is not a recognized feature for this target"   # printed by the host pass; harmless
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if noise not in l and l.strip())
    if out.strip():
        sys.stderr.write(out + "\n")
    return obj


def _compile_marshal() -> None:
    """The binding's extension module: host C++ against torch's and HIP's headers."""
    import torch
    base = os.path.dirname(torch.__file__)
    libs = os.path.join(base, "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL,
           "-L" + libs, "-Wl,-rpath," + libs, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("g++ failed on marshal.cpp")


def build(verbose: bool = True) -> str:
    """Compile every kernel source for gfx950 and link libglenside.so and _marshal.so next to this file."""
    workers = min(len(UNITS), max(1, len(os.sched_getaffinity(0))))
    with ThreadPoolExecutor(max_workers=workers) as pool:
        marshal = pool.submit(_compile_marshal)
        objs = list(pool.map(_compile, UNITS))
        marshal.result()
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()

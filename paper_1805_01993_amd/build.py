"""Build libccdc.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libccdc.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["ccdc.hip", "pipeline.hip", "node.hip", "noalloc.hip", "map.hip", "receive.hip", "plan.cpp"]
# pipeline.hip has hundreds of kernel instantiations: it is compiled in pieces, two per payload algebra; receive.hip and node.hip in one each
PIECES = {"pipeline.hip": ("CCDC_PIPELINE_PART", 10), "receive.hip": ("CCDC_RECEIVE_PART", 5), "node.hip": ("CCDC_NODE_PART", 5)}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed-fp32 instruction forms are kept out of the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter", "-Wno-unused-command-line-argument",
    "-fno-gpu-rdc",
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, cwd=CSRC, capture_output=True, text=True)
    out = (res.stdout + res.stderr).strip()
    # the host pass does not know the device-only target feature; that warning is harmless
    out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out:
        print(out, flush=True)


def build_marshal(verbose: bool = False) -> str:
    """Compile the native argument marshalling (a CPython module over torch's C++ tensors)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    flags = ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM=1", "-D__HIP_PLATFORM_AMD__=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    inc = [f for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"] for f in ("-isystem", d)]
    libs = [f for d in cpp_extension.library_paths() for f in ("-L" + d,)] + ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    _run(["g++"] + flags + inc + [os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL] + libs, verbose)
    return MARSHAL


def build_library(verbose: bool = False) -> str:
    """Compile every source (in parallel) and link the shared library."""
    os.makedirs(OBJ, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    units = []                                      # (source, object, extra flags), the long ones first
    for src in sorted(SOURCES, key=lambda s: s not in PIECES):
        name, n = PIECES.get(src, ("", 0))
        if n:
            units += [(src, os.path.join(OBJ, f"{src}.{i}.o"), [f"-D{name}={i}"]) for i in range(n)]
        else:
            units.append((src, os.path.join(OBJ, src + ".o"), []))
    objs = [obj for _, obj, _ in units]

    def compile_one(unit):
        src, obj, extra = unit
        _run([HIPCC] + FLAGS + extra + inc + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj], verbose)

    with ThreadPoolExecutor(max_workers=min(len(units) + 1, 8)) as pool:
        marshal = pool.submit(build_marshal, verbose)
        list(pool.map(compile_one, units))
        marshal.result()
    _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-fno-gpu-rdc"] + objs + ["-o", LIB], verbose)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)

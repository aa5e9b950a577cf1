"""Builds libatts.so (the C-ABI HIP library) in-tree for gfx950 with hipcc, and _marshal.so (the short calls' argument marshalling,
host code over torch's C++ headers) with g++.

    python -m paper_2509_15148_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libatts.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["api.hip", "gemm.hip", "attention.hip", "elementwise.hip", "calib.hip", "sort.hip", "decode.hip", "skinny.hip", "streamed.hip", "small.hip", "classic.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed fp32 instructions are switched off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
] + os.environ.get("ATTS_HIPCC_EXTRA", "").split()     # extra hipcc flags (e.g. -save-temps when reading the ISA)


def _compile(src: str) -> str:
    obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
    os.makedirs(os.path.dirname(obj), exist_ok=True)
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr[-8000:]}")
    noise = "is not a recognized feature for this target"
    warn = "\n".join(l for l in r.stderr.splitlines() if noise not in l).strip()
    if warn:
        print(f"[build] {src}:\n{warn}", file=sys.stderr)
    return obj


def _compile_marshal() -> str:
    import torch
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(HERE, "_build", "marshal.o")
    os.makedirs(os.path.dirname(obj), exist_ok=True)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    for path in include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    r = subprocess.run([*cmd, "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on marshal.cpp:\n{r.stderr[-8000:]}")
    return obj


def _link_marshal(obj: str) -> None:
    import torch
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-o", MARSHAL, obj, "-L", HERE, "-latts", "-Wl,-rpath,$ORIGIN", "-L", libs, "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link of _marshal.so failed:\n{r.stderr[-8000:]}")


def build(verbose: bool = True) -> str:
    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, 8)) as ex:
        marshal = ex.submit(_compile_marshal)
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-8000:]}")
    _link_marshal(marshal.result())
    if verbose:
        print(f"[build] wrote {LIB}")
    return LIB


if __name__ == "__main__":
    build()

"""Builds libhgnn.so (gfx950) in-tree with hipcc, and the module of its Python entry points. Usable as `python -m paper_2506_21788_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhgnn.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["neighbor.hip", "gemm.hip", "edge.hip", "edge_fused.hip", "layer.hip", "wide.hip", "heads.hip", "heads_deep.hip", "optim.hip", "prof.hip"]

COMMON = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]
# the cutoff test must not be contracted into fused multiply-adds
PER_FILE = {"neighbor.hip": ["-ffp-contract=off"]}


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _compile(src: str, objdir: str) -> str:
    obj = os.path.join(objdir, src.replace(".hip", ".o"))
    cmd = [hipcc(), *COMMON, *PER_FILE.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_native(objdir: str) -> str:
    """The Python entry points (host code against torch's C++ headers)."""
    from torch.utils.cpp_extension import include_paths
    obj = os.path.join(objdir, "native.o")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           *("-I" + d for d in (*include_paths(), sysconfig.get_path("include"), "/opt/rocm/include")),
           "-c", os.path.join(CSRC, "native.cpp"), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on native.cpp:\n" + r.stderr)
    return obj


def build(verbose: bool = True) -> str:
    from torch.utils.cpp_extension import library_paths
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        native = ex.submit(_compile_native, objdir)
        objs = list(ex.map(lambda s: _compile(s, objdir), SOURCES))
        native = native.result()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    # (torch's libraries are loaded by the time this one is: no path to them is kept)
    cmd = ["g++", "-shared", native, "-o", NATIVE, *("-L" + d for d in library_paths()), "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_python", "-L" + HERE, "-l:libhgnn.so", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print(f"built {LIB} and {NATIVE}")
    return LIB


if __name__ == "__main__":
    build()

"""Builds libhg.so (the gfx950 kernels and the C ABI of include/hg.h) and the
Python binding's native module _hgviews in-tree.

Every source of the library is compiled with hipcc for gfx950 only, then linked
into one shared library next to this file; _hgviews is host code against the
installed PyTorch, whose version its file name has.  `python -m paper_2112_15345_amd.build` runs it.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
REPO = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(REPO, "include")
LIB = os.path.join(HERE, "libhg.so")
OBJDIR = os.path.join(REPO, "_build", "hg")

SOURCES = ["hg_sample.hip", "hg_compact.hip", "hg_gather.hip", "hg_edges.hip",
           "hg_layers.hip", "hg_runtime.cpp", "hg_pipeline.cpp"]
ARCH = "gfx950"

# Packed FP32 instructions stay off (the kernels do hardly any float math; the flag
# keeps the compiler from forming them anywhere).
COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wall", "-Wno-unused-function", "-I", INCLUDE, "-I", CSRC]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; the HIP library cannot be built")


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    cmd = [hipcc(), "-x", "hip", *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{res.stdout}\n{res.stderr}")
    return obj


def _build_views(verbose: bool) -> None:
    """Compiles and links _hgviews (host code only)."""
    import torch
    from . import VIEWS_PATH
    import torch.utils.cpp_extension as ext
    libdir = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = VIEWS_PATH + ".tmp"
    inc = [x for p in (*ext.include_paths(), sysconfig.get_paths()["include"], "/opt/rocm/include")
           for x in ("-isystem", p)]
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           "-D__HIP_PLATFORM_AMD__=1", "-I", INCLUDE, *inc,
           os.path.join(CSRC, "hg_views.cpp"), "-o", tmp, "-L", libdir, "-ltorch", "-ltorch_cpu",
           "-lc10", "-ltorch_python", f"-Wl,-rpath,{libdir}"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed on hg_views.cpp:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, VIEWS_PATH)


def build(verbose: bool = False) -> str:
    """Compiles every source for gfx950 and links libhg.so (returns its path), and
    builds _hgviews."""
    os.makedirs(OBJDIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        views = ex.submit(_build_views, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
        views.result()
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

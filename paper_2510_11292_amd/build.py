"""Build libLouisKV (HIP, gfx950) in-tree with hipcc, and its Python binding.

    python -m paper_2510_11292_amd.build

compiles every csrc/*.hip for gfx950, links paper_2510_11292_amd/liblouiskv.so,
and builds csrc/binding.cpp (host code, against torch's headers) into
paper_2510_11292_amd/_binding.so.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "liblouiskv.so")
BINDING = os.path.join(PKG, "_binding.so")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed fp32 ops in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE, "-I", CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    return obj


def build_binding() -> str:
    """Compile the Python binding against the linked library; returns its path."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    # DT_RPATH (old tags): the library beside the binding comes before any
    # other of its name on LD_LIBRARY_PATH
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = BINDING + ".tmp"
    cmd = [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
           "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE,
           *[x for p in cpp_extension.include_paths() for x in ("-I", p)], "-I", "/opt/rocm/include",
           "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L", PKG, "-llouiskv",
           "-L", torch_lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-Wl,--disable-new-dtags",
           "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for binding.cpp:\n{r.stderr}")
    os.replace(tmp, BINDING)
    return BINDING


def build(verbose: bool = True) -> str:
    """Compile and link the library and its binding; returns the library's path."""
    os.makedirs(BUILD, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    build_binding()
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    try:
        build()
    except RuntimeError as e:
        print(e, file=sys.stderr)
        sys.exit(1)

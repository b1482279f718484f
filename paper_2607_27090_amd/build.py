"""Builds libinferscale.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libinferscale.so")
BINDING = os.path.join(PKG, "_binding.so")
SOURCES = ["abi.hip", "retrieve.hip", "scan_direct.hip", "place.hip", "inject.hip", "consumer.hip", "ann.hip",
           "copy.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17", "-Wall",
    # keep the compiler from emitting packed fp32 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE,
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def _compile_binding() -> None:
    """The Python binding's marshalling module (host code only). Where there is
    no host compiler or no Python header the package works without it."""
    import torch
    from torch.utils import cpp_extension
    cxx = os.environ.get("CXX", "g++")
    python_h = os.path.join(sysconfig.get_paths()["include"], "Python.h")
    if shutil.which(cxx) is None or not os.path.exists(python_h):
        print(f"not built: {BINDING} (needs {cxx} and {python_h})", file=sys.stderr)
        return
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [cxx, "-O2", "-fPIC", "-std=c++17", "-shared",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE,
           "-I", sysconfig.get_paths()["include"],
           *[a for d in cpp_extension.include_paths() for a in ("-isystem", d)],
           os.path.join(CSRC, "binding.cpp"), "-o", BINDING + ".tmp",
           "-L", libs, f"-Wl,-rpath,{libs}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed on binding.cpp:\n{r.stderr}")
    os.replace(BINDING + ".tmp", BINDING)


def build(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950, link libinferscale.so and build the
    binding's marshalling module."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        binding = ex.submit(_compile_binding)
        objs = list(ex.map(_compile, SOURCES))
        binding.result()
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)

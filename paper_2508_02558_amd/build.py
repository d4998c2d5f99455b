"""Builds libsdllm.so (the C-ABI library of HIP kernels) in-tree with hipcc for gfx950.

Usage: python -m paper_2508_02558_amd.build          (always recompiles)
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB_PATH = os.path.join(HERE, "libsdllm.so")
# tensors to entry points without ctypes (binding.py); named for the interpreter that it is built for, as others cannot load it
PYCALL_PATH = os.path.join(HERE, "_pycall" + sysconfig.get_config_var("EXT_SUFFIX"))
BUILD_DIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-fno-gpu-rdc",
    # packed-fp32 VALU forms stay off for every kernel in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _build_pycall() -> None:
    """Host code for the running interpreter.  Without its headers there is none, and the binding goes through ctypes."""
    for old in (PYCALL_PATH, os.path.join(os.path.dirname(PYCALL_PATH), "_pycall.so")):   # the second: any interpreter would load it
        if os.path.exists(old):
            os.remove(old)
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        return
    tmp = PYCALL_PATH + ".tmp"
    # by the compiler that the library is built with; it calls nothing of the HIP runtime and is not linked to it
    cmd = [HIPCC, "-no-hip-rt", "-x", "c++", "-O2", "-shared", "-fPIC", "-std=c++17", "-I", INCLUDE, "-I", include,
           os.path.join(CSRC, "pycall.cpp"), "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for pycall.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, PYCALL_PATH)


def build_library(verbose: bool = True) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB_PATH + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    _build_pycall()
    if verbose:
        print(f"built {LIB_PATH} from {len(srcs)} sources", file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    build_library()

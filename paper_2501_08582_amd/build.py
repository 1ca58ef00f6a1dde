"""Build ``liblors.so`` (the C-ABI library) for gfx950 with hipcc.

Usage: ``python -m paper_2501_08582_amd.build`` (or ``build()`` from Python).
Objects go to ``paper_2501_08582_amd/_build/``; the shared library is written
next to this file.  Every call recompiles.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "liblors.so")

ARCH = "gfx950"
SOURCES = ["abi.cpp", "fwd_bf16.hip", "fwd_thin_bf16.hip", "fwd_few_bf16.hip", "fwd24_bf16.hip", "dx_bf16.hip", "dx_thin_bf16.hip",
           "g_bf16.hip", "ste_bf16.hip", "f32_path.hip", "misc.hip"]

# Packed-fp32 VALU forms are disabled for all device code (their wrong-result
# hazard is not worth the VALU throughput on a matrix-core bound path); the
# host pass ignores the feature with a warning.
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", INCLUDE, "-I", CSRC,
          "-Wall", "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; ROCm is required to build liblors.so")
    return exe


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *COMMON, *DEVICE_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd.insert(1, "-xhip")
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stderr}")
    return obj


def _check_no_shared_weak_symbols(objs) -> None:
    """Fail if two objects define the same weak (template/inline) host symbol
    from this library's namespace: the linker would keep one definition and
    silently route both callers to it."""
    seen = {}
    for obj in objs:
        out = subprocess.run(["nm", "--defined-only", obj], capture_output=True, text=True).stdout
        for line in out.splitlines():
            parts = line.split()
            if len(parts) == 3 and parts[1] in ("W", "V") and parts[2].startswith("_ZN4lors"):
                if parts[2] in seen and seen[parts[2]] != obj:
                    raise RuntimeError(f"symbol {parts[2]} defined in both {seen[parts[2]]} and {obj}")
                seen[parts[2]] = obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(SOURCES), max(1, min(8, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    _check_no_shared_weak_symbols(objs)
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", f"--offload-arch={ARCH}", "-fPIC", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)

"""Compile the HIP library (gfx950) in-tree: paper_2405_12491_amd/libbridger.so.

Each source is compiled to an object in parallel under paper_2405_12491_amd/_build, then the
objects are linked into the shared library (written to a temporary name, then renamed).
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libbridger.so")
CALIB_LIB = os.path.join(PKG, "libbridger_calib.so")
CALIB_SOURCES = [os.path.join(CSRC, "calib.hip")]
SOURCES = [os.path.join(CSRC, n) for n in
           ("bridger_host.cpp", "perfect.hip", "perfect_binned.hip", "perfect_fixed.hip",
            "perfect_global.hip", "ragged.hip", "ragged_heap5.hip", "ragged_heap6.hip",
            "ragged_heap7.hip", "direct.hip", "gemm.hip", "bin.hip",
            "normalize.hip")]
# Sources compiled once per value of a macro (one trees' depth each: their kernels are many), and
# once without it; every other source once.
UNITS = {"perfect_global.hip": ["BRIDGER_DEPTH=%d" % d for d in range(10, 0, -1)]}
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

ARCH = ["--offload-arch=gfx950"]
FLAGS = ARCH + [
    "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _units(srcs):
    """(source, macro or None) of every object."""
    parts = [(s, m) for s in srcs for m in UNITS.get(os.path.basename(s), [])]
    return [(s, None) for s in srcs] + parts


def _object(src: str, macro) -> str:
    return os.path.join(BUILD_DIR, os.path.basename(src) + ("." + macro if macro else "") + ".o")


def _compile(src: str, macro, verbose: bool) -> str:
    obj = _object(src, macro)
    cmd = [HIPCC, *FLAGS, *(["-D" + macro] if macro else []), "-c", "-o", obj]
    cmd += ["-x", "hip", src] if src.endswith(".cpp") else [src]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"hipcc failed compiling {os.path.basename(src)}")
    return obj


def _link(objs, lib: str, verbose: bool):
    tmp = lib + ".tmp"
    cmd = [HIPCC, *ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"linking {os.path.basename(lib)} failed")
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    """Build libbridger.so (the prediction library) and libbridger_calib.so (the calibration
    microbenchmarks used by the benchmark); returns the prediction library's path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    lib, calib = _units(SOURCES), _units(CALIB_SOURCES)
    units = lib + calib
    keep = {os.path.basename(_object(*u)) for u in units}
    for name in os.listdir(BUILD_DIR):  # objects of sources that are no longer built
        if name.endswith(".o") and name not in keep:
            os.remove(os.path.join(BUILD_DIR, name))
    jobs = max(1, min(len(units), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))
    with ThreadPoolExecutor(jobs) as ex:
        list(ex.map(lambda u: _compile(*u, verbose), units))
    _link([_object(*u) for u in lib], LIB, verbose)
    _link([_object(*u) for u in calib], CALIB_LIB, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

"""Builds libjc.so in-tree with hipcc for gfx950.

Usage: python paper_2102_12416_amd/build.py [-v]
(run as a file: importing the package would load the library being built)
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libjc.so")

SOURCES = ["jc_kernels.hip", "jc_temporal.hip", "jc_resident.hip", "jc_rows.hip", "jc_synth.hip", "jc_host.cpp", "jc_group.cpp"]

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # bitwise parity: no fused multiply-add contraction anywhere
    "-ffp-contract=off",
    "-fno-fast-math",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    """Compile every source (in parallel) into libjc.so (always recompiles)."""
    tmp = LIB + ".tmp%d" % os.getpid()

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    with tempfile.TemporaryDirectory() as objdir:
        objs = [os.path.join(objdir, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        with ThreadPoolExecutor(max_workers=8) as pool:
            for _ in pool.map(lambda so: run([hipcc()] + FLAGS + ["-I", INCLUDE, "-I", CSRC, "-c", "-o", so[1],
                                                                  os.path.join(CSRC, so[0])]), zip(SOURCES, objs)):
                pass
        run([hipcc(), "--offload-arch=gfx950", "-shared", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


def build_device_check(verbose: bool = False) -> str:
    """Compile the tests' device checks of the shared helpers."""
    tests = os.path.join(ROOT, "tests")
    lib = os.path.join(tests, "libdevice_check.so")
    tmp = lib + ".tmp%d" % os.getpid()
    cmd = [hipcc()] + FLAGS + ["-shared", "-I", CSRC, "-o", tmp, os.path.join(tests, "device_check.hip")]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))

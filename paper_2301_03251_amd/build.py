"""Build ``libqlayer.so`` (the HIP library behind ``include/qlayer.h``) for gfx950.

Sources are compiled in parallel with hipcc into ``_build/`` at the repository
root and linked into ``paper_2301_03251_amd/libqlayer.so``. Every call
recompiles (the build check runs it on a machine without a GPU; hipcc
cross-compiles the device code).

Device code is built without packed-FP32 instructions (v_pk_*_f32), and with
uniform control-flow regions left unstructurised.
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libqlayer.so")
SOURCES = ["tile.hip", "kernels.hip", "runs.hip", "api.cpp", "plan.cpp", "runs.cpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]
# Uniform branches (the tile kernels' op dispatch) are left unstructurised so
# the register-resident tile keeps its registers across the dispatch.
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-mllvm", "-structurizecfg-skip-uniform-regions=true"]
# The tile kernels fetch a handler per op; handlers that start on a 32-byte
# boundary are fetched faster (21 qubits, 7 samples forward in complex128 2.28
# -> 2.21 ms, 20 qubits forward and adjoint 495 -> 490 us, 30 qubits 201.6 ->
# 200.5 ms; 64 and 128 bytes give the same). The run kernel's steps do not gain
# (41.5 -> 42.2 us at 10 qubits).
SOURCE_FLAGS = {"tile.hip": ["-mllvm", "-align-all-nofallthru-blocks=5"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src + ".o")
    cmd = [HIPCC, *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".hip"):
        cmd[1:1] = ["-x", "hip", *DEVICE, *SOURCE_FLAGS.get(src, [])]
    elif src == "api.cpp":
        cmd[1:1] = ["-x", "hip", *DEVICE]
    else:
        cmd[1:1] = ["-x", "c++"]
    subprocess.run(cmd, check=True)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)

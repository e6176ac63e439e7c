"""Builds the HIP library (gfx950) in-tree: ``paper_1205_0282_amd/libbrickcast.so``.

    python -m paper_1205_0282_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbrickcast.so")
SOURCES = ["bc_api.cpp", "bc_load.hip", "bc_frame.hip", "bc_render.hip", "bc_cnn.hip"]
ARCH = os.environ.get("BC_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if p and os.path.exists(p):
            return p
    return "hipcc"


def flags() -> list:
    return [
        "-O3", "-std=c++17", "-fPIC", "-shared", f"--offload-arch={ARCH}",
        "-fhip-fp32-correctly-rounded-divide-sqrt",
        # no packed FP32 instructions in the device code
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-pthread", "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
        "-I", os.path.join(HERE, "..", "include"),
    ]


def build(verbose: bool = False) -> str:
    srcs = []
    for s in SOURCES:
        p = os.path.join(CSRC, s)
        srcs += (["-x", "hip", p] if p.endswith(".cpp") else [p])
    tmp = LIB + ".tmp"
    cmd = [hipcc()] + flags() + srcs + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed ({r.returncode})")
    if verbose and r.stderr.strip():
        sys.stderr.write(r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

"""Build the HIP library in-tree: paper_2007_12216_amd/librnswino.so (gfx950)."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "librnswino.so")
SOURCES = ("rnswino.hip", "plan_math.cpp")


def compile_command(out: str) -> list:
    """The hipcc command that compiles every source for gfx950 and links them to `out`."""
    cmd = ["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           # matrix-core results straight into ordinary vector registers: no accumulator-register copies in the
           # epilogues, and fewer registers per wave
           "-mllvm", "-amdgpu-mfma-vgpr-form=1",
           "-Wno-unused-command-line-argument",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    return cmd + ["-o", out]


def build_library(verbose: bool = False) -> str:
    """Compile every source with hipcc for gfx950 and link the shared library."""
    cmd = compile_command(LIB)
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that is expected
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))

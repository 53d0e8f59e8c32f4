"""Build libjulia.so (HIP kernels + host runtime + C ABI) for gfx950 with hipcc.

Every translation unit is compiled with -ffp-contract=off, so a*b + c stays a
rounded product and a rounded sum unless fma is written out, and with the
packed-FP32 target feature disabled.
"""
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libjulia.so")
SOURCES = [os.path.join(CSRC, "julia_kernels.hip"), os.path.join(CSRC, "julia_host.cpp")]
HEADERS = [os.path.join(CSRC, "julia_device.h"), os.path.join(CSRC, "julia_trap.h"),
           os.path.join(ROOT, "include", "julia.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep each work-queue claim a single lane-0 atomic whose result is read
    # later, instead of a wave-wide reduction that waits for it at once
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build(verbose: bool = False, extra=()) -> str:
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, *FLAGS, *extra, *SOURCES, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if err.strip() and verbose:
        print(err)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

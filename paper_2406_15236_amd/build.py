"""Build the gfx950 library libmpc355.so in-tree with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libmpc355.so")
SOURCES = [os.path.join(HERE, "csrc", "mpc_kernels.hip"),
           os.path.join(HERE, "csrc", "mpc_probe.hip"),
           os.path.join(HERE, "csrc", "mpc_capi.cpp")]

# -ffp-contract=off: every written floating-point operation is one IEEE
# operation (fma() only where the streaming rule asks for it), so FP64 results
# follow the operation order documented in the sources.  Packed FP32 ops are
# switched off for the device code.  -disable-machine-licm: the collide is one
# long loop over tiles, and what is hoisted out of it takes registers for its
# whole length (VGPRs without the flag and with it: FP64 144 and 123, with the
# thermostat 154 and 130, SRD+a 168 with 25 spilled and with 1, split 127 and
# 113).  A step without it and with it: 256^3 FP64 with the thermostat 5.09 and
# 4.50 ms, split 3.79 and 3.39, 384^3 FP64 15.8 and 14.5, 100^3 SRD+a 0.56 and
# 0.42, 41x33x27 FP32 28.2 and 27.6 us; the other kernels take the same time.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-disable-machine-licm", "-Wall", "-Werror=unused"]


def hipcc() -> str:
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def build(verbose: bool = False) -> str:
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
    tmp = LIB + ".tmp"
    cmd = [hipcc(), *FLAGS, *inc, "-x", "hip", *SOURCES, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(res.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))

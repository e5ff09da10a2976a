"""Build libvstitch.so in-tree with hipcc for gfx950.

  python -m paper_2308_09209_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCES = [os.path.join(HERE, "csrc", n) for n in
           ("vs_host.cpp", "vs_kernels.hip", "vs_flow.hip", "vs_surr.hip", "vs_nn.hip", "vs_nn_host.cpp", "vs_nn_net.cpp", "vs_calib.hip", "vs_var.hip", "vs_noalloc.hip")]
OUT = os.path.join(HERE, "libvstitch.so")
# the device header's arithmetic as the tests call it (test_gpu_math.py)
MATH_SOURCES = [os.path.join(os.path.dirname(HERE), "tests", "device_math.hip")]
MATH_OUT = os.path.join(os.path.dirname(HERE), "tests", "libdevice_math.so")

# -ffp-contract=off: every fused multiply-add in the kernels is explicit, so
# the FP32 results follow one operation order.  Packed FP32 instructions are
# disabled for all device code.
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall"]


def build(verbose: bool = False, sources=SOURCES, out: str = OUT) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + ["-o", out + ".tmp"] + list(sources)
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("hipcc failed")
    if verbose and noise:
        print("\n".join(noise))
    os.replace(out + ".tmp", out)
    return out


def build_math(verbose: bool = False) -> str:
    return build(verbose, MATH_SOURCES, MATH_OUT)


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_math(verbose=True))

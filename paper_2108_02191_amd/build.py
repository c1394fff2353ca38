"""Compile the HIP library for gfx950 in-tree: ``python -m paper_2108_02191_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librobe.so")
CALL = os.path.join(HERE, "_robe_call.so")      # the Python side of a call (csrc/robe_call.cpp)
SOURCES = ["robe_api.hip"]
HEADERS = ["robe_device.h", "robe_kernels.h", "robe_forward_distinct.h", "robe_forward_places.h", "robe_backward_dedup.h", "robe_backward_regions.h", "robe_backward_places.h", "robe_radix_sort.h", os.path.join("..", "..", "include", "robe.h")]


def hipcc_command(out: str = LIB) -> list:
    return [
        "hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
        # hardware float atomics (global_atomic_add_f32) instead of a compare-and-swap loop
        "-munsafe-fp-atomics",
        # keep the device compiler from forming packed fp32 instructions (v_pk_*_f32).  The flag reaches
        # the host pass too, which has no such feature and says so once per inclusion: build() drops
        # exactly those lines from the log.
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-Wall", "-Wextra", "-Wno-unused-parameter", "-Wno-unknown-warning-option",
        "-o", out,
    ] + [os.path.join(CSRC, s) for s in SOURCES]


def call_command(out: str = CALL) -> list:
    """Host code only: the torch headers, the header of the library, nothing linked that torch has not loaded."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return [
        "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
        f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
        "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
        "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
        "-Wall", "-Wextra", "-Wno-unused-parameter", "-o", out, os.path.join(CSRC, "robe_call.cpp"),
        "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
    ]


def is_stale() -> bool:
    def older(out, deps):
        return not os.path.exists(out) or any(os.path.getmtime(d) > os.path.getmtime(out) for d in deps)

    abi = os.path.join(CSRC, "..", "..", "include", "robe.h")
    return older(LIB, [os.path.join(CSRC, f) for f in SOURCES + HEADERS]) or older(CALL, [os.path.join(CSRC, "robe_call.cpp"), abi])


def build(verbose: bool = False) -> str:
    cmd = hipcc_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    for line in r.stderr.splitlines():
        if "'-packed-fp32-ops' is not a recognized feature for this target" in line:
            continue            # the host pass declining a device-only feature
        print(line, file=sys.stderr)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)
    cmd = call_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print("built", LIB)
    sys.exit(0)

"""Build libsmha.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsmha.so")
SOURCES = ["plan.cpp", "kernels.hip"]
HEADERS = ["smha_internal.hpp", "device_pool.hpp", "block_fwd2.inc", "block_fwd16.inc", "wave_fwd.inc", os.path.join(ROOT, "include", "smha.h")]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def command(extra=()):
    return [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-pthread",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            # instruction scheduler that keeps memory operations in clauses: 2 % (d = 128) to 7 % (gathered
            # tiles) faster block kernel than the default, never slower on the five workloads
            "-mllvm", "-amdgpu-sched-strategy=max-memory-clause",
            "-Wno-unused-command-line-argument",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, *extra,
            *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + [h if os.path.isabs(h) else os.path.join(CSRC, h) for h in HEADERS]
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(force: bool = True, verbose: bool = False) -> str:
    if force or stale():
        cmd = command(("-Rpass-analysis=kernel-resource-usage",) if verbose else ())
        subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library(True, verbose="-v" in sys.argv))

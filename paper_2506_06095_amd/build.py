"""Build libsmha.so (HIP, gfx950) with hipcc and the native call path for torch (_smha_torch.so) with g++, in-tree."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsmha.so")
EXT = os.path.join(HERE, "_smha_torch.so")
EXT_SOURCE = os.path.join(CSRC, "torch_binding.cpp")
ABI_HEADER = os.path.join(ROOT, "include", "smha.h")
SOURCES = ["plan.cpp", "kernels.hip"]
HEADERS = ["smha_internal.hpp", "device_pool.hpp", "block_fwd2.inc", "block_fwd16.inc", "wave_fwd.inc", ABI_HEADER]


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


def extension_stamp() -> str:
    """What _smha_torch.so has to be built from and against: its sources (smha_forward's signature is compiled in), torch and Python."""
    import torch
    sources = hashlib.sha256()
    for path in (EXT_SOURCE, ABI_HEADER):
        with open(path, "rb") as f:
            sources.update(f.read())
    return f"smha-torch-binding:{sources.hexdigest()[:32]}:{torch.__version__}:{sys.implementation.cache_tag}:"


def extension_current() -> bool:
    """_smha_torch.so is there and holds that stamp (asked of the file: a module cannot be loaded twice)."""
    if not os.path.exists(EXT):
        return False
    with open(EXT, "rb") as f:
        return extension_stamp().encode() in f.read()


def build_extension() -> str:
    """_smha_torch.so against the installed torch's headers (torch has its libraries loaded when the module is imported).  It takes its
    place when it is whole: another process may be loading the old one, or building it too."""
    from torch.utils import cpp_extension
    import torch
    part = f"{EXT}.{os.getpid()}"
    try:
        subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                        f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DSMHA_STAMP="{extension_stamp()}"',
                        *[f"-isystem{d}" for d in (*cpp_extension.include_paths(), "/opt/rocm/include")],
                        "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), EXT_SOURCE, "-o", part,
                        *[f"-L{d}" for d in cpp_extension.library_paths()], "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], check=True)
        os.replace(part, EXT)
    finally:
        if os.path.exists(part):
            os.remove(part)
    return EXT


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + [h if os.path.isabs(h) else os.path.join(CSRC, h) for h in HEADERS]
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(force: bool = True, verbose: bool = False, extension: bool = True) -> str:
    if force or stale():
        cmd = command(("-Rpass-analysis=kernel-resource-usage",) if verbose else ())
        subprocess.run(cmd, check=True)
    if extension and (force or not extension_current()):
        build_extension()
    return LIB


if __name__ == "__main__":
    print(build_library(True, verbose="-v" in sys.argv))

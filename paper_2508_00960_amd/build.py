"""Build libphantom.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's native module, in-tree."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libphantom.so")
MARSHAL = os.path.join(HERE, "_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def build_library(verbose: bool = True) -> str:
    """Compile every .hip file under csrc/ into one shared library.  Always recompiles.
    PHANTOM_TUNING=1 in the environment of THIS script builds the measurement variant, whose launch-schedule
    choices can be forced through PHANTOM_* variables; the default build reads no environment variable."""
    extra = ["-DPHANTOM_TUNING_ENV"] if os.environ.get("PHANTOM_TUNING") == "1" else []
    cmd = [HIPCC, *FLAGS, *extra, *sources(), "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc failed ({proc.returncode}):\n{err}")
    return LIB


def marshal_stamp() -> str:
    """What the native module depends on: its source, the C ABI, this Python and this torch.  Built into the file."""
    import torch
    h = hashlib.sha256(f"{sys.implementation.cache_tag} {torch.__version__}".encode())
    for path in (os.path.join(CSRC, "marshal.cpp"), os.path.join(HERE, "..", "include", "phantom.h")):
        with open(path, "rb") as src:
            h.update(src.read())
    return "phantom-marshal-" + h.hexdigest()


def marshal_is_current() -> bool:
    """Is there a native module, built from the present sources for this Python and torch?"""
    try:
        with open(MARSHAL, "rb") as f:
            return marshal_stamp().encode() in f.read()
    except OSError:
        return False


def build_marshal(verbose: bool = True) -> str:
    """Compile csrc/marshal.cpp, a CPython module that reads torch tensors (host code only).  The file appears whole: other
    processes may be loading it."""
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(base, "include"), os.path.join(base, "lib")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    part = f"{MARSHAL[:-3]}.{os.getpid()}.so"
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f'-DPHANTOM_MARSHAL_STAMP="{marshal_stamp()}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", part,
           f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"g++ failed ({proc.returncode}):\n{proc.stderr}")
    os.replace(part, MARSHAL)
    return MARSHAL


if __name__ == "__main__":
    print(build_library())
    print(build_marshal())

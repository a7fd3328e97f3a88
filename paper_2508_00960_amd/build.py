"""Build libphantom.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's native module, in-tree."""
from __future__ import annotations

import hashlib
import os
import re
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libphantom.so")
MARSHAL = os.path.join(HERE, "_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # Every kernel on a page of its own: where a kernel lies within its pages changes its time by up to 2 %, and without this that moves with the size of every
    # kernel ahead of it (gradients of 64 ranks of 256 + 8 at batch 512, two trees alike but for unreached code, us a step: on 256 bytes 421.5, 425.0, on
    # 1024 423, on 4096 420, 416, on 16384 419).
    "-Xarch_device", "-falign-functions=4096",
    "-Wall", "-Wno-unused-function",
]


LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC) or HIPCC))), "llvm", "bin")


def _on_device_object(library: str, tool: str, *args: str) -> str:
    """What an LLVM tool prints about the kernels in a library that was built here."""
    with tempfile.TemporaryDirectory() as tmp:
        fat, obj = os.path.join(tmp, "fat"), os.path.join(tmp, "obj")
        run = lambda name, *a: subprocess.run([os.path.join(LLVM, name), *a], check=True, capture_output=True, text=True).stdout
        run("llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", library, os.path.join(tmp, "copy"))
        run("clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={fat}", f"--output={obj}")
        return run(tool, *args, obj)


def device_code(library: str) -> str:
    """Disassembly of the kernels."""
    return _on_device_object(library, "llvm-objdump", "-d", "--no-show-raw-insn", "--symbolize-operands")


def scratch_bytes(library: str):
    """{kernel: bytes of scratch memory per lane} of the kernels that have any: registers spilled, or arrays that did not fit them."""
    out = {}
    for kernel in re.split(r"\n\s+- \.agpr_count", _on_device_object(library, "llvm-readelf", "--notes"))[1:]:
        entry = dict(re.findall(r"\.(\w+):\s+(\S+)", kernel))
        if int(entry["private_segment_fixed_size"]):
            out[entry["name"]] = int(entry["private_segment_fixed_size"])
    return out


def _scalar_registers(operand: str):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return range(int(m[1]), int(m[2]) + 1)
    m = re.fullmatch(r"s(\d+)", operand)
    return (int(m[1]),) if m else {"m0": ("m0",), "vcc": ("vcc_lo", "vcc_hi"), "vcc_lo": ("vcc_lo",), "vcc_hi": ("vcc_hi",)}.get(operand, ())


def missing_wait_states(disassembly: str):
    """[what is wrong] where a scalar register is read by a vector-memory instruction sooner than five wait states after a vector
    instruction wrote it, or M0 is written right ahead of a direct-to-LDS load.  The compiler keeps these distances (CDNA3 ISA,
    "Manually Inserted Wait States") for its own instructions and not for those of an inline assembly statement (mfma_ring.h)."""
    code = []                   # (operation, operands, label or None, the line)
    function = ""
    for line in disassembly.splitlines():
        text = line.split("//")[0].strip()
        m = re.fullmatch(r"(?:[0-9a-f]+ )?<(.+)>:", text)
        if m:
            function = function if re.fullmatch(r"L\d+", m[1]) else m[1]
            code.append((None, (), (function, m[1]), line))
        elif text and function:
            words = re.split(r"[,\s]+", text)
            code.append((words[0], words[1:], function, text))
    wrong = []
    into, changed = {}, True    # label -> {register: wait states since the write}, the least over all ways there
    while changed:
        changed, wrong, age = False, [], {}
        for op, operands, where, text in code:
            if op is None:
                known = into.setdefault(where, {})
                if where[0] == where[1]:
                    age = {}
                for r, waited in age.items():
                    if waited < known.get(r, 5):
                        known[r], changed = waited, True
                age = dict(known)
                continue
            if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
                read = {r for w in operands for r in _scalar_registers(w)}
                wrong += [f"{where}: {text}: a vector instruction wrote s{r} {age[r]} wait states before" for r in read if age.get(r, 5) < 5]
                if "_lds_" in op and age.get("m0", 5) < 1:
                    wrong.append(f"{where}: {text}: M0 was written by the instruction before")
            waits = int(operands[0], 0) + 1 if op == "s_nop" else 1
            age = {r: waited + waits for r, waited in age.items() if waited + waits < 5}
            if op.startswith("v_"):
                second = operands[1:2] if "_co_" in op or op.startswith(("v_mad_u64_u32", "v_mad_i64_i32", "v_div_scale")) else []
                age.update({r: 0 for w in operands[:1] + second for r in _scalar_registers(w)})
            elif op.startswith("s_") and operands:
                for r in _scalar_registers(operands[0]):
                    age.pop(r, None)
                    if r == "m0":
                        age[r] = 0
            m = re.search(r"<?(L\d+)>?$", text) if "branch" in op else None
            if m:
                known = into.setdefault((where, m[1]), {})
                for r, waited in age.items():
                    if waited < known.get(r, 5):
                        known[r], changed = waited, True
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                age = {}
    return wrong


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
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        print(f"no llvm-objdump under {LLVM}: the wait states ahead of inline assembly are not checked", file=sys.stderr)
        return LIB
    wrong = missing_wait_states(device_code(LIB))
    if wrong:
        os.remove(LIB)
        raise RuntimeError("the compiler left too few wait states ahead of inline assembly:\n" + "\n".join(wrong[:20]))
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

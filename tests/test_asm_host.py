"""What the inline assembly of csrc/ owes the compiler and the hardware, and what the compiler made of the kernels, on the host."""
import os
import re
import subprocess

import pytest

from paper_2508_00960_amd.build import CSRC, FLAGS, HIPCC, LIB, LLVM, device_code, missing_wait_states, scratch_bytes

# base and LDS address are known per lane only: v_readfirstlane brings them to scalar registers right ahead of the loads
PROBE = """
#include "mfma_ring.h"
using namespace phantom;
__global__ void probe(const __bf16 *const *bases, const uint32_t *offsets, const uint32_t *at, float *out)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LdsBytes)smem + at[threadIdx.x >> 6], off = offsets[threadIdx.x];
    ring_load<0>(bases[threadIdx.x >> 6], off, lds);
    ring_wait<0>();
    out[threadIdx.x] = *lds_at<float>(lds + threadIdx.x % 64 * 16);
}
"""
needs_compiler = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(os.path.join(LLVM, "llvm-objdump"))), reason="no hipcc")


def asm_statements():
    """[(file, text of the statement)] of every inline assembly statement in csrc/"""
    out = []
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(CSRC, name)) as f:
                out += [(name, m.group(0)) for m in re.finditer(r"asm\s+volatile\s*\(.*?\)\s*;", f.read(), re.S)]
    return out


def test_statements_that_write_m0_say_so():
    writes = [(name, text) for name, text in asm_statements() if re.search(r"s_\w+ m0,", text)]
    assert writes
    for name, text in writes:
        assert '"m0"' in text.rsplit(":", 1)[1], f"{name}: {text}"


@needs_compiler
def test_the_library_keeps_the_wait_states():
    if not os.path.exists(LIB):
        pytest.skip("not built")
    code = device_code(LIB)
    assert code.count("global_load_lds_dwordx4") > 100
    assert missing_wait_states(code) == []


@needs_compiler
def test_a_kernel_without_them_is_found(tmp_path):
    src, lib = tmp_path / "probe.hip", tmp_path / "probe.so"
    src.write_text(PROBE)
    subprocess.run([HIPCC, *FLAGS, "-w", "-I", CSRC, str(src), "-o", str(lib)], check=True, capture_output=True)
    wrong = missing_wait_states(device_code(str(lib)))
    assert wrong and all("probe" in w and "global_load_lds_dwordx4" in w for w in wrong), wrong


# The one kernel that keeps values in scratch memory: eight registers, three of them read again in its loop.
SCRATCH = {"gemm_flex_f32_kernelILb0ELb1E": 36}


@needs_compiler
def test_no_kernel_spills():
    """(A loop of the 128 x 128 kernels written for one set of sums once spilled 179 registers with two, at 1.5 times the time, and gave the same results.)"""
    if not os.path.exists(LIB):
        pytest.skip("not built")
    for kernel, size in scratch_bytes(LIB).items():
        assert size <= max((most for name, most in SCRATCH.items() if name in kernel), default=0), f"{kernel}: {size} bytes of scratch a lane"


@needs_compiler
def test_a_kernel_that_spills_is_found(tmp_path):
    src, lib = tmp_path / "probe.hip", tmp_path / "probe.so"
    src.write_text("""
#include <hip/hip_runtime.h>
__global__ __launch_bounds__(64) void fits(float *out) { out[threadIdx.x] = 1.f; }
__global__ __launch_bounds__(64) void spills(float *out, const int *at)
{
    float a[1000];
    for (int i = 0; i < 1000; ++i) a[i] = out[i];
    for (int i = 0; i < 1000; ++i) a[at[i]] += 1.f;
    for (int i = 0; i < 1000; ++i) out[i] = a[i];
}
""")
    subprocess.run([HIPCC, *FLAGS, "-w", str(src), "-o", str(lib)], check=True, capture_output=True)
    found = scratch_bytes(str(lib))
    assert len(found) == 1 and "spills" in next(iter(found)) and next(iter(found.values())) >= 4000


INSTRUCTIONS = """
0000000000001000 <kernel>:
	{}
	s_cbranch_scc1 L0
	s_mov_b32 s9, 0
	s_branch L1
<L0>:
	{}
<L1>:
	global_load_dwordx4 v[0:3], v4, s[2:3]
	s_endpgm
"""


@pytest.mark.parametrize("first,second,found", [
    ("v_readfirstlane_b32 s3, v1", "s_nop 2", True),        # four on one way, three on the other
    ("v_readfirstlane_b32 s3, v1", "s_nop 3", True),
    ("s_nop 0", "v_readlane_b32 s2, v1, 3", True),
    ("v_readfirstlane_b32 s4, v1", "s_nop 0", False),       # another register
    ("s_mov_b32 s3, s1", "s_nop 0", False),                 # a scalar instruction wrote it
    ("v_readfirstlane_b32 s3, v1\n\ts_mov_b64 s[2:3], s[4:5]", "s_nop 0", False),
    ("v_readfirstlane_b32 s3, v1\n\ts_nop 4", "s_nop 0", False),
    ("v_cmp_gt_u32_e64 s[2:3], s7, v0", "s_nop 0", True),
    ("v_add_u32_e32 v1, s3, v1", "s_nop 0", False),         # read, not written
    ("v_add_co_u32_e64 v1, s[2:3], v1, v2", "s_nop 0", True),
])
def test_distances_over_all_ways_to_an_instruction(first, second, found):
    assert bool(missing_wait_states(INSTRUCTIONS.format(first, second))) == found

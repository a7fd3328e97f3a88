"""csrc/lds_reserve.h on the host, against a HIP runtime of this test's own: the reservation of a kernel's LDS belongs to a device, not to a thread."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_00960_amd.build import CSRC

PROGRAM = r"""
#include "lds_reserve.h"
#include <cstdio>
#include <thread>
#include <vector>

static thread_local int current = 0;
static int calls[80], refuse = 0;
extern "C" {
hipError_t hipGetDevice(int *dev) { *dev = current; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute attr, int bytes)
{
    if (attr != hipFuncAttributeMaxDynamicSharedMemorySize || bytes != 150000) return hipErrorUnknown;
    if (refuse) return hipErrorInvalidValue;
    ++calls[current];
    return hipSuccess;
}
}
#define EXPECT(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main()
{
    static phantom::LdsReserved first, second;
    const int kernel = 0;
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && calls[0] == 1);
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && calls[0] == 1);         // once
    current = 1;                                                                   // the same thread on another device
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && calls[1] == 1);
    EXPECT(second.reserve(&kernel, 150000) == hipSuccess && calls[1] == 2);        // another kernel
    current = 63;
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && first.reserve(&kernel, 150000) == hipSuccess && calls[63] == 1);
    current = 64;                                                                  // past the word: still reserved, every time
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && first.reserve(&kernel, 150000) == hipSuccess && calls[64] == 2);
    current = 2;
    refuse = 1;                                                                    // a refusal is reported and not remembered as done
    EXPECT(first.reserve(&kernel, 150000) == hipErrorInvalidValue && calls[2] == 0);
    refuse = 0;
    EXPECT(first.reserve(&kernel, 150000) == hipSuccess && calls[2] == 1);
    hipError_t other = hipErrorUnknown;
    std::thread([&] { current = 1; other = first.reserve(&kernel, 150000); }).join();
    EXPECT(other == hipSuccess && calls[1] == 2);                                  // another thread on a device that has it
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_once_per_device(tmp_path):
    src, exe = tmp_path / "reserve.cpp", tmp_path / "reserve"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-isystem", os.path.join(rocm, "include"), str(src), "-o", str(exe),
                    "-pthread"], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True)
    assert done.returncode == 0, done.stdout


def test_every_reservation_goes_through_it():
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".h", ".hip", ".cpp")) and name != "lds_reserve.h":
            with open(os.path.join(CSRC, name)) as f:
                text = f.read()
            assert "hipFuncSetAttribute" not in text, name
            for m in re.finditer(r"^.*\bLdsReserved (?!&).*$", text, re.M):
                assert re.match(r"\s*static LdsReserved \w+;$", m.group(0)), f"{name}: {m.group(0)}"

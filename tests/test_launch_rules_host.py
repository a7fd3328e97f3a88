"""csrc/launch_rules.h on the host: the cases of the GPU tests reach the kernels that they are there for."""
import ctypes
import shutil
import subprocess

import pytest

from paper_2508_00960_amd.build import CSRC
from test_gpu_f32_whole import FEW
from test_gpu_few_rows import LAYERS, MORE_LAYERS
from test_gpu_forward_bits import BF16, F32

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")

SOURCE = """
#include "launch_rules.h"
extern "C" int f32_few(int64_t workgroups, int64_t longest) { return phantom::f32_few_groups_for(workgroups, longest); }
extern "C" int few_rows(int64_t B, int64_t so, int64_t k, int64_t Kc) { return phantom::few_rows_blocks_for(B, so, k, Kc); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rules")
    (tmp / "rules.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(tmp / "rules.cpp"), "-o", str(tmp / "rules.so")], check=True)
    lib = ctypes.CDLL(str(tmp / "rules.so"))
    for f in (lib.f32_few, lib.few_rows):
        f.argtypes = [ctypes.c_int64] * len("xx" if f is lib.f32_few else "xxxx")
    return lib


def f32_groups(rules, held, *products):
    """groups of a launch of products (rows, columns, reduction) for each of `held` ranks"""
    tiles = sum(-(-m // 32) * -(-n // 32) * held for m, n, _ in products)
    return rules.f32_few(tiles, max(k for _, _, k in products))


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode,groups", FEW)
def test_f32_few_tiles(rules, n, p, k, B, L, act, rank, mode, groups):
    s, q, held = n // p, p - 1, p if rank < 0 else 1
    update, compress = (B, s, s + q * k), [(B, k, s)] if q else []
    gradients = [(s, s + q * k, B)] + ([(k, s, B)] if q else [])
    launches = (f32_groups(rules, held, update, *(compress if rank >= 0 else [])), f32_groups(rules, held, (B, s, s + k)), f32_groups(rules, held, *gradients))
    assert all(want is None or got == want for got, want in zip(launches, groups)), launches


@pytest.mark.parametrize("n,p,k,B,act,blocks", LAYERS + MORE_LAYERS)
def test_few_rows(rules, n, p, k, B, act, blocks):
    s = n // p
    assert rules.few_rows(B, s, k, s + (p - 1) * k) == blocks


@pytest.mark.parametrize("n,p,k,B,L,act", BF16)
def test_forward_bits_few_rows(rules, n, p, k, B, L, act):
    s = n // p
    assert rules.few_rows(B, s, k, s + (p - 1) * k) > 0


@pytest.mark.parametrize("n,p,k,B,L,act,rank", F32)
def test_forward_bits_f32_lines(rules, n, p, k, B, L, act, rank):
    s, held = n // p, p if rank < 0 else 1
    update, compress = (B, s, s + (p - 1) * k), (B, k, s)
    assert f32_groups(rules, held, update) > 0
    assert rank < 0 or f32_groups(rules, held, update, compress) == 0


@pytest.mark.parametrize("B,so,k,Kc,blocks", [
    (40, 1280, 40, 1560, 2),         # 33 workgroups of one block on some XCDs
    (96, 1280, 40, 1560, 4),         # ... of two
    (64, 1472, 0, 1472, 2),
    (64, 1536, 0, 1536, 0),          # dense: gemm_flex.h's teams are evenly loaded, and it is the faster one
    (64, 2048, 0, 2048, 0),
    (32, 2048, 0, 2048, 1),
    (128, 1024, 0, 1024, 2),
    (728, 288, 32, 768, 0),          # two teams, one workgroup to a compute unit: 36 of the update on an XCD
    (662, 312, 40, 912, 0),          # ... 33
    (637, 288, 56, 680, 4),          # ... 30, and 10 of the short compression in a second round
    (257, 704, 8, 824, 0),           # ... a long one
    (476, 400, 8, 520, 4),           # ... at the line
    (146, 768, 8, 824, 4),           # ... 30 and 5 of two blocks; one step more fits
    (609, 144, 8, 200, 2),           # two to a compute unit: 40 of the update
])
def test_few_rows_lines(rules, B, so, k, Kc, blocks):
    assert rules.few_rows(B, so, k, Kc) == blocks

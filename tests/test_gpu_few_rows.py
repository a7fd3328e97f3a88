"""The forward kernel for a batch of few rows (csrc/few_rows.h) where it can go wrong: one row and the edges of its blocks of 16 rows and 16
columns; reductions of less than one chunk of 32, with wavefronts that have none, and of more chunks than are in flight; head blocks and segments at every
alignment that 8-element vectors allow.  Element by element against the oracle, at the bar of the other kernels."""
import numpy as np
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from stage_check import check_stages
from test_gpu_parity import run_layer_one_rank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,act", [
    (8, 1, 0, 1, "identity"),        # a quarter of a chunk
    (16, 2, 8, 1, "gelu"),           # one row, shard 8, half a chunk
    (80, 2, 24, 15, "relu"),         # shard 40: head block and segment straddle chunks
    (192, 8, 8, 17, "gelu"),         # shard 24, segments of 8
    (2048, 8, 16, 16, "relu"),       # 1 block of rows
    (8192, 8, 64, 48, "gelu"),
    (8192, 8, 64, 49, "relu"),       # 2 blocks
    (8192, 8, 64, 113, "gelu"),      # 4 blocks
    (6080, 8, 24, 81, "relu"),       # shard 760: the last tile of columns is half empty
    (8192, 16, 256, 33, "identity"), # 17 chunks a wavefront: more than are in flight, 1 block
    (8192, 16, 160, 130, "relu"),    # ... 2 blocks
    (5120, 4, 200, 97, "gelu"),      # past the line: gemm_flex.h
    (1024, 4, 16, 768, "relu"),      # many blocks of rows
])
def test_layer(n, p, k, B, act):
    print(f"case few rows layer n={n} p={p} k={k} B={B} {act}", flush=True)
    run_layer_one_rank(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype="bf16", rank=p - 1), seed=3)


# The cases of test_layer, and the blocks of 16 rows that a workgroup takes (test_launch_rules_host.py)
LAYERS = [
    (8, 1, 0, 1, "identity", 1),        # a quarter of a chunk
    (16, 2, 8, 1, "gelu", 1),           # one row, shard 8, half a chunk
    (80, 2, 24, 15, "relu", 1),         # shard 40: head block and segment straddle chunks
    (192, 8, 8, 17, "gelu", 1),         # shard 24, segments of 8
    (2048, 8, 16, 16, "relu", 1),
    (8192, 8, 64, 48, "gelu", 1),
    (8192, 8, 64, 49, "relu", 2),
    (8192, 8, 64, 113, "gelu", 4),      # 4 to 6 chunks a wavefront, 3 of them in flight
    (6080, 8, 24, 81, "relu", 2),       # shard 760: the last tile of columns is half empty
    (8192, 16, 256, 33, "identity", 1), # 16 to 18 chunks a wavefront, 8 of them in flight
    (8192, 16, 160, 130, "relu", 2),    # ... 10 to 12, 6 of them
    (5120, 4, 200, 97, "gelu", 0),      # past the line: gemm_flex.h
    (1024, 4, 16, 768, "relu", 4),      # many blocks of rows
]
MORE_LAYERS = [
    (5120, 4, 168, 97, "gelu", 4),      # 6 to 8 chunks a wavefront, 3 of them in flight
    (1600, 2, 144, 60, "relu", 1),      # two teams: 944 indices, the longest; half a chunk left over
    (1280, 2, 312, 200, "gelu", 4),     # ... 952, 4 blocks: all of the LDS
]


@pytest.mark.parametrize("n,p,k,B,act,blocks", MORE_LAYERS)
def test_layer_with_all_blocks(n, p, k, B, act, blocks):
    test_layer(n, p, k, B, act)


@pytest.mark.parametrize("n,p,k,B,L,act,mode", [
    (8192, 8, 64, 48, 3, "relu", "forward"),
    (8192, 8, 64, 70, 2, "gelu", "forward"),
    (2048, 8, 20, 40, 2, "gelu", "forward"),       # on padded copies
    (2048, 8, 16, 33, 3, "gelu", "train"),         # sigma' kept in float; the last layer goes another way
    (1024, 2, 40, 30, 3, "relu", "train"),
    (512, 1, 0, 48, 3, "gelu", "no_update"),
])
def test_step_every_stage(n, p, k, B, L, act, mode):
    print(f"case few rows stages n={n} p={p} k={k} B={B} L={L} {act} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=0), seed=5, lr=0.02, mode=mode)


def test_rows_past_the_end_and_infinities():
    """An infinity in one row stays in that row, also where rows repeat and the reduction's last chunk is cleared."""
    n, p, k, B = 320, 4, 24, 19                    # shard 80 + 72: the last chunk is three quarters full
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *shape: (torch.randn(shape, device="cuda", generator=gen) * 0.1).bfloat16()
    s, q = n // p, p - 1
    prob = ph.make_problem(n, p, k, B, 1, "relu", "bf16", 0)
    X, G = rand(B, s), rand(q, B, k)
    X[B - 1, s - 1], G[q - 1, 3, k - 1] = float("inf"), float("-inf")
    Lw, Cw, Dw, bias = rand(s, s), rand(k, s), rand(q, s, k), rand(s)
    Y, g = torch.empty_like(X), torch.empty((B, k), device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(ph.workspace_bytes(prob), device="cuda", dtype=torch.uint8)
    ph.layer_fwd(prob, X, Lw, Cw, Dw, bias, G, Y, g, None, ws)
    pre = X.double() @ Lw.double().T + sum(G[i].double() @ Dw[i].double().T for i in range(q)) + bias.double()
    own = X.double() @ Cw.double().T
    for got, want in ((Y, pre.clamp(min=0)), (g, own)):
        assert torch.equal(torch.isfinite(got), torch.isfinite(want))
        fine = torch.isfinite(want)
        assert torch.equal(got.double()[~fine], want[~fine])
        assert (got.double()[fine] - want[fine]).abs().max() <= 2 ** -8 * want[fine].abs().max() + 1e-6

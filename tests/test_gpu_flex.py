"""The kernels for any shape and storage type (csrc/gemm_flex.h) at the sizes where they can go wrong: around their tiles
(32 and 64) and vectors (4 and 8 elements), widths and phantom widths that no vector divides, buffers shorter than one
vector, and each of their tile shapes.  Element by element against the oracle."""
import pytest

import phantom_inputs as pin

from stage_check import check_stages
from test_gpu_parity import run_layer_all_ranks, run_layer_one_rank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,p,k,B,act", [
    (2, 2, 1, 1, "identity"),        # one neuron, one row: every buffer is shorter than a vector
    (9, 3, 2, 3, "gelu"),
    (21, 3, 7, 5, "relu"),           # shard 7 = k
    (63, 1, 0, 33, "gelu"),          # around one tile
    (130, 2, 64, 31, "relu"),        # shard 65
    (268, 4, 9, 127, "gelu"),        # shard 67: rows that start on no vector, segments of 9
    (1030, 2, 33, 65, "relu"),       # shard 515
    (2002, 2, 5, 300, "gelu"),       # shard 1001: tiles enough for 64 x 64 with two teams
    (2002, 2, 129, 1030, "relu"),    # ... and with one
])
def test_layer_of_odd_sizes(n, p, k, B, act, dtype):
    print(f"case flex layer n={n} p={p} k={k} B={B} {act} {dtype}", flush=True)
    run_layer_one_rank(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype=dtype, rank=p - 1), seed=3)
    if p > 1 and n * B < 200000:
        run_layer_all_ranks(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype=dtype, rank=-1))


@pytest.mark.parametrize("n,p,k,B,L,act,dtype,rank,mode", [
    (6, 3, 1, 2, 2, "gelu", "bf16", -1, "train"),
    (201, 3, 11, 70, 4, "gelu", "bf16", -1, "train"),        # all ranks, four layers: three error buffers in turn
    (402, 2, 13, 90, 5, "relu", "bf16", 1, "train"),         # one rank: the layer below's launch carries the gradients
    (402, 2, 13, 90, 3, "relu", "f32", 0, "no_update"),
    (402, 2, 13, 90, 3, "identity", "bf16", 0, "train"),
    (1024, 2, 64, 512, 3, "gelu", "bf16", 0, "train"),       # shapes of the 128 x 128 kernels, too few tiles for them
    (300, 1, 0, 130, 4, "relu", "f32", 0, "train"),          # dense
    (700, 7, 100, 64, 2, "relu", "f32", -1, "forward"),      # k = shard
])
def test_step_every_stage(n, p, k, B, L, act, dtype, rank, mode):
    print(f"case flex stages n={n} p={p} k={k} B={B} L={L} {act} {dtype} rank={rank} {mode}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype=dtype, rank=rank)
    check_stages(prob, seed=5, lr=0.02, mode=mode)

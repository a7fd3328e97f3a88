"""Tiles at the edges of an operand's pieces, where kernels take a path of their own.  Against the oracle.

Weight gradients of widths that 4 and not 8 divides: tiles that straddle the head block and the peers' segments, in a reduction of less than
one step, of a few and of many, with one and with two tiles per workgroup.

What the epilogue of the kernels without the ring reads ahead: whole vectors only, those that the end of a piece cuts it reads for itself.
"""
import pytest

import phantom_inputs as pin

from stage_check import check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode", [
    (592, 4, 4, 63, 2, "relu", -1, "train"),         # shard 148: the straddling tile is the last one; part of a step
    (592, 4, 12, 64, 2, "gelu", -1, "no_update"),    # one whole step
    (1072, 4, 28, 130, 3, "relu", -1, "train"),      # shard 268, two steps and a part, an odd number for the two teams
    (4784, 4, 32, 600, 2, "gelu", 1, "train"),       # shard 1196, one rank; so few tiles that gemm_flex.h takes them, as in the next
    (5464, 2, 12, 333, 2, "relu", 0, "train"),
    (4784, 4, 32, 1300, 2, "gelu", 1, "train"),      # one rank on the 128 x 128 kernels: two teams on a tile
    (4216, 2, 12, 1600, 1, "relu", 0, "train"),      # shard 2108, 306 tiles: two tiles per workgroup
    (4216, 2, 12, 1400, 1, "relu", 1, "train"),      # ... one team per workgroup (a batch of at most 1536)
    (6336, 16, 12, 1600, 1, "gelu", -1, "no_update"),        # shard 396, all ranks, 320 + 64 tiles: two per workgroup
])
def test_straddling_tiles_of_weight_gradients(n, p, k, B, L, act, rank, mode):
    print(f"case straddling n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=rank), seed=9, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,p,k,B,L,act,dtype,rank,mode", [
    (36, 4, 3, 17, 2, "relu", "f32", -1, "train"),       # shard 9: vectors of 4 at the pieces' ends are not whole; 32 x 32 tiles
    (132, 4, 5, 33, 2, "gelu", "f32", -1, "no_update"),  # shard 33: a tile of one column
    (66, 2, 7, 65, 3, "relu", "bf16", -1, "train"),      # shard 33, vectors of 8
    (1300, 4, 9, 321, 2, "gelu", "bf16", -1, "train"),   # shard 325: 64 x 64 tiles, one and two passes
    (750, 1, 0, 500, 3, "gelu", "bf16", 0, "train"),     # dense
    (2002, 2, 33, 290, 2, "relu", "bf16", 1, "train"),   # shard 1001, one rank
])
def test_what_the_epilogue_reads(n, p, k, B, L, act, dtype, rank, mode):
    print(f"case epilogue reads n={n} p={p} k={k} B={B} L={L} {act} {dtype} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype=dtype, rank=rank), seed=10, lr=0.02, mode=mode)

"""fp32 on the fp32 matrix instructions where 4 divides the widths: against the oracle where steps, segments and tiles end."""
import pytest

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from stage_check import check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,L,rank", [
    (1040, 4, 4, 2100, 2, -1),       # shard 260, segments of one vector: every step of the cut part on its own; 660 workgroups forward
    (2048, 8, 16, 1100, 2, -1),      # two segments a step; 576 workgroups
    (4128, 8, 12, 130, 2, -1),       # shard 516: weight-gradient tiles that straddle the cut, 720 workgroups; a batch that 4 does not divide
    (2048, 4, 64, 300, 2, -1),       # two steps a segment, two workgroups to a compute unit
    (1536, 4, 96, 33, 2, -1),        # three steps a segment, a reduction of 33 rows
    (1032, 2, 8, 2500, 2, 1),        # one rank
    (96, 2, 4, 3, 2, -1),            # shorter than a step in every direction
])
def test_parity(n, p, k, B, L, rank):
    print(f"case f32 whole n={n} p={p} k={k} B={B} L={L} rank={rank}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act="relu", dtype="f32", rank=rank), seed=12, lr=0.02, mode="train")


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode", [
    (256, 4, 8, 32, 2, "relu", -1, "train"),
    (288, 4, 12, 127, 3, "gelu", -1, "train"),       # shard 72 + 36: tiles of eight and four columns left over; 127 terms in the weight gradients
    (384, 4, 8, 128, 2, "relu", 1, "train"),         # one rank, 120 and 128 terms: all teams
    (20, 5, 4, 2, 3, "gelu", -1, "no_update"),       # shard 4 = k: one team with terms, one vector to a piece
    (64, 1, 0, 16, 2, "relu", 0, "train"),           # dense
    (512, 8, 4, 36, 2, "identity", -1, "forward"),
    (512, 4, 16, 130, 2, "gelu", -1, "train"),       # two groups to a team: 176 and 130 terms
    (1008, 4, 4, 256, 2, "relu", -1, "train"),       # ... 264: four, the last of them in part; 256: two
    (1024, 4, 64, 500, 2, "gelu", -1, "train"),      # 448, 320 and 500 terms in 512 and more tiles: past the line
    (512, 1, 0, 512, 2, "relu", 0, "train"),         # dense, 512 terms: all groups of all teams
    (768, 3, 120, 90, 3, "identity", 2, "train"),    # one rank
    (1024, 8, 20, 300, 2, "relu", -1, "no_update"),  # reduce-scatter on read with segments of 20
    (576, 9, 8, 100, 2, "gelu", -1, "train"),        # nine ranks: a launch for the sums
])
def test_few_tiles_and_short_reductions(n, p, k, B, L, act, rank, mode):
    """32 x 32 tiles, one, two or four groups of 16 terms to each of eight teams."""
    print(f"case f32 few n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="f32", rank=rank), seed=12, lr=0.02, mode=mode)


# ..., (groups of 16 terms to a team in the update, the input gradient, the first layer's gradients; 0: another kernel; None: it shares its launch)
FEW = [
    (256, 4, 8, 32, 2, "relu", -1, "train", (1, 1, 1)),
    (288, 4, 12, 127, 3, "gelu", -1, "train", (1, 1, 1)),       # shard 72 + 36: tiles of eight and four columns left over; 127 terms in the weight gradients
    (384, 4, 8, 128, 2, "relu", 1, "train", (1, None, 1)),      # one rank, 120 and 128 terms: all teams
    (20, 5, 4, 2, 3, "gelu", -1, "no_update", (1, 1, 1)),       # shard 4 = k: one team with terms, one vector to a piece
    (64, 1, 0, 16, 2, "relu", 0, "train", (1, None, 1)),        # dense
    (512, 8, 4, 36, 2, "identity", -1, "forward", (1, None, None)),
    (512, 4, 16, 130, 2, "gelu", -1, "train", (2, 2, 2)),       # 176, 144 and 130 terms
    (1008, 4, 4, 256, 2, "relu", -1, "train", (4, 2, 2)),       # 264 in the update: the last of the four in part; 256: all of two
    (1024, 4, 64, 500, 2, "gelu", -1, "train", (0, 0, 0)),      # 448, 320 and 500 terms in 512 and more tiles: past the line
    (1024, 4, 64, 250, 2, "gelu", -1, "train", (4, 4, 2)),      # 448 and 320 terms in 256 tiles: at it
    (512, 4, 16, 300, 2, "relu", -1, "train", (2, 2, 4)),       # 300 terms: the compressor gradient sums three groups on read, the last of them in part
    (512, 4, 16, 512, 1, "identity", -1, "no_update", (2, None, 4)),   # one layer; 512: all groups of all teams
    (896, 2, 64, 288, 3, "gelu", -1, "train", (4, 4, 0)),       # ... of the input gradient; one sender; a launch for the first layer's sums
    (2048, 8, 32, 100, 2, "relu", -1, "no_update", (4, 4, 0)),  # seven senders, a group that is partly dg_own
    (512, 1, 0, 512, 2, "relu", 0, "train", (4, None, 4)),      # dense, 512 terms: all groups of all teams
    (768, 3, 120, 90, 3, "identity", 2, "train", (4, None, 1)),     # one rank
    (1024, 8, 20, 300, 2, "relu", -1, "no_update", (0, 2, 0)),  # reduce-scatter on read with segments of 20; the first layer's in a launch of its own
    (576, 9, 8, 100, 2, "gelu", -1, "train", (1, 1, 1)),        # nine ranks: a launch for the sums
]


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode,groups", FEW)
def test_groups_of_terms_and_sums_on_read(n, p, k, B, L, act, rank, mode, groups):
    """32 x 32 tiles, one, two or four groups of 16 terms to each of eight teams (that the rule says so: test_launch_rules_host.py)."""
    print(f"case f32 few n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    ph.profile_begin()
    try:
        check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="f32", rank=rank), seed=12, lr=0.02, mode=mode)
    finally:
        launches = ph.profile_end()
    if rank < 0 and mode != "forward":
        # a launch for the sums of dg_own where the launch that needs them first does not add them up on read
        apart = sum(e["calls"] for e in launches if e["name"] == "reduce-scatter")
        assert apart == (L if p > 8 else (L - 1) * (groups[1] == 0) + (groups[2] == 0))

"""fp32 on the fp32 matrix instructions where 4 divides the widths (ReLU training): against the oracle where steps, segments and tiles end."""
import pytest

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

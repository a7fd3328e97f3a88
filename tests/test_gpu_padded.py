"""One rank's bf16 step on padded copies of what the phantom width cuts into rows (widths that 8 divides, phantom widths that it does not): every
stage against the oracle, and infinities, which the zeros must not meet."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import workspace
from stage_check import check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,L,act,mode,widths,ks", [
    (2048, 2, 4, 2100, 2, "relu", "train", None, None),               # 128 x 128 kernels, 4-element vectors without the copies
    (2048, 2, 4, 2100, 2, "gelu", "forward", None, None),
    (2048, 2, 10, 2100, 3, "gelu", "train", None, None),              # rows of 20 bytes
    (4096, 2, 2, 1100, 2, "relu", "train", None, None),               # the gradients of large layers together
    (1024, 16, 44, 130, 2, "relu", "no_update", None, None),          # shard 64: long peers' parts, few tiles; gradients handed out
    (1024, 16, 62, 67, 2, "gelu", "train", None, None),
    (2048, 8, 100, 300, 2, "relu", "forward", None, None),            # more than 64: the compressions of all layers together
    (8192, 8, 32, 1100, 2, "relu", "train", (8192, 8192, 4096), (20, 32)),       # one layer's phantom width is left as it is; a table
])
def test_parity(n, p, k, B, L, act, mode, widths, ks):
    print(f"case padded n={n} p={p} k={k} B={B} L={L} {act} {mode}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=0, widths=widths, ks=ks)
    check_stages(prob, seed=8, lr=0.02, mode=mode)


def test_infinities():
    """An infinite input element reaches its own row of the output alone, an infinite element of a peer's buffer likewise."""
    print("case padded infinities", flush=True)
    n, p, k, B = 2048, 2, 10, 2100
    s, q = n // p, p - 1
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *shape: torch.rand(shape, device="cuda", generator=gen).bfloat16() + 0.5      # (positive: infinities do not meet)
    X, G = rand(B, s), [rand(q, B, k)]
    W = {"Lw": [rand(s, s)], "Cw": [rand(k, s)], "Dw": [rand(q, s, k)], "bias": [rand(s)]}
    X[5, 7], G[0][0, 70, k - 1] = float("inf"), float("inf")
    Y = torch.zeros(B, s, device="cuda", dtype=torch.bfloat16)
    pc = ph.make_problem(n, p, k, B, 1, "relu", "bf16", 0)
    ph.ffn_step(pc, X, None, W["Lw"], W["Cw"], W["Dw"], W["bias"], G=G, Y_out=Y, mode="forward", workspace=workspace(ph.workspace_bytes(pc)))
    torch.cuda.synchronize()
    infinite = torch.zeros(B, s, dtype=torch.bool, device="cuda")
    infinite[5], infinite[70] = True, True
    assert torch.equal(torch.isinf(Y), infinite) and not torch.isnan(Y).any()

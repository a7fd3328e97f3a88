"""One rank's bf16 step on padded copies of what the phantom width cuts into rows (widths that 8 divides, phantom widths that it does not): every
stage against the oracle, and infinities, which the zeros must not meet."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import empty_f32, to_gpu, to_gpu_f32, workspace
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


def test_gradients_that_nobody_takes():
    """Layers alike on the copies, of which some need none, deltas where a launch per layer has its gradients: the weights come out the same, bit for
    bit, whether or not the caller takes the gradients (the launches add the same terms in the same order)."""
    print("case padded, gradients not taken", flush=True)
    n, p, B, L, ks = 4096, 2, 1100, 4, (28, 32, 28, 32)
    prob = pin.Problem(n=n, p=p, k=32, batch=B, layers=L, act="relu", dtype="bf16", rank=0, widths=(n,) * (L + 1), ks=ks)
    data = pin.one_rank_step_inputs(prob, 3)
    pc = ph.make_problem(n, p, 32, B, L, "relu", "bf16", 0, widths=prob.widths, ks=ks)
    names = ("Lw", "Cw", "Dw", "bias")
    outs = []
    for taken in (True, False):
        W = {nm: [to_gpu(P[nm], "bf16") for P in data["layers"]] for nm in names}
        M = {nm: [to_gpu_f32(P[nm]) for P in data["layers"]] for nm in names}
        Gd = {nm: [empty_f32(P[nm].shape) for P in data["layers"]] if taken else None for nm in names}
        ph.ffn_step(pc, to_gpu(data["X0"], "bf16"), to_gpu(data["T"], "bf16"), W["Lw"], W["Cw"], W["Dw"], W["bias"], Lw_master=M["Lw"], Cw_master=M["Cw"],
                    Dw_master=M["Dw"], bias_master=M["bias"], G=[to_gpu(P["G"], "bf16") for P in data["layers"]],
                    dg_own=[to_gpu(P["dg_own"], "bf16") for P in data["layers"]], dLw=Gd["Lw"], dCw=Gd["Cw"], dDw=Gd["Dw"], dbias=Gd["bias"],
                    loss=empty_f32((4,)), lr=0.02, mode="train", workspace=workspace(ph.workspace_bytes(pc)))
        torch.cuda.synchronize()
        outs.append(M)
    for nm in ("Lw", "Cw", "Dw"):                      # (the bias gradients are added with atomics)
        for l in range(L):
            assert torch.equal(outs[0][nm][l], outs[1][nm][l]), (nm, l)


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

"""Calls whose output lies over an input, where include/phantom.h allows it: the same bits as with buffers of their own."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import empty, empty_f32, to_gpu, to_gpu_f32, workspace

pytestmark = pytest.mark.gpu


def run_step(prob, over, mode):
    """One step; over: the input that Y_out lies over ("X0", "T", "G") or None.  Returns its outputs by name."""
    dt, q, L = prob.dtype, prob.peers, prob.layers
    one = prob.rank >= 0
    data = pin.one_rank_step_inputs(prob, 3) if one else pin.all_rank_step_inputs(prob, 3)
    pc = ph.make_problem(prob.n, prob.p, prob.k, prob.batch, L, prob.act, dt, prob.rank)
    ws = workspace(ph.workspace_bytes(pc))
    ws.fill_(0xFF)
    names = ["Lw", "bias"] + (["Cw", "Dw"] if q else [])
    train = mode != "forward"
    W = {nm: [to_gpu(P[nm], dt) for P in data["layers"]] for nm in names}
    M = {nm: [to_gpu_f32(P[nm]) for P in data["layers"]] for nm in names} if (dt == "bf16" and mode == "train") else {}
    Gd = {nm: [empty_f32(P[nm].shape) for P in data["layers"]] for nm in names} if train else {}
    G = [to_gpu(P["G"], dt) for P in data["layers"]] if (q and one) else None
    dg = [to_gpu(P["dg_own"], dt) for P in data["layers"]] if (q and one and train) else None
    X0, T = to_gpu(data["X0"], dt), to_gpu(data["T"], dt)
    Y = {None: empty(data["T"].shape, dt), "X0": X0, "T": T, "G": G[0] if G else None}[over]
    loss = empty_f32((4,))
    ph.ffn_step(pc, X0, T if train else None, W["Lw"], W.get("Cw"), W.get("Dw"), W["bias"], Lw_master=M.get("Lw"),
                Cw_master=M.get("Cw"), Dw_master=M.get("Dw"), bias_master=M.get("bias"), G=G, dg_own=dg, dLw=Gd.get("Lw"),
                dCw=Gd.get("Cw"), dDw=Gd.get("Dw"), dbias=Gd.get("bias"), Y_out=Y, loss=loss if train else None, lr=0.02,
                mode=mode, workspace=ws)
    torch.cuda.synchronize()
    out = {"Y": Y.flatten()[:data["T"].size].clone()}
    if train:
        out["loss"] = loss[:1].clone()
        for kind in (Gd, W, M):
            for nm, per_layer in kind.items():
                if nm != "bias":               # (column sums added up with float atomics: their last bits vary by design)
                    out.update({f"{len(out)} {nm}[{l}]": t.clone() for l, t in enumerate(per_layer)})
    return out


@pytest.mark.parametrize("over,mode,n,p,k,B,L,act,dtype,rank", [
    ("X0", "forward", 128, 2, 8, 96, 1, "relu", "f32", 0),
    ("X0", "forward", 260, 2, 9, 200, 1, "gelu", "bf16", 1),           # odd phantom width
    ("X0", "forward", 4096, 2, 64, 2100, 1, "relu", "bf16", 0),        # 128 x 128 tiles
    ("X0", "forward", 2048, 4, 16, 300, 1, "relu", "bf16", -1),        # all ranks
    ("X0", "train", 128, 2, 8, 96, 2, "gelu", "f32", 0),               # the first layer's weight gradient reads X0 last
    ("X0", "train", 2048, 4, 16, 300, 2, "relu", "bf16", -1),
    ("T", "train", 128, 2, 8, 96, 2, "relu", "f32", -1),
    ("T", "no_update", 260, 2, 9, 200, 2, "gelu", "bf16", 0),
    ("T", "train", 4096, 2, 64, 2100, 2, "gelu", "bf16", 0),
    ("T", "train", 2048, 4, 16, 300, 2, "relu", "bf16", -1),
    ("G", "train", 128, 2, 64, 96, 2, "relu", "f32", 0),               # the first layer's peer buffer, as wide as the output
])
def test_step_output_over_an_input(over, mode, n, p, k, B, L, act, dtype, rank):
    print(f"case overlap step {over} {mode} n={n} p={p} k={k} B={B} L={L} {act} {dtype} rank={rank}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype=dtype, rank=rank)
    want, got = run_step(prob, None, mode), run_step(prob, over, mode)
    assert want.keys() == got.keys()
    for name, t in want.items():
        assert bool(torch.isfinite(t.float()).all()), name
        assert torch.equal(t, got[name]), name

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
    ("X0", "forward", 2048, 4, 16, 300, 1, "relu", "bf16", -1),        # all ranks, few tiles
    ("X0", "forward", 2048, 4, 16, 1700, 1, "relu", "bf16", -1),       # ... 128 x 128 tiles
    ("X0", "train", 128, 2, 8, 96, 2, "gelu", "f32", 0),               # the first layer's weight gradient reads X0 last
    ("X0", "train", 2048, 4, 16, 300, 2, "relu", "bf16", -1),
    ("X0", "train", 2048, 4, 16, 1700, 2, "relu", "bf16", -1),
    ("T", "train", 128, 2, 8, 96, 2, "relu", "f32", -1),
    ("T", "no_update", 260, 2, 9, 200, 2, "gelu", "bf16", 0),
    ("T", "train", 4096, 2, 64, 2100, 2, "gelu", "bf16", 0),
    ("T", "train", 2048, 4, 16, 300, 2, "relu", "bf16", -1),
    ("T", "train", 2048, 4, 16, 1700, 2, "relu", "bf16", -1),
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


def run_layer_bwd(prob, over):
    """A layer's backward call; over: "dX" lies over dY, "A" dX lies over the pre-activation, None: nothing overlaps."""
    dt, q, p = prob.dtype, prob.peers, prob.p
    one = prob.rank >= 0
    lead = () if one else (p,)
    P = (pin.one_rank_step_inputs(prob, 4) if one else pin.all_rank_step_inputs(prob, 4))["layers"][0]
    B, s, k = prob.batch, prob.s_in(0), prob.k_of(0)
    pc = ph.make_problem(prob.n, p, prob.k, B, 1, prob.act, dt, prob.rank)
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen).to(torch.float32 if dt == "f32" else torch.bfloat16)

    dY, X, A = normal(*lead, B, s), normal(*lead, B, s), normal(*lead, B, s)
    dg_own = normal(*lead, B, k) if q else None
    G = (normal(q, B, k) if one else normal(p, B, k)) if q else None
    dX = {"dX": dY, "A": A, None: empty(lead + (B, s), dt)}[over]
    grads = {nm: empty_f32(P[nm].shape) for nm in P if nm in ("Lw", "Cw", "Dw", "bias")}
    W = {nm: to_gpu(P[nm], dt) for nm in grads}
    dG_send = empty(lead + (q, B, k), dt) if q else None
    ph.layer_bwd(pc, dY, X, A, W["Lw"], W.get("Cw"), W.get("Dw"), G, dg_own, dX, grads["Lw"], grads.get("Cw"), grads.get("Dw"),
                 grads["bias"], dG_send, workspace(ph.workspace_bytes(pc)))
    torch.cuda.synchronize()
    return {"dX": dX, "dG_send": dG_send, "dg_own": dg_own, **{"d" + nm: t for nm, t in grads.items() if nm != "bias"}}


@pytest.mark.parametrize("over,n,p,k,B,act,dtype,rank", [
    ("dX", 128, 2, 8, 96, "identity", "f32", 0),
    ("dX", 390, 3, 7, 130, "identity", "bf16", 2),
    ("dX", 4096, 2, 64, 2100, "identity", "bf16", 0),          # 128 x 128 tiles
    ("dX", 4096, 4, 16, 1100, "identity", "bf16", -1),
    ("dX", 128, 1, 0, 96, "identity", "f32", 0),
    ("dX", 390, 3, 7, 130, "gelu", "bf16", 2),
    ("A", 4096, 4, 16, 1100, "relu", "bf16", -1),
    ("A", 128, 2, 8, 96, "gelu", "f32", 0),
])
def test_layer_gradient_over_an_input(over, n, p, k, B, act, dtype, rank):
    print(f"case overlap layer {over} n={n} p={p} k={k} B={B} {act} {dtype} rank={rank}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype=dtype, rank=rank)
    want, got = run_layer_bwd(prob, None), run_layer_bwd(prob, over)
    for name, t in want.items():
        assert t is None or torch.equal(t, got[name]), name


@pytest.mark.parametrize("n,p,k,B,act,dtype", [
    (128, 2, 8, 96, "relu", "f32"),
    (390, 3, 7, 136, "gelu", "bf16"),
    (4096, 2, 32, 4200, "relu", "bf16"),           # 128 x 128 tiles, thin compression
    (4096, 2, 96, 4200, "relu", "bf16"),           # ... and a product of its own
])
def test_own_phantom_layer_over_the_peers(n, p, k, B, act, dtype):
    print(f"case overlap g_own n={n} p={p} k={k} B={B} {act} {dtype}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype=dtype, rank=0)
    d = {nm: to_gpu(v, dtype) for nm, v in pin.one_rank_layer_inputs(prob, 0, 6).items()}
    pc = ph.make_problem(n, p, k, B, 1, act, dtype, 0)
    out = []
    for over in (False, True):
        G = d["G"].clone()
        Y, g_own = empty((B, n // p), dtype), G[p - 2] if over else empty((B, k), dtype)
        ph.layer_fwd(pc, d["X"], d["Lw"], d["Cw"], d["Dw"], d["bias"], G, Y, g_own, None, workspace(ph.workspace_bytes(pc)))
        torch.cuda.synchronize()
        out.append((Y, g_own))
    assert torch.equal(out[0][0], out[1][0])
    # the two schedules may split the compression's sum differently: fp32 sums that differ by their own rounding errors (some
    # 1e-7 of values around 1), which moves a bf16 result by one unit of its last place at most (2^-7 of the value)
    assert torch.allclose(out[0][1].float(), out[1][1].float(), rtol=1e-5 if dtype == "f32" else 2 ** -7, atol=1e-6)

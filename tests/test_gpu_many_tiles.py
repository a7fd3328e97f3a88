"""Steps with more 128 x 128 tiles than compute units in one-team workgroups (all ranks), and one rank's steps and layer calls
with more 128 x 128 tiles than gemm_flex.h takes, at the smallest sizes that still reach each launch: the compressions of all
layers together, all layers' gradients in one launch (equal layers: blocks in the kernel arguments; different ones: a
table), compressor gradients in one to four pieces, a launch per layer, and more layers than one list of clears holds.
Against the oracle, batches ragged."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import workspace
from stage_check import check_stages
from test_gpu_parity import run_layer_one_rank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode,widths,ks", [
    (8192, 8, 32, 1630, 3, "relu", 1, "train", None, None),            # 13 x 8 tiles, the compressor gradients whole
    (8192, 8, 32, 2100, 2, "gelu", 0, "no_update", None, None),        # in two pieces, gradients handed out
    (4096, 8, 16, 3150, 9, "relu", 0, "train", None, None),            # in three, nine layers
    (4096, 8, 128, 4099, 3, "relu", 7, "train", None, None),           # in four; k > 64: compressions of all layers together
    (8192, 8, 68, 1630, 2, "gelu", 0, "train", None, None),            # 4-element vectors: a launch per layer
    (16384, 8, 16, 1100, 2, "relu", 0, "train", None, None),           # 272 weight-gradient tiles per layer
    (4096, 8, 16, 3150, 17, "relu", 0, "no_update", None, None),       # more layers than the table holds
    (8192, 8, 32, 2100, 2, "relu", 0, "train", (8192, 4096, 12288), (32, 16)),       # layers that differ
    (2816, 2, 1408, 1990, 5, "relu", 0, "train", None, None),          # k = n/p: 605 tiles of compressor gradients in pieces
    (2816, 2, 1408, 1990, 5, "relu", 1, "no_update", (2816, 2816, 2816, 2816, 2816, 2560), (1408,) * 4 + (1400,)),   # ... by a table
])
def test_step_every_stage(n, p, k, B, L, act, rank, mode, widths, ks):
    print(f"case many tiles n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode} widths={widths}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=rank, widths=widths, ks=ks)
    check_stages(prob, seed=6, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,p,k,B,L,act,mode", [
    (2048, 64, 16, 72, 2, "relu", "train"),        # shard 32, so few tiles that gemm_flex.h takes them ...
    (2048, 64, 16, 400, 2, "relu", "train"),       # ... and more: weight gradients with the update, and the error compression, of 64 ranks
    (8192, 64, 12, 100, 2, "gelu", "no_update"),   # 4-element vectors
    (4096, 16, 16, 2100, 2, "relu", "train"),      # the input gradient; 34 tile rows, the last ragged
    (4096, 1, 0, 200, 2, "gelu", "train"),         # dense, few tiles (gemm_flex.h) ...
    (2176, 1, 0, 1000, 2, "gelu", "train"),        # ... and more: 289 weight-gradient tiles
])
def test_one_team_workgroups(n, p, k, B, L, act, mode):
    print(f"case one team n={n} p={p} k={k} B={B} L={L} {act} {mode}", flush=True)
    prob = pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=-1 if p > 1 else 0)
    check_stages(prob, seed=7, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,p,k,B,act,rank", [
    (8192, 8, 32, 3210, "relu", 3),                # 26 x 8 tiles: the compression inside the update's loop
    (8192, 8, 68, 3210, "gelu", 0),                # 4-element vectors, a compression of its own
    (16384, 8, 16, 2100, "gelu", 7),               # two-tile workgroups: the compression behind the epilogue
    (1536, 1, 0, 2200, "identity", 0),             # dense
])
def test_layer_calls_of_one_rank(n, p, k, B, act, rank):
    print(f"case many tiles layer n={n} p={p} k={k} B={B} {act} rank={rank}", flush=True)
    run_layer_one_rank(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype="bf16", rank=rank), seed=4)


@pytest.mark.parametrize("n,p,k,B,L,act,mode", [
    (4096, 2, 8, 1100, 4, "relu", "train"),          # 1088 + 64 tiles: one a workgroup; a fourth delta beside the first set of gradients
    (18432, 9, 256, 1030, 2, "gelu", "no_update"),   # 1024 + 64: two a workgroup
])
def test_all_gradients_of_large_layers_together(n, p, k, B, L, act, mode):
    print(f"case large layers n={n} p={p} k={k} B={B} L={L} {act} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=0), seed=5, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode", [
    (4160, 4, 8, 1100, 1, "relu", -1, "no_update"),       # shard 1040: half a chunk of the reduction is left; one block of 16 columns, half of it empty
    (4160, 4, 12, 1100, 1, "gelu", -1, "forward"),        # 4-element vectors in the update
    (2176, 4, 16, 2001, 1, "relu", -1, "forward"),        # shard 544: chunks that the wavefronts share unevenly; a last block of 17 rows
    (2112, 4, 24, 2000, 2, "relu", -1, "no_update"),      # shard 528, two blocks
    (4160, 4, 64, 1100, 1, "relu", -1, "forward"),        # four blocks
    (3168, 2, 24, 1200, 2, "relu", -1, "no_update"),      # shard 1584: up to seven chunks a wavefront, four in flight, behind the stores that clear the bias gradients
    (3168, 2, 64, 1200, 2, "gelu", -1, "train"),          # ... three in flight
    (4128, 2, 40, 2100, 1, "relu", 0, "forward"),         # one rank's step of one layer: behind the update's epilogue, shares of 16 rows
    (4128, 2, 24, 2100, 1, "relu", 1, "forward"),
])
def test_thin_compression(n, p, k, B, L, act, rank, mode):
    print(f"case thin n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=rank), seed=13, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,p,k,B,L", [
    (8192, 16, 64, 4096, 8),         # 416 tiles of 128 x 128, one a workgroup
    (8192, 16, 64, 2000, 8),         # ... and the last step of the range in part
    (8192, 4, 64, 4096, 2),          # more than 256 weight-gradient tiles a layer
    (16384, 16, 64, 4096, 8),        # two a workgroup, the compressor gradients in pieces
])
@pytest.mark.parametrize("mean", [0.0, 1.0])
def test_precision_of_compressor_gradients(n, p, k, B, L, mean):
    """2-norm error against 64 bits of the first layer's, whose operands are the caller's.  Sums of 32 steps of 16 terms and then those: some 1.6e-7 at 4096
    rows, with 4.0e-7 for 256 steps in one running sum."""
    print(f"case compressor gradient n={n} p={p} k={k} B={B} L={L} mean={mean}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(14)
    s, q = n // p, p - 1
    normal = lambda *shape, scale=1.0, mean=0.0: (torch.randn(shape, device="cuda", generator=gen) * scale + mean).bfloat16()
    X, T, dg = normal(B, s, mean=mean), normal(B, s), [normal(B, k, scale=1 / B, mean=mean / B) for _ in range(L)]
    G = [normal(q, B, k) for _ in range(L)]
    W = {"Lw": [normal(s, s, scale=s ** -0.5) for _ in range(L)], "Cw": [normal(k, s, scale=s ** -0.5) for _ in range(L)],
         "Dw": [normal(q, s, k, scale=(q * k) ** -0.5) for _ in range(L)], "bias": [normal(s) for _ in range(L)]}
    D = {nm: [torch.empty(w.shape, device="cuda") for w in W[nm]] for nm in W}
    pc = ph.make_problem(n, p, k, B, L, "gelu", "bf16", 0)
    ph.ffn_step(pc, X, T, W["Lw"], W["Cw"], W["Dw"], W["bias"], G=G, dg_own=dg, dLw=D["Lw"], dCw=D["Cw"], dDw=D["Dw"], dbias=D["bias"],
                loss=torch.zeros(4, device="cuda"), mode="no_update", workspace=workspace(ph.workspace_bytes(pc)))
    torch.cuda.synchronize()
    want = dg[0].double().t().contiguous() @ X.double()
    err = float((D["Cw"][0].double() - want).norm() / want.norm())
    print(f"dC {err:.2e}", flush=True)
    assert err <= 2e-7, err

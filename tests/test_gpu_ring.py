"""The reduction loop on a ring of LDS stages (csrc/mfma_ring.h), in the 64 x 64 kernel of gemm_flex.h and in the 128 x 128 ones, where it can
go wrong: reductions of fewer stages than the ring holds, of just as many, and of more; a last stage that is not full; the
head block and the peers' segments at every alignment to the stage that 8-element vectors allow; the block that is summed on
read.  Against the oracle."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import workspace
from stage_check import check_stages
from test_gpu_parity import run_layer_all_ranks, run_layer_one_rank

pytestmark = pytest.mark.gpu

# 64 x 64 tiles
SMALL = [
    (32, 4, 8, 1, "identity"),       # shard 8: one stage, half empty
    (96, 4, 24, 7, "relu"),          # shard 24, segments of 24
    (256, 4, 16, 64, "relu"),        # two stages forward, one in the weight gradients
    (288, 4, 24, 129, "gelu"),       # shard 72: stages straddle the head block's end and the segments
    (544, 4, 72, 193, "gelu"),       # shard 136; segments longer than a stage
    (640, 2, 64, 256, "relu"),
    (768, 3, 192, 321, "gelu"),      # segments of several stages; one row in the last stage
    (1312, 4, 40, 330, "relu"),      # shard 328; one team
]
# more than 192 tiles of 128 x 128
LARGE = [
    (512, 64, 8, 400, "relu"),       # shard 8
    (1536, 64, 24, 385, "gelu"),     # shard 24, segments of 24; one row in the last tile
    (2304, 32, 72, 900, "relu"),     # shard 72 = k
    (4352, 32, 8, 400, "gelu"),      # shard 136
    (6400, 32, 40, 390, "relu"),     # shard 200
    (5248, 16, 64, 530, "identity"), # shard 328, whole segments in a stage that the head block shifts
    # regular shapes: runs of stages whose loads move by a constant
    (4096, 64, 8, 1300, "relu"),     # eight segments in a stage, the skipped slot at every place in one; a run ends on either side of it
    (2048, 16, 32, 2000, "gelu"),    # two; shard 128
    (2048, 8, 128, 1700, "relu"),    # a segment of two stages: a run each
    (1536, 2, 768, 8200, "identity"), # ... of twelve
]
# between the lines of use_flex for all ranks: forward on the one kind of kernels, backward on the other
BETWEEN = [
    (1024, 16, 16, 2100, "relu"),    # 528 tiles of 64 x 64, peers' part 3.75 times the shard: 128 x 128 ones forward, 64 x 64 backward
    (2048, 16, 64, 1030, "gelu"),    # 544, peers' part 7.5 times the shard, 64 phantom neurons: the other way round
]


@pytest.mark.parametrize("n,p,k,B,act", SMALL + LARGE + BETWEEN)
def test_layer_all_ranks(n, p, k, B, act):
    print(f"case ring layer n={n} p={p} k={k} B={B} {act}", flush=True)
    run_layer_all_ranks(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype="bf16", rank=-1))


@pytest.mark.parametrize("n,p,k,B,act", [
    (272, 2, 24, 200, "gelu"),       # two teams throughout
    (2048, 2, 128, 1030, "relu"),    # one team
    (8192, 16, 8, 1500, "relu"),     # backward: few tiles with the long reduction of the weight gradients among many
])
def test_layer_one_rank(n, p, k, B, act):
    print(f"case ring layer of one rank n={n} p={p} k={k} B={B} {act}", flush=True)
    run_layer_one_rank(pin.Problem(n=n, p=p, k=k, batch=B, layers=1, act=act, dtype="bf16", rank=p - 1), seed=3)


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode", [
    (288, 4, 24, 129, 3, "gelu", -1, "train"),
    (544, 2, 40, 300, 3, "gelu", 1, "train"),
    (1024, 4, 64, 330, 2, "gelu", -1, "no_update"),
    (1040, 1, 0, 200, 3, "relu", 0, "train"),                # dense
    (2560, 8, 32, 1154, 2, "relu", -1, "train"),             # 128 x 128: the summed block in a stage of its own behind the head's
    (2048, 8, 64, 1665, 2, "gelu", -1, "no_update"),         # ... a full stage
    (8192, 8, 24, 2100, 2, "gelu", 0, "train"),              # one rank on the 128 x 128 kernels, irregular segments
    (8256, 8, 16, 2100, 2, "relu", 3, "train"),              # ... irregular shard 1032
    (8256, 8, 24, 3600, 2, "gelu", 5, "train"),              # ... both, and more than 256 tiles: two to a workgroup
    (8192, 8, 24, 4200, 2, "relu", 0, "forward"),            # ... forward only, the compression behind the epilogue
    (8256, 8, 24, 3600, 2, "relu", 1, "forward"),            # ... beside it
    (1024, 8, 16, 64, 3, "relu", 2, "train"),                # four tiles a layer: the ring backward, too
    (64, 8, 8, 33, 2, "gelu", 0, "train"),                   # ... one
    (1024, 16, 16, 2100, 2, "gelu", -1, "forward"),          # all ranks, between the lines, as above
    (2048, 16, 64, 1030, 2, "relu", -1, "train"),
    # 32 x 32 tiles, eight teams: weight gradients of more than 768 rows, forward reductions of 512, and of 960 and more
    (256, 4, 8, 1100, 2, "relu", 2, "train"),
    (128, 1, 0, 2050, 2, "gelu", 0, "train"),
    (256, 4, 16, 769, 2, "relu", -1, "no_update"),
    (512, 1, 0, 100, 2, "gelu", 0, "no_update"),             # (forward alone, and the first layer here: few rows, csrc/few_rows.h)
    (512, 1, 0, 100, 2, "gelu", 0, "forward"),
    (2048, 4, 8, 72, 2, "relu", -1, "train"),                # (the compressions of all ranks)
    (1792, 2, 64, 70, 2, "relu", 1, "no_update"),            # (... 960)
    (1792, 2, 64, 70, 2, "relu", 1, "forward"),
    (8192, 8, 64, 225, 2, "gelu", 1, "forward"),             # a forward reduction of 1472 in 256 tiles of 32 x 32
    (8192, 8, 64, 257, 2, "relu", 1, "forward"),             # ... of 64 x 64, two teams
])
def test_step_every_stage(n, p, k, B, L, act, rank, mode):
    print(f"case ring stages n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=rank), seed=8, lr=0.02, mode=mode)


@pytest.mark.parametrize("n,B,bound", [
    # 2-norm errors of a dense layer's float gradient.  A running sum of m matrix instructions' results errs by some sqrt(m / 2) roundings: eight
    # sums of m = 32 give 6.4e-8 and 7.3e-8, four of 64 9.2e-8 and 1.02e-7
    (64, 4096, 7.8e-8),
    (256, 4096, 8.7e-8),
])
def test_partial_sums_of_few_tiles(n, B, bound):
    print(f"case ring partial sums n={n} B={B}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape, scale=1.0):
        return (torch.randn(shape, device="cuda", generator=gen) * scale).bfloat16()

    X, T = normal(B, n), normal(B, n)
    Lw, bias = normal(n, n, scale=n ** -0.5), normal(n)
    delta, dLw, dbias = torch.empty_like(X), torch.empty((n, n), device="cuda"), torch.empty(n, device="cuda")
    pc = ph.make_problem(n, 1, 0, B, 1, "identity", "bf16", 0)
    ph.ffn_step(pc, X, T, [Lw], None, None, [bias], dLw=[dLw], dbias=[dbias], loss=torch.zeros(4, device="cuda"), mode="no_update",
                workspace=workspace(ph.workspace_bytes(pc)), taps={"delta": [delta]})
    torch.cuda.synchronize()
    want = delta.double().t().contiguous() @ X.double()
    err = float((dLw.double() - want).norm() / want.norm())
    print(f"dLw {err:.2e}", flush=True)
    assert err <= bound, f"{err:.2e} > {bound:.1e}"


@pytest.mark.parametrize("s,B,L", [
    (1000, 2001, 2),      # 128 tiles a layer; the last stage is five eighths full
    (2040, 3100, 2),      # 512 tiles, two to a workgroup, the gradients of both layers in one round of workgroups
    (1032, 8200, 3),      # rows of 16 lines and an eighth; the last stage one eighth full
])
def test_rows_off_cache_lines(s, B, L):
    """Dense layers whose rows start off the cache lines load a stage in bursts (rows_off_lines in phantom_api.hip).  Each product against 64 bits, from the step's
    own operands: a bf16 output within one rounding (2^-8 of the value and of the sum's rms for what cancels), gradients in float within 1e-6 (2-norm)."""
    print(f"case rows off lines s={s} B={B} L={L}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    rand = lambda *shape, by=1.0: (torch.randn(shape, device="cuda", generator=gen) * by).bfloat16()
    X, T = rand(B, s), rand(B, s)
    Lw, bias = [rand(s, s, by=s ** -0.5) for _ in range(L)], [rand(s, by=0.1) for _ in range(L)]
    dLw, dbias = [torch.full((s, s), float("nan"), device="cuda") for _ in range(L)], [torch.empty(s, device="cuda") for _ in range(L)]
    Y, delta = [torch.empty_like(X) for _ in range(L)], [torch.empty_like(X) for _ in range(L)]
    prob = ph.make_problem(s, 1, 0, B, L, "relu", "bf16", 0)
    ph.ffn_step(prob, X, T, Lw, None, None, bias, dLw=dLw, dbias=dbias, loss=torch.zeros(4, device="cuda"), mode="no_update",
                workspace=workspace(ph.workspace_bytes(prob)), taps={"Y": Y, "delta": delta})
    for l in range(L):
        x = (X if l == 0 else Y[l - 1]).double()
        want = (x @ Lw[l].double().t().contiguous() + bias[l].double()).clamp(min=0)
        assert ((Y[l].double() - want).abs() <= 2 ** -8 * (want.abs() + 1e-3)).all()
        want = delta[l].double().t().contiguous() @ x
        assert float((dLw[l].double() - want).norm() / want.norm()) <= 1e-6

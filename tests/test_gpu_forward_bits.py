"""A step's output is the same bits whether the step stops there (mode "forward") or goes on to the gradients, although the last layer's update then forms the
output error, too, and goes out without a compression beside it: the kernels that the two take add in the same order."""
import pytest
import torch

import paper_2508_00960_amd as ph

pytestmark = pytest.mark.gpu


def outputs(n, p, k, B, L, act, dtype, rank=0):
    """(Y of a forward step, the last layer's output within a step with gradients)"""
    gen = torch.Generator(device="cuda").manual_seed(3)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    s, q = n // p, p - 1
    lead = (p,) if rank < 0 else ()
    rand = lambda *shape, by=1.0: (torch.randn(shape, device="cuda", generator=gen) * by).to(dt)
    prob = ph.make_problem(n, p, k, B, L, act, dtype, rank)
    X, T = rand(*lead, B, s), rand(*lead, B, s)
    Lw = [rand(*lead, s, s, by=s ** -0.5) for _ in range(L)]
    bias = [rand(*lead, s, by=0.1) for _ in range(L)]
    Cw = [rand(*lead, k, s, by=s ** -0.5) for _ in range(L)] if q else None
    Dw = [rand(*lead, q, s, k, by=k ** -0.5) for _ in range(L)] if q else None
    G = [rand(q, B, k) for _ in range(L)] if q and rank >= 0 else None
    dg = [rand(B, k) for _ in range(L)] if q and rank >= 0 else None
    ws = torch.empty(ph.workspace_bytes(prob), device="cuda", dtype=torch.uint8)
    got = []
    for mode in ("forward", "no_update"):
        Y = [torch.full((*lead, B, s), float("nan"), device="cuda", dtype=dt) for _ in range(L)]
        train = mode != "forward"
        ph.ffn_step(prob, X, T if train else None, Lw, Cw, Dw, bias, G=G, dg_own=dg if train else None, mode=mode, workspace=ws,
                    loss=torch.zeros(4, device="cuda") if train else None, taps={"Y": Y})
        got.append(Y[-1])
    return got


BF16 = [
    # few rows (csrc/few_rows.h).  In tiles with eight teams: reductions of 960 and more, and of 512
    (8192, 8, 64, 48, 2, "relu"),        # 23 tiles of 64: the last two wavefronts have one less
    (8192, 8, 64, 96, 2, "gelu"),        # 2 blocks of rows
    (8192, 8, 64, 128, 2, "relu"),       # 4 blocks
    (8192, 8, 8, 40, 1, "relu"),         # 1080: the last tile is seven eighths full and has a wavefront of its own
    (512, 1, 0, 100, 3, "gelu"),         # dense, 512
    (1024, 1, 0, 17, 2, "identity"),
    (2560, 2, 200, 33, 2, "relu"),       # 1480: half a chunk left over
    # ... with two teams: shorter ones
    (2048, 8, 16, 48, 2, "relu"),        # 368: six tiles
    (2048, 8, 48, 384, 2, "gelu"),       # 592: ten tiles, the last of them a quarter; 2 blocks
    (2048, 8, 48, 768, 2, "relu"),       # 4 blocks
    (1600, 2, 144, 20, 2, "gelu"),       # 944: the longest
    (16, 2, 8, 5, 2, "relu"),            # one tile, a quarter full: the second team has none
    (320, 4, 24, 19, 3, "identity"),     # 152: two and a half
    (576, 8, 24, 260, 2, "relu"),        # 240: an odd number of chunks
]
F32 = [
    # without the compression the launch is one of few tiles (gemm_flex_f32_few_kernel), with it it is not
    (192, 2, 32, 4480, 1, "relu", 0),    # one group of 16 terms to a team: 420 and 560 workgroups, at most 512
    (384, 2, 64, 2560, 1, "gelu", 1),    # two groups: 480 and 640
    (896, 2, 64, 544, 1, "relu", 0),     # four groups: 238 and 272, at most 256
    (640, 2, 64, 360, 1, "identity", -1),    # ... all ranks, in two launches: 240
]


@pytest.mark.parametrize("n,p,k,B,L,act", BF16)
def test_bf16(n, p, k, B, L, act):
    print(f"case forward bits bf16 n={n} p={p} k={k} B={B} L={L} {act}", flush=True)
    assert torch.equal(*outputs(n, p, k, B, L, act, "bf16"))


@pytest.mark.parametrize("n,p,k,B,L,act,rank", F32)
def test_f32(n, p, k, B, L, act, rank):
    print(f"case forward bits f32 n={n} p={p} k={k} B={B} L={L} {act} rank={rank}", flush=True)
    assert torch.equal(*outputs(n, p, k, B, L, act, "f32", rank))

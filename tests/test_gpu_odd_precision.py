"""bf16 problems with an odd width or phantom width: precision of what is computed in 32 bits, against 64 bits."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import workspace
from stage_check import check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,bound", [
    # 2-norm errors of the float gradients.  One running sum over the batch: 1.3e-7 at 1030 terms, 1.7e-6 at 65536.  Levels of 64
    # and 256 terms: roundings of 4 to 16 terms' sums, 4, and B / 256, i.e. some 0.25 ulp * sqrt(B / 256 + 20) of 6e-8
    (402, 2, 13, 1030, 1e-7),
    (2002, 2, 5, 4096, 1.5e-7),
    (402, 2, 13, 65536, 4e-7),
])
@pytest.mark.parametrize("mean", [0.0, 1.0])
def test_weight_gradients_of_long_batches(n, p, k, B, bound, mean):
    print(f"case odd gradients n={n} p={p} k={k} B={B} mean={mean}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(1)
    s, q = n // p, p - 1

    def normal(*shape, scale=1.0, mean=0.0):
        return (torch.randn(shape, device="cuda", generator=gen) * scale + mean).bfloat16()

    X, dY, G, dg = normal(B, s, mean=mean), normal(B, s, scale=1 / B, mean=mean / B), normal(q, B, k, mean=mean), normal(B, k, scale=1 / B)
    Lw, Cw, Dw = normal(s, s, scale=s ** -0.5), normal(k, s, scale=s ** -0.5), normal(q, s, k, scale=k ** -0.5)
    dLw, dCw, dDw, dbias = (torch.empty(shape, device="cuda") for shape in ((s, s), (k, s), (q, s, k), (s,)))
    pc = ph.make_problem(n, p, k, B, 1, "identity", "bf16", 0)
    ph.layer_bwd(pc, dY, X, None, Lw, Cw, Dw, G, dg, torch.empty_like(X), dLw, dCw, dDw, dbias, torch.empty_like(G),
                 workspace(ph.workspace_bytes(pc)))
    torch.cuda.synchronize()
    d, X64 = dY.double(), X.double()
    for name, got, want in (("dLw", dLw, d.t().contiguous() @ X64), ("dCw", dCw, dg.double().t().contiguous() @ X64),
                            ("dDw", dDw[0], d.t().contiguous() @ G[0].double()), ("dbias", dbias, d.sum(0))):
        err = float((got.double() - want).norm() / want.norm())
        print(f"{name} {err:.2e}", flush=True)
        assert err <= bound, f"{name}: {err:.2e} > {bound:.1e}"


def test_bias_gradient_of_a_very_long_batch():
    """2^21 rows: one running sum per thread adds 32768 partial sums of 16 rows, in three levels 16, 64 and 512."""
    print("case odd bias gradient", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(2)
    n, p, k, B = 66, 2, 1, 1 << 21
    s = n // p
    X, G, dg = (torch.zeros(shape, device="cuda", dtype=torch.bfloat16) for shape in ((B, s), (1, B, k), (B, k)))
    dY = (torch.rand((B, s), device="cuda", generator=gen) / B).bfloat16()
    Lw, Cw, Dw = (torch.zeros(shape, device="cuda", dtype=torch.bfloat16) for shape in ((s, s), (k, s), (1, s, k)))
    dLw, dCw, dDw, dbias = (torch.empty(shape, device="cuda") for shape in ((s, s), (k, s), (1, s, k), (s,)))
    pc = ph.make_problem(n, p, k, B, 1, "identity", "bf16", 0)
    ph.layer_bwd(pc, dY, X, None, Lw, Cw, Dw, G, dg, None, dLw, dCw, dDw, dbias, torch.empty_like(G), workspace(ph.workspace_bytes(pc)))
    torch.cuda.synchronize()
    want = dY.double().sum(0)
    err = float((dbias.double() - want).norm() / want.norm())
    print(f"dbias {err:.2e}", flush=True)
    # positive terms: a rounding at a level of m sums is at most half an ulp of the running sum, in rms 0.29 ulp of half of it;
    # 16, 64 and 512 of them (two teams or one): 0.17 * 6e-8 * sqrt(592) = 2.5e-7, 32768: 1.8e-6
    assert err <= 6e-7, err


@pytest.mark.parametrize("n,p,k,B,L,act,rank,widths,ks", [
    (66, 2, 3, 1100, 2, "gelu", 0, None, None),                 # weight gradients alone in a launch: 32 x 32 tiles, eight teams
    (2202, 2, 3, 5, 2, "gelu", 1, None, None),                  # forward in such tiles, 1104 terms
    (1002, 2, 9, 700, 3, "relu", -1, None, None),               # two teams, 700 terms
    (256, 2, 8, 300, 3, "gelu", 0, (256, 260, 258, 256), (8, 8, 8)),       # one odd shard (129) among even ones
])
def test_step_every_stage(n, p, k, B, L, act, rank, widths, ks):
    print(f"case odd stages n={n} p={p} k={k} B={B} L={L} {act} rank={rank} widths={widths}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="bf16", rank=rank, widths=widths, ks=ks), seed=9, lr=0.02)


@pytest.mark.parametrize("p", [1, 2])
def test_gelu_derivative_of_an_odd_width(p):
    """A training step keeps sigma' of its first layer in float, right behind y_0 at the start of the workspace (256-byte
    steps).  With one neuron per rank and a weight of 1 it is sigma' of the network's input, free of any other rounding."""
    print(f"case odd gelu p={p}", flush=True)
    B = 1 << 16
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = ((torch.rand((B, 1), device="cuda", generator=gen) * 2 - 1) * 3).bfloat16()
    zeros = lambda *shape: torch.zeros(shape, device="cuda", dtype=torch.bfloat16)
    kk = 1 if p > 1 else 0
    one = torch.ones((1, 1), device="cuda", dtype=torch.bfloat16)
    prob = ph.make_problem(p, p, kk, B, 2, "gelu", "bf16", 0)
    ws = workspace(ph.workspace_bytes(prob))
    peers = lambda *shape: [zeros(*shape), zeros(*shape)] if p > 1 else None
    loss = torch.zeros(4, device="cuda")
    ph.ffn_step(prob, a, zeros(B, 1), [one, one], peers(kk, 1), peers(p - 1, 1, kk), [zeros(1), zeros(1)], G=peers(p - 1, B, kk),
                dg_own=peers(B, kk), loss=loss, mode="no_update", workspace=ws)
    torch.cuda.synchronize()
    at = -(-B * 2 // 256) * 256
    got = ws[at:at + 4 * B].view(torch.float32).double()
    x = a.double().flatten()
    want = 0.5 * torch.special.erfc(-x / 2 ** 0.5) + x * torch.exp(-x * x / 2) / (2 * torch.pi) ** 0.5
    rms = float((got - want).pow(2).mean().sqrt())
    print(f"sigma' rms {rms:.2e} max {float((got - want).abs().max()):.2e}", flush=True)
    # erff and the sum of its two parts: an ulp or two of numbers below 1, rms 3e-8; the five-term formula adds 6e-8 of its own
    assert rms <= 4.5e-8

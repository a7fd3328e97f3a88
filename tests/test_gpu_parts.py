"""fp32 products in three bf16 parts (widths that 4 divides, reductions of up to 2048 terms): against the oracle at the edges of tiles and steps,
against 64 bits in precision, and where infinities, NaN and overflow send a tile back to the fp32 instructions."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin

from helpers import workspace
from stage_check import check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,k,B,L,act,rank,mode", [
    (528, 4, 12, 130, 2, "relu", -1, "train"),       # shard 132: 64 x 64 tiles, the last of 4 columns; 5 steps and part of one
    (528, 4, 4, 67, 3, "gelu", -1, "no_update"),     # segments of one vector; a batch that 4 does not divide
    (520, 2, 132, 333, 2, "gelu", 1, "train"),       # one rank; segments longer than a step
    (508, 1, 0, 2048, 2, "relu", 0, "train"),        # dense; the longest reduction
    (508, 1, 0, 2049, 2, "relu", 0, "train"),        # ... and past it, the fp32 instructions
    (4064, 8, 12, 1020, 2, "gelu", -1, "train"),     # shard 508: 128 x 128 tiles in every layout
    (2056, 2, 12, 3000, 1, "relu", 0, "forward"),    # shard 1028, one rank: 240 of 128 x 128
    (1000, 4, 10, 300, 2, "relu", -1, "train"),      # 4 does not divide the phantom width: the fp32 instructions
])
def test_parity(n, p, k, B, L, act, rank, mode):
    print(f"case parts n={n} p={p} k={k} B={B} L={L} {act} rank={rank} {mode}", flush=True)
    check_stages(pin.Problem(n=n, p=p, k=k, batch=B, layers=L, act=act, dtype="f32", rank=rank), seed=11, lr=0.02, mode=mode)


def _layer(s, p, k, B, seed, scale=1.0):
    """One rank's layer, identity: inputs, and its results with their values in 64 bits."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = p - 1
    normal = lambda *shape, by=1.0: torch.randn(shape, device="cuda", generator=gen) * by
    t = {"X": normal(B, s, by=scale), "G": normal(q, B, k, by=scale), "dY": normal(B, s, by=scale / B), "dg": normal(B, k, by=scale / B),
         "Lw": normal(s, s, by=s ** -0.5), "Cw": normal(k, s, by=s ** -0.5), "Dw": normal(q, s, k, by=k ** -0.5), "bias": normal(s, by=scale)}
    return t


def _run(t):
    (B, s), (q, _, k) = t["X"].shape, t["G"].shape
    pc = ph.make_problem(s * (q + 1), q + 1, k, B, 1, "identity", "f32", 0)
    ws = workspace(ph.workspace_bytes(pc))
    new = lambda *shape: torch.full(shape, 7.0, device="cuda")
    o = {"Y": new(B, s), "g": new(B, k), "dX": new(B, s), "dL": new(s, s), "dC": new(k, s), "dD": new(q, s, k), "db": new(s), "dG": new(q, B, k)}
    ph.layer_fwd(pc, t["X"], t["Lw"], t["Cw"], t["Dw"], t["bias"], t["G"], o["Y"], o["g"], None, ws)
    ph.layer_bwd(pc, t["dY"], t["X"], o["Y"], t["Lw"], t["Cw"], t["Dw"], t["G"], t["dg"], o["dX"], o["dL"], o["dC"], o["dD"], o["db"], o["dG"], ws)
    torch.cuda.synchronize()
    d = {name: v.double() for name, v in t.items()}
    want = {"Y": d["X"] @ d["Lw"].T + d["bias"], "g": d["X"] @ d["Cw"].T, "dX": d["dY"] @ d["Lw"] + d["dg"] @ d["Cw"], "dL": d["dY"].T @ d["X"],
            "dC": d["dg"].T @ d["X"], "db": d["dY"].sum(0), "dD": torch.stack([d["dY"].T @ d["G"][i] for i in range(q)]),
            "dG": torch.stack([d["dY"] @ d["Dw"][i] for i in range(q)])}
    for i in range(q):
        want["Y"] = want["Y"] + d["G"][i] @ d["Dw"][i].T
    return o, want


@pytest.mark.parametrize("s,p,k,B,scale", [(132, 4, 12, 200, 1.0), (512, 8, 32, 1024, 1.0), (1024, 4, 64, 2000, 1.0), (512, 2, 64, 700, 1e-17),
                                           (512, 2, 64, 700, 1e17)])
def test_precision(s, p, k, B, scale):
    """2-norm errors.  On the fp32 instructions 0.9e-7 to 1.2e-7 (a sum of 16 terms has 16 roundings of 2^-24 of its size or less, those of 256 and
    of all terms as many); in parts a sixteenth of the first, of 128 terms 8, of all terms up to 16: at most what they were."""
    print(f"case precision s={s} p={p} k={k} B={B} scale={scale}", flush=True)
    got, want = _run(_layer(s, p, k, B, seed=3, scale=scale))
    for name in want:
        err = float((got[name].double() - want[name]).norm() / want[name].norm())
        print(f"{name} {err:.2e}", flush=True)
        assert err <= 1.2e-7, f"{name}: {err:.2e}"


@pytest.mark.parametrize("s,p,k,B", [(132, 4, 12, 200), (1028, 2, 12, 3000)])
def test_infinities_and_overflow(s, p, k, B):
    """Results that are not finite are those of the sums in 64 bits, and so are their finite neighbours in the same tile."""
    print(f"case infinities s={s} p={p} k={k} B={B}", flush=True)
    t = _layer(s, p, k, B, seed=4)
    inf, big = float("inf"), 3.4e38                    # (big: rounded to bf16 it would be an infinity)
    t["X"][3, 5], t["X"][70, 40], t["X"][71, s - 1], t["X"][B - 1, 0] = inf, float("nan"), big, -inf
    t["Lw"][2, 5], t["Lw"][3, 40] = 1.0, 0.0           # a weight whose smaller parts are zero; 0 * NaN
    t["Lw"][:, s - 1] *= 0.1
    t["Cw"][:, s - 1] *= 0.1
    t["X"][100, 7], t["Lw"][9, 7] = 3e38, 4.0          # a product that overflows
    t["dY"][5, 1], t["G"][0, 9, 2] = -inf, inf
    got, want = _run(t)
    for name in want:
        w = want[name].float()                         # (what is beyond the largest float becomes an infinity)
        g = got[name]
        assert torch.equal(torch.isnan(g), torch.isnan(w)), f"{name}: NaN"
        assert torch.equal(torch.isinf(g), torch.isinf(w)) and torch.equal(g[torch.isinf(g)], w[torch.isinf(w)]), f"{name}: infinities"
        fine = torch.isfinite(w) & (w.abs() < 1e30)
        rms = float(want[name][fine].pow(2).mean().sqrt())
        assert float((g.double() - want[name])[fine].abs().max()) <= 1e-5 * rms, f"{name}: finite values"

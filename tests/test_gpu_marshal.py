"""The native marshalling (csrc/marshal.cpp) against the Python path that it stands in for: it takes the ordinary calls, with
the same results, and leaves the others to the Python path, which raises."""
import pytest
import torch

import paper_2508_00960_amd as ph
import phantom_inputs as pin
from paper_2508_00960_amd import binding

from helpers import empty, empty_f32, to_gpu, to_gpu_f32, workspace

pytestmark = pytest.mark.gpu

NAMES = ("Lw", "Cw", "Dw", "bias")


class Calls:
    """The arguments of the three calls for one small problem, as a user's program holds them."""

    def __init__(self, dtype, rank):
        prob = pin.Problem(n=512, p=4, k=8, batch=40, layers=2, act="gelu", dtype=dtype, rank=rank)
        one = rank >= 0
        data = pin.one_rank_step_inputs(prob, 1) if one else pin.all_rank_step_inputs(prob, 1)
        self.prob = ph.make_problem(512, 4, 8, 40, 2, "gelu", dtype, rank)
        self.ws = workspace(ph.workspace_bytes(self.prob))
        self.W = {nm: [to_gpu(P[nm], dtype) for P in data["layers"]] for nm in NAMES}
        self.M = {nm: [to_gpu_f32(P[nm]) for P in data["layers"]] if dtype == "bf16" else None for nm in NAMES}
        self.D = {nm: [empty_f32(P[nm].shape) for P in data["layers"]] for nm in NAMES}
        self.G = [to_gpu(P["G"], dtype) for P in data["layers"]] if one else None
        self.dg = [to_gpu(P["dg_own"], dtype) for P in data["layers"]] if one else None
        self.X, self.T = to_gpu(data["X0"], dtype), to_gpu(data["T"], dtype)
        lead = () if one else (4,)
        self.Y, self.A, self.dX = (empty(lead + (40, 128), dtype) for _ in range(3))
        self.g_own, self.dg_own = (empty(lead + (40, 8), dtype) for _ in range(2))
        self.dG_send = empty(lead + (3, 40, 8), dtype)
        self.loss = empty_f32((4,))

    def fwd(self, **change):
        a = dict(X=self.X, Lw=self.W["Lw"][0], Cw=self.W["Cw"][0], Dw=self.W["Dw"][0], bias=self.W["bias"][0],
                 G=self.G[0] if self.G else None, Y=self.Y, g_own=self.g_own, A_save=self.A, workspace=self.ws, stream=None)
        a.update(change)
        return ("layer_fwd", (self.prob, *a.values()))

    def bwd(self, **change):
        a = dict(dY=self.T, X=self.X, A_or_Y=self.A, Lw=self.W["Lw"][0], Cw=self.W["Cw"][0], Dw=self.W["Dw"][0],
                 G=self.G[0] if self.G else self.g_own, dg_own=self.dg[0] if self.dg else self.dg_own, dX=self.dX, dLw=self.D["Lw"][0],
                 dCw=self.D["Cw"][0], dDw=self.D["Dw"][0], dbias=self.D["bias"][0], dG_send=self.dG_send, workspace=self.ws, stream=None)
        a.update(change)
        return ("layer_bwd", (self.prob, *a.values()))

    def step(self, mode="train", **change):
        a = dict(Lw_master=self.M["Lw"], Cw_master=self.M["Cw"], Dw_master=self.M["Dw"], bias_master=self.M["bias"], G=self.G,
                 dg_own=self.dg, dLw=self.D["Lw"], dCw=self.D["Cw"], dDw=self.D["Dw"], dbias=self.D["bias"], Y_out=self.Y,
                 loss=self.loss, lr=0.1, mode=mode, workspace=self.ws)
        a.update(change)
        return lambda: ph.ffn_step(self.prob, self.X, self.T, *(self.W[nm] for nm in NAMES), **a)

    def results(self):
        torch.cuda.synchronize()
        t = [self.Y, self.A, self.g_own, self.dX, self.dG_send, self.loss[:1]]
        for kind in (self.W, self.M, self.D):
            for per_layer in kind.values():
                t += per_layer or []
        return [x.clone() for x in t]


def through(route, call):
    """Runs the call by the native route alone ("native": it has to take it) or by the Python path alone."""
    name, args = call
    if route == "native":
        assert binding._fast.layer_fwd is not binding._PythonOnly.layer_fwd, "the native module is missing"
        assert getattr(binding._fast, name)(*args) == 0
    else:
        getattr(ph, name)(*args)


@pytest.mark.parametrize("dtype,rank", [("f32", 0), ("bf16", 2), ("f32", -1)])
def test_both_routes_give_the_same_bits(dtype, rank, monkeypatch):
    print(f"case marshal {dtype} rank={rank}", flush=True)
    ph.load()
    out = []
    for route in ("native", "python"):
        c = Calls(dtype, rank)
        if route == "python":
            monkeypatch.setattr(binding, "_fast", binding._PythonOnly)
        with torch.cuda.stream(torch.cuda.Stream()):
            through(route, c.fwd())
            through(route, c.bwd())
            torch.cuda.synchronize()
        through(route, c.fwd(stream=torch.cuda.current_stream().cuda_stream))
        c.step("no_update")()
        c.step("train")()
        c.step("train", static=True, workspace=None)()
        c.step("forward", loss=None)()
        out.append(c.results())
    for i, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a, b), i


def test_what_the_native_route_leaves_alone_raises():
    c = Calls("bf16", 0)
    ph.load()
    for change, error, text in [
        (dict(X=c.X[:20]), ValueError, "X: 2560 elements"),
        (dict(X=c.X.float()), ValueError, "X: elements of 4 bytes"),
        (dict(X=c.X.cpu()), ValueError, "X: tensor is on cpu"),
        (dict(X=c.X.t()), ValueError, "X: tensor is not contiguous"),
        (dict(G=c.G[0].cpu()), ValueError, "G: tensor is on cpu"),
        (dict(A_save=c.A[:, :64]), ValueError, "A_save: tensor is not contiguous"),
        (dict(X=torch.sparse_coo_tensor(torch.zeros(2, 1, dtype=torch.long), torch.ones(1, dtype=torch.bfloat16), (40, 128)).cuda()),
         ValueError, "X: tensor is not contiguous"),
    ]:
        name, args = c.fwd(**change)
        assert getattr(binding._fast, name)(*args) is None, change.keys()
        with pytest.raises(error, match=text):
            getattr(ph, name)(*args)
    # taken by the Python path: a raw address, a workspace as address and length, a stream object
    for change in (dict(X=c.X.data_ptr()), dict(workspace=(c.ws.data_ptr(), c.ws.numel())), dict(stream=torch.cuda.current_stream())):
        name, args = c.fwd(**change)
        assert getattr(binding._fast, name)(*args) is None
        getattr(ph, name)(*args)
    with pytest.raises(ValueError, match="expected 2 per-layer tensors"):
        ph.ffn_step(c.prob, c.X, c.T, c.W["Lw"][:1], c.W["Cw"], c.W["Dw"], c.W["bias"], G=c.G, mode="forward", workspace=c.ws)
    # an argument error of the library, found by the native route itself
    name, args = c.fwd(Y=None)
    assert getattr(binding._fast, name)(*args) == -1
    with pytest.raises(ph.PhantomError, match="Y is NULL"):
        getattr(ph, name)(*args)
    torch.cuda.synchronize()

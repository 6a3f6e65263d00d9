"""GPU: products whose row counts the host knows (shared experts, the router), which may be summed in parts along K.

Each shape runs with the workspace that the query asks for and with the least that the call accepts (no room for parts);
both against products in fp64.  Sizes: one row, remainders of every tile height, K that ends inside a step or a
part.  Tolerances as in test_gpu_tiles.py, fp32 sums of K <= 2 * 3 * 1368 terms: sqrt(K) * 2^-24 = 5.4e-6 a product at
worst, 1e-5 over two.
"""
import re

import pytest
import torch

from .helpers import small_tiles

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 5e-3}
TALL = [(1, 560, 6144, 128), (2, 3400, 1024, 192), (3, 1200, 3000, 200)]   # bf16: the tall tiles, without and with a K tail (those of SHARED take the small ones)
SHARED = [(1, 1, 512, 1024), (3, 16, 320, 1368), (4, 33, 1000, 712), (2, 200, 136, 2048), (1, 700, 264, 520), (1, 3001, 136, 200)]
ROUTER = [(1, 512, 5), (130, 2000, 60), (700, 1024, 128), (2500, 328, 64)]


def rel(got, ref):
    return float((got.double().cpu() - ref).norm() / ref.norm())


def least(call, moe):
    """The workspace that a call needs, from its refusal of 16 bytes."""
    with pytest.raises(moe.MoEError, match="need") as e:
        call(torch.empty(16, dtype=torch.uint8, device="cuda"))
    return int(re.search(r"need (\d+)", str(e.value)).group(1))


def workspaces(call, query, moe):
    n = least(call, moe)
    assert n <= query
    for size in sorted({n, query}):
        ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")  # NaNs
        call(ws)
        torch.cuda.synchronize()
        yield size


@pytest.mark.parametrize("ffn", ["swiglu", "gelu"])
@pytest.mark.parametrize("dtype,S,T,d,F", [(t, *s) for t in ("f32", "bf16") for s in SHARED] + [("bf16", *s) for s in TALL])
def test_shared_calls(dtype, S, T, d, F, ffn):
    import paper_2502_02581_amd as moe

    assert dtype == "f32" or small_tiles(S, T, d, F) == ((S, T, d, F) in SHARED)
    shape = moe.MoEShape(T, d, max(S, 2), 1, F, dtype)
    dt, gated = shape.torch_dtype, ffn == "swiglu"
    g = torch.Generator().manual_seed(d * 1000 + F)
    rnd = lambda std, *s: (torch.randn(*s, generator=g) * std).to(dt)
    X, dY = rnd(1.0, T, d), rnd(1.0, T, d)
    Wg, Wd = rnd(d ** -0.5, S, d, F), rnd(F ** -0.5, S, F, d)
    Wu = rnd(d ** -0.5, S, d, F) if gated else None
    x = X.double().requires_grad_(True)
    w64 = [None if t is None else t.double().requires_grad_(True) for t in (Wg, Wu, Wd)]
    z = torch.stack([x @ w64[0][s] for s in range(S)])
    if gated:
        h = torch.nn.functional.silu(z) * torch.stack([x @ w64[1][s] for s in range(S)])
    else:
        h = torch.nn.functional.gelu(z)
    y = sum(h[s] @ w64[2][s] for s in range(S))
    y.backward(dY.double())
    dev = "cuda"
    gpu = lambda t: None if t is None else t.to(dev)
    Xd, dYd, w = gpu(X), gpu(dY), [gpu(t) for t in (Wg, Wu, Wd)]
    new = lambda *s: torch.full(s, float("nan"), dtype=dt, device=dev)
    G, U, H, Y, dX = new(S, T, F), new(S, T, F), new(S, T, F), new(T, d), new(T, d)
    dWg, dWu, dWd = new(S, d, F), new(S, d, F), new(S, F, d)
    ids = torch.full((S,), -7, dtype=torch.int32, device=dev)
    n_act = torch.full((1,), -7, dtype=torch.int32, device=dev)

    def fwd(ws):
        moe.moe_expert_fwd(shape, S, None, T, Xd, *w, G, U, H, Y, ws)

    def bwd(ws):
        moe.moe_expert_bwd(shape, S, None, T, Xd, *w, G, U, H, dYd, dX, ids, n_act, dWg, dWu, dWd, ws)

    def check(pairs):
        worst = {k: rel(got, ref.detach()) for k, (got, ref) in pairs.items()}
        print(dtype, S, T, d, F, ffn, {k: f"{v:.1e}" for k, v in worst.items()})
        assert all(v <= TOL[dtype] for v in worst.values()), worst

    for _ in workspaces(fwd, moe.moe_expert_fwd_workspace_bytes(shape, S, T, True), moe):
        check({"G": (G, z), "H": (H, h), "Y": (Y, y)})
    for _ in workspaces(bwd, moe.moe_expert_bwd_workspace_bytes(shape, S, T, True), moe):
        assert ids.tolist() == list(range(S)) and int(n_act) == S
        pairs = {"dX": (dX, x.grad), "dWg": (dWg, w64[0].grad), "dWd": (dWd, w64[2].grad)}
        if gated:
            pairs["dWu"] = (dWu, w64[1].grad)
        check(pairs)
        for t in (dX, dWg, dWu, dWd):
            t.fill_(float("nan"))
        ids.fill_(-7)


@pytest.mark.parametrize("dtype,S,T,d,F", [("f32", 4, 33, 1024, 712), ("bf16", 4, 33, 1024, 712), ("bf16", 1, 560, 6144, 128)])
def test_same_bits_with_any_larger_workspace(dtype, S, T, d, F):
    """Where a call has what the query answers, how much more there is changes nothing (all four calls use parts here)."""
    import paper_2502_02581_amd as moe

    E = 128
    assert dtype == "f32" or small_tiles(S, T, d, F) == (T == 33)
    shape, rshape = moe.MoEShape(T, d, S, 1, F, dtype), moe.MoEShape(700, d, E, 1, F, dtype)
    dt, dev = shape.torch_dtype, "cuda"
    g = torch.Generator().manual_seed(3)
    rnd = lambda *s: (torch.randn(*s, generator=g) * d ** -0.5).to(dt).to(dev)
    X, dY, w = rnd(T, d), rnd(T, d), [rnd(S, d, F), rnd(S, d, F), rnd(S, F, d)]
    Xr, Wr, dl = rnd(700, d), rnd(d, E), torch.randn(700, E, generator=g).to(dev)
    new = lambda *s, t=dt: torch.full(s, float("nan"), dtype=t, device=dev)
    i32 = lambda n: torch.empty(n, dtype=torch.int32, device=dev)
    fwd, bwd = [new(S, T, F) for _ in range(3)] + [new(T, d)], [new(T, d), new(S, d, F), new(S, d, F), new(S, F, d)]
    logits, dWr, dXr = new(700, E, t=torch.float32), new(d, E), new(700, d)
    calls = [(moe.moe_expert_fwd_workspace_bytes(shape, S, T, True), fwd,
              lambda ws: moe.moe_expert_fwd(shape, S, None, T, X, *w, *fwd, ws)),
             (moe.moe_expert_bwd_workspace_bytes(shape, S, T, True), bwd,
              lambda ws: moe.moe_expert_bwd(shape, S, None, T, X, *w, *fwd[:3], dY, bwd[0], i32(S), i32(1), *bwd[1:], ws)),
             (moe.moe_router_fwd_workspace_bytes(rshape), [logits], lambda ws: moe.moe_router_fwd(rshape, Xr, Wr, logits, ws)),
             (moe.moe_router_bwd_workspace_bytes(rshape), [dWr, dXr],
              lambda ws: moe.moe_router_bwd(rshape, Xr, Wr, dl, dWr, dXr, False, ws))]
    for query, outs, call in calls:
        assert least(call, moe) < query
        call(torch.empty(query, dtype=torch.uint8, device=dev))
        first = [t.clone() for t in outs]
        for more in (16, 4096, 3 * query):
            for t in outs:
                t.fill_(float("nan"))
            call(torch.empty(query + more, dtype=torch.uint8, device=dev))
            assert all(torch.equal(a, b) for a, b in zip(first, outs))


def test_shared_backward_without_rows():
    """No token: no group is active, and nothing else is written."""
    import paper_2502_02581_amd as moe

    S, d, F = 3, 64, 128
    shape = moe.MoEShape(0, d, 4, 1, F, "bf16")
    new = lambda *s: torch.full(s, 3.0, dtype=torch.bfloat16, device="cuda")
    ids = torch.full((S,), -7, dtype=torch.int32, device="cuda")
    n_act = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    w, dw = [new(S, d, F), new(S, d, F), new(S, F, d)], [new(S, d, F), new(S, d, F), new(S, F, d)]
    e, f = new(0, d), new(S, 0, F)
    ws = torch.empty(moe.moe_expert_bwd_workspace_bytes(shape, S, 0, True), dtype=torch.uint8, device="cuda")
    moe.moe_expert_bwd(shape, S, None, 0, e, *w, f, f, f, e, e, ids, n_act, *dw, ws)
    torch.cuda.synchronize()
    assert ids.tolist() == [-1] * S and int(n_act) == 0 and all(bool((t == 3.0).all()) for t in dw)


@pytest.mark.parametrize("T,d,E", ROUTER)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_router_calls(dtype, T, d, E):
    import paper_2502_02581_amd as moe

    shape = moe.MoEShape(T, d, E, 1, 64, dtype)
    dt, dev = shape.torch_dtype, "cuda"
    g = torch.Generator().manual_seed(T + d)
    X, Wr = torch.randn(T, d, generator=g).to(dt), (torch.randn(d, E, generator=g) * d ** -0.5).to(dt)
    dl, dX0 = torch.randn(T, E, generator=g), torch.randn(T, d, generator=g).to(dt)
    Xd, Wd, dld = X.to(dev), Wr.to(dev), dl.to(dev)
    logits = torch.full((T, E), float("nan"), device=dev)
    dl_in = dl.to(dt).double()
    for _ in workspaces(lambda ws: moe.moe_router_fwd(shape, Xd, Wd, logits, ws), moe.moe_router_fwd_workspace_bytes(shape), moe):
        assert rel(logits, X.double() @ Wr.double()) <= TOL["f32"]
    for acc in (False, True):
        dWr, dX = torch.full((d, E), float("nan"), dtype=dt, device=dev), torch.empty(T, d, dtype=dt, device=dev)

        def bwd(ws):
            dX.copy_(dX0)
            moe.moe_router_bwd(shape, Xd, Wd, dld, dWr, dX, acc, ws)

        for _ in workspaces(bwd, moe.moe_router_bwd_workspace_bytes(shape), moe):
            assert rel(dWr, X.double().T @ dl_in) <= TOL[dtype]
            assert rel(dX, dl_in @ Wr.double().T + (dX0.double() if acc else 0.0)) <= TOL[dtype]
            dWr.fill_(float("nan"))

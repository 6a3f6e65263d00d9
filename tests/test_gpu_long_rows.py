"""GPU: hidden sizes and widths whose tiles span 4 GiB and more, beyond the 32-bit offsets of the tile cores.

Few rows, so that memory stays small: the tile cores went wrong there through the rows of a tile beyond its valid ones.
References in fp64.  fp32 sums of up to 8.5 million terms, 64 lanes each: sqrt(d / 64) * 2^-24 = 2.2e-5 a product at worst,
6e-5 over the chain; bf16 as in test_gpu_tiles.py.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = {"f32": 6e-5, "bf16": 5e-3}


def rel(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


def inputs(shape, G, T, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    d, F = shape.d, shape.d_ff
    rnd = lambda std, *s: (torch.randn(*s, generator=g, device=DEV) * std).to(shape.torch_dtype)
    return rnd(1.0, T, d), rnd(1.0, T, d), rnd(d ** -0.5, G, d, F), rnd(d ** -0.5, G, d, F), rnd(F ** -0.5, G, F, d)


def new(shape, *s):
    return torch.full(s, float("nan"), dtype=shape.torch_dtype, device=DEV)


# the least sizes of each type, one whose offsets wrap into the valid rows of every kind of tile, a long width
SIZES = [("f32", 4194304, 16), ("f32", 8500000, 8), ("bf16", 8388616, 16), ("bf16", 16778240, 8), ("bf16", 64, 8388672)]


@pytest.mark.parametrize("gather", [False, True])
@pytest.mark.parametrize("dtype,d,F", SIZES)
def test_grouped(dtype, d, F, gather):
    import paper_2502_02581_amd as moe

    T, E = 5, 3
    shape = moe.MoEShape(T, d, E, 1, F, dtype)
    X, dY, Wg, Wu, Wd = inputs(shape, E, T, F)
    off = torch.tensor([0, 3, 3, 5], dtype=torch.int32, device=DEV)
    src = torch.tensor([1, 4, 2, 0, 3], dtype=torch.int32, device=DEV)
    w = torch.tensor([[0.5], [1.0], [2.0], [0.25], [4.0]], device=DEV)   # powers of two: no rounding in dYp
    Xp, dYp = X[src.long()], (dY * w.to(dY.dtype))[src.long()]
    G, U, H = new(shape, T, F), new(shape, T, F), new(shape, T, F)
    Y, dX, dWg, dWu, dWd = new(shape, T, d), new(shape, T, d), new(shape, E, d, F), new(shape, E, d, F), new(shape, E, F, d)
    ids, n_act = torch.empty(E, dtype=torch.int32, device=DEV), torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.full((moe.moe_expert_bwd_workspace_bytes(shape, E, T, False),), 0xff, dtype=torch.uint8, device=DEV)
    if gather:
        moe.moe_expert_fwd_gather(shape, off, src, X, Wg, Wu, Wd, G, U, H, Y, ws)
        moe.moe_expert_bwd_gather(shape, off, src, Xp, Wg, Wu, Wd, G, U, H, dY, w, dYp, dX, ids, n_act, dWg, dWu, dWd, ws)
    else:
        moe.moe_expert_fwd(shape, E, off, T, Xp, Wg, Wu, Wd, G, U, H, Y, ws)
        moe.moe_expert_bwd(shape, E, off, T, Xp, Wg, Wu, Wd, G, U, H, dYp, dX, ids, n_act, dWg, dWu, dWd, ws)
    assert ids.tolist() == [0, 2, -1] and int(n_act) == 2
    for slot, (e, a, b) in enumerate(((0, 0, 3), (2, 3, 5))):
        leaves = [t.double().requires_grad_(True) for t in (Xp[a:b], Wg[e], Wu[e], Wd[e])]
        x, wg, wu, wd = leaves
        y = (torch.nn.functional.silu(x @ wg) * (x @ wu)) @ wd
        y.backward(dYp[a:b].double())
        for name, got, ref in (("Y", Y[a:b], y.detach()), ("dX", dX[a:b], x.grad), ("dWg", dWg[slot], wg.grad), ("dWu", dWu[slot], wu.grad),
                               ("dWd", dWd[slot], wd.grad)):
            assert rel(got, ref) <= TOL[dtype], name
    assert bool(dWd[2].isnan().all())


@pytest.mark.parametrize("dtype,d,F", SIZES)
def test_shared(dtype, d, F):
    import paper_2502_02581_amd as moe

    T, S = 3, 2
    shape = moe.MoEShape(T, d, 2, 1, F, dtype)
    X, dY, Wg, _, Wd = inputs(shape, S, T, F + 1)
    G, H, Y, dX = new(shape, S, T, F), new(shape, S, T, F), new(shape, T, d), new(shape, T, d)
    dWg, dWd = new(shape, S, d, F), new(shape, S, F, d)
    ids, n_act = torch.empty(S, dtype=torch.int32, device=DEV), torch.empty(1, dtype=torch.int32, device=DEV)
    ws = torch.full((max(moe.moe_expert_fwd_workspace_bytes(shape, S, T, True), moe.moe_expert_bwd_workspace_bytes(shape, S, T, True)),), 0xff,
                    dtype=torch.uint8, device=DEV)
    moe.moe_expert_fwd(shape, S, None, T, X, Wg, None, Wd, G, None, H, Y, ws)
    moe.moe_expert_bwd(shape, S, None, T, X, Wg, None, Wd, G, None, H, dY, dX, ids, n_act, dWg, None, dWd, ws)
    assert ids.tolist() == [0, 1] and int(n_act) == S
    x, wg, wd = (t.double().requires_grad_(True) for t in (X, Wg, Wd))
    y = sum(torch.nn.functional.gelu(x @ wg[i]) @ wd[i] for i in range(S))
    y.backward(dY.double())
    for name, got, ref in (("Y", Y, y.detach()), ("dX", dX, x.grad), ("dWg", dWg, wg.grad), ("dWd", dWd, wd.grad)):
        assert rel(got, ref) <= TOL[dtype], name


@pytest.mark.parametrize("dtype,d", [("f32", 8500000), ("bf16", 8388616)])
def test_router(dtype, d):
    import paper_2502_02581_amd as moe

    T, E = 3, 5
    shape = moe.MoEShape(T, d, E, 1, 64, dtype)
    g = torch.Generator(device=DEV).manual_seed(d)
    rnd = lambda std, *s: (torch.randn(*s, generator=g, device=DEV) * std).to(shape.torch_dtype)
    X, Wr, dX = rnd(1.0, T, d), rnd(d ** -0.5, d, E), rnd(1.0, T, d)
    dl, logits, dWr = torch.randn(T, E, generator=g, device=DEV), torch.empty(T, E, device=DEV), new(shape, d, E)
    ws = torch.full((max(moe.moe_router_fwd_workspace_bytes(shape), moe.moe_router_bwd_workspace_bytes(shape)),), 0xff, dtype=torch.uint8, device=DEV)
    ref = dl.to(shape.torch_dtype).double() @ Wr.double().T + dX.double()
    moe.moe_router_fwd(shape, X, Wr, logits, ws)
    moe.moe_router_bwd(shape, X, Wr, dl, dWr, dX, True, ws)
    assert rel(logits, X.double() @ Wr.double()) <= TOL["f32"]
    assert rel(dX, ref) <= TOL[dtype] and rel(dWr, X.double().T @ dl.to(shape.torch_dtype).double()) <= TOL[dtype]


def test_sums_over_more_than_2_gib_of_an_operand():
    """One group's weight gradients step through operands of 2.3 GB: the tile loads' byte counts are 32 bits and start anew
    on the way.  Only the last rows, beyond that point, are not zero."""
    import paper_2502_02581_amd as moe

    R, d, F, last = 140032, 8192, 64, 3000   # rows of 16 KB: 2 GiB are 131072 of them
    shape = moe.MoEShape(R, d, 1, 1, F, "bf16")
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: (torch.randn(*s, generator=g, device="cuda") * s[-1] ** -0.5).bfloat16()
    new = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    X, dY, dX, G, U, H = new(R, d), new(R, d), new(R, d), new(R, F), new(R, F), new(R, F)
    for t in (X, dY, G, U, H):
        t[-last:] = rnd(last, t.shape[1])
    Wg, Wu, Wd, dWg, dWu, dWd = rnd(1, d, F), rnd(1, d, F), rnd(1, F, d), new(1, d, F), new(1, d, F), new(1, F, d)
    off = torch.tensor([0, R], dtype=torch.int32, device="cuda")
    ids, n_act = torch.empty(1, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.moe_expert_bwd_workspace_bytes(shape, 1, R, False), dtype=torch.uint8, device="cuda")
    moe.moe_expert_bwd(shape, 1, off, R, X, Wg, Wu, Wd, G, U, H, dY, dX, ids, n_act, dWg, dWu, dWd, ws)
    x, dy, gg, u, h = (t[-last:].float() for t in (X, dY, G, U, H))
    s = torch.sigmoid(gg)
    dh = dy @ Wd[0].float().T
    dg, du = dh * u * s * (1 + gg * (1 - s)), dh * gg * s
    for got, ref in ((dWd[0], h.T @ dy), (dWg[0], x.T @ dg), (dWu[0], x.T @ du), (dX[-last:], dg @ Wg[0].float().T + du @ Wu[0].float().T)):
        assert float((got.float() - ref).norm() / ref.norm()) <= 1e-2   # operands and results in bf16: a few times 2^-9
    assert not dX[:-last].any()

"""GPU: the expert calls at the edges of their tiles, group by group against products in fp64.

Row counts straddle every tile height and its remainder rule, hidden sizes and widths end inside a K step and
inside a column tile.  Tolerances (2-norm of the error over the 2-norm of the result): a value passes at most five
roundings of relative size 2^-9 in bf16 on its way (operand, activation, its derivative, product, store):
sqrt(5) * 2^-9 / sqrt(3) = 2.5e-3, and twice that for correlated ones; in fp32 the sums of K <= 520 terms contribute
sqrt(K) * 2^-24 each, 1.4e-6, over three products: 5e-6.
"""
import pytest
import torch

from .helpers import small_tiles

pytestmark = pytest.mark.gpu

TOL = {"f32": 5e-6, "bf16": 5e-3}
# rows per group: empty, single, both sides of every tile height, several full tiles with a remainder
ROWS = [1, 0, 15, 17, 33, 64, 65, 95, 97, 0, 128, 129, 161, 192, 193, 255, 257, 449, 600]
DIMS = [(72, 104), (136, 200), (264, 520), (64, 192), (320, 64)]   # bf16: the tiles of short calls
TALL_DIMS = [(1280, 192), (1240, 520), (1288, 200)]                # bf16: the tall tiles, without and with a K tail


def rel(got, ref):
    return float((got.double().cpu() - ref).norm() / ref.norm()) if ref.numel() else 0.0


@pytest.mark.parametrize("ffn", ["swiglu", "gelu"])
@pytest.mark.parametrize("dtype,d,F", [(t, *s) for t in ("f32", "bf16") for s in DIMS] + [("bf16", *s) for s in TALL_DIMS])
def test_expert_tiles(dtype, d, F, ffn):
    import paper_2502_02581_amd as moe

    dev, E, n = "cuda:0", len(ROWS), sum(ROWS)
    assert dtype == "f32" or small_tiles(E, n, d, F) == ((d, F) in DIMS)
    shape = moe.MoEShape(n, d, E, 1, F, dtype)
    dt = shape.torch_dtype
    g = torch.Generator().manual_seed(d * 1000 + F)
    rnd = lambda std, *s: (torch.randn(*s, generator=g) * std).to(dt)
    gated = ffn == "swiglu"
    X, dY = rnd(1.0, n, d), rnd(1.0, n, d)
    Wg, Wd = rnd(d ** -0.5, E, d, F), rnd(F ** -0.5, E, F, d)
    Wu = rnd(d ** -0.5, E, d, F) if gated else None
    off = torch.tensor([0] + ROWS).cumsum(0)
    gpu = lambda t: None if t is None else t.to(dev)
    new = lambda *s: torch.full(s, float("nan"), dtype=dt, device=dev)
    G, U, H, Y, dX = new(n, F), new(n, F), new(n, F), new(n, d), new(n, d)
    dWg, dWu, dWd = new(E, d, F), new(E, d, F), new(E, F, d)
    ids, n_act = torch.empty(E, dtype=torch.int32, device=dev), torch.empty(1, dtype=torch.int32, device=dev)
    ws = torch.empty(max(moe.moe_expert_fwd_workspace_bytes(shape, E, n, False),
                         moe.moe_expert_bwd_workspace_bytes(shape, E, n, False)), dtype=torch.uint8, device=dev)
    ws.fill_(0xff)   # NaNs: nothing may be read before it is written
    offs, Xd, dYd, w = gpu(off.int()), gpu(X), gpu(dY), [gpu(Wg), gpu(Wu), gpu(Wd)]
    moe.moe_expert_fwd(shape, E, offs, n, Xd, *w, G, U, H, Y, ws)
    moe.moe_expert_bwd(shape, E, offs, n, Xd, *w, G, U, H, dYd, dX, ids, n_act, dWg, dWu, dWd, ws)
    torch.cuda.synchronize()
    active = [e for e in range(E) if ROWS[e]]
    assert ids.tolist() == active + [-1] * (E - len(active)) and int(n_act) == len(active)
    worst = {}
    for slot, e in enumerate(active):
        r = slice(int(off[e]), int(off[e + 1]))
        x, dy = X[r].double(), dY[r].double()
        x.requires_grad_(True)
        ws_ = [t[e].double().requires_grad_(True) for t in ([Wg, Wu, Wd] if gated else [Wg, Wd])]
        z = x @ ws_[0]
        h = torch.nn.functional.silu(z) * (x @ ws_[1]) if gated else torch.nn.functional.gelu(z)
        y = h @ ws_[-1]
        y.backward(dy)
        pairs = {"G": (G[r], z), "H": (H[r], h), "Y": (Y[r], y), "dX": (dX[r], x.grad), "dWg": (dWg[slot], ws_[0].grad),
                 "dWd": (dWd[slot], ws_[-1].grad)}
        if gated:
            pairs["dWu"] = (dWu[slot], ws_[1].grad)
        for k, (got, ref) in pairs.items():
            worst[k] = max(worst.get(k, 0.0), rel(got, ref.detach()))
    print(dtype, d, F, ffn, {k: f"{v:.1e}" for k, v in worst.items()})
    assert all(v <= TOL[dtype] for v in worst.values()), worst


@pytest.mark.parametrize("poison", [float("inf"), float("nan")])
@pytest.mark.parametrize("ffn", ["swiglu", "gelu"])
@pytest.mark.parametrize("dtype,d,F", [(t, *s) for t in ("f32", "bf16") for s in ((72, 104), (264, 520), (64, 192))] +
                         [("bf16", 1096, 104), ("bf16", 1152, 192)])   # the last two: the tall tiles
def test_nothing_leaks_from_other_groups(dtype, d, F, ffn, poison):
    """Tiles read past the rows and columns of their group, into the next group's rows, weights and K values: whatever
    stands there, the outputs of a group are the same bits."""
    import paper_2502_02581_amd as moe

    dev, rows = "cuda:0", [33, 70, 1, 300, 17] + ([700, 1100, 900] if d > 1000 else [])
    E, n = len(rows), sum(rows)
    assert dtype == "f32" or small_tiles(E, n, d, F) == (d < 1000)
    shape = moe.MoEShape(n, d, E, 1, F, dtype)
    dt = shape.torch_dtype
    g = torch.Generator().manual_seed(d + F)
    rnd = lambda std, *s: (torch.randn(*s, generator=g) * std).to(dt).to(dev)
    X, dY, w = rnd(1.0, n, d), rnd(1.0, n, d), [rnd(d ** -0.5, E, d, F), rnd(d ** -0.5, E, d, F), rnd(F ** -0.5, E, F, d)]
    if ffn == "gelu":
        w[1] = None
    off = [sum(rows[:e]) for e in range(E + 1)]
    offs = torch.tensor(off, dtype=torch.int32, device=dev)
    ws = torch.full((max(moe.moe_expert_fwd_workspace_bytes(shape, E, n, False), moe.moe_expert_bwd_workspace_bytes(shape, E, n, False)),),
                    0xff, dtype=torch.uint8, device=dev)

    def run(X, dY, w):
        new = lambda *s: torch.full(s, 7.0, dtype=dt, device=dev)
        G, U, H, Y, dX, dWg, dWu, dWd = (new(*s) for s in ((n, F), (n, F), (n, F), (n, d), (n, d), (E, d, F), (E, d, F), (E, F, d)))
        ids, n_act = torch.empty(E, dtype=torch.int32, device=dev), torch.empty(1, dtype=torch.int32, device=dev)
        moe.moe_expert_fwd(shape, E, offs, n, X, *w, G, U, H, Y, ws)
        moe.moe_expert_bwd(shape, E, offs, n, X, *w, G, U, H, dY, dX, ids, n_act, dWg, dWu, dWd, ws)
        return [G, U, H, Y, dX], [dWg, dWu, dWd]

    clean = run(X, dY, w)
    for bad in range(E):
        X2, dY2, w2 = X.clone(), dY.clone(), [None if t is None else t.clone() for t in w]
        for t in (X2, dY2):
            t[off[bad]:off[bad + 1]] = poison
        for t in w2:
            if t is not None:
                t[bad] = poison
        got = run(X2, dY2, w2)
        for e in range(E):
            if e != bad:
                assert all(torch.equal(a[off[e]:off[e + 1]], b[off[e]:off[e + 1]]) for a, b in zip(clean[0], got[0])), (bad, e)
                assert all(torch.equal(a[e], b[e]) for a, b in zip(clean[1], got[1])), (bad, e)


# hidden size, rows of one group, width: row tiles x column tiles that fill no round of 256 tiles, one exactly, a few, and more than are
# dealt in short runs; last bands of one to four row tiles.  Tiles of short calls, 64 x 64 of each product: 255, 256, 264, 1536, 1792,
# 1800 and 300, and 600 to 14400; tall ones, 256 x 128: the same numbers, the last of 64-row tiles.
@pytest.mark.parametrize("d,n,F", [(64, 320, 51 * 64), (64, 256, 64 * 64), (64, 449, 33 * 64), (64, 384, 256 * 64), (64, 448, 256 * 64),
                                   (64, 576, 200 * 64 - 8), (64, 40, 300 * 64),
                                   (64, 1280, 51 * 128), (64, 1024, 64 * 128), (64, 1793, 33 * 128), (64, 1536, 256 * 128),
                                   (64, 1792, 256 * 128), (64, 2304, 200 * 128 - 8), (64, 40, 300 * 128),
                                   (2688, 1280, 51 * 128), (3392, 1024, 64 * 128), (1920, 1793, 33 * 128), (2240, 1536, 256 * 128),
                                   (1984, 1792, 256 * 128), (1536, 2304, 200 * 128 - 8), (4672, 40, 300 * 128)])
def test_every_tile_of_a_launch_is_computed(d, n, F):
    import paper_2502_02581_amd as moe

    dev = "cuda:0"
    assert small_tiles(1, n, d, F) == (d == 64)
    shape = moe.MoEShape(n, d, 1, 1, F, "bf16")
    g = torch.Generator(device=dev).manual_seed(n)
    rnd = lambda std, *s: torch.empty(*s, dtype=torch.bfloat16, device=dev).normal_(0.0, std, generator=g)
    X, Wg, Wu, Wd = rnd(1.0, n, d), rnd(d ** -0.5, 1, d, F), rnd(d ** -0.5, 1, d, F), rnd(F ** -0.5, 1, F, d)
    G, U, H = (torch.full((n, F), float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(3))
    Y = torch.empty(n, d, dtype=torch.bfloat16, device=dev)
    ws = torch.empty(moe.moe_expert_fwd_workspace_bytes(shape, 1, n, False), dtype=torch.uint8, device=dev)
    moe.moe_expert_fwd(shape, 1, torch.tensor([0, n], dtype=torch.int32, device=dev), n, X, Wg, Wu, Wd, G, U, H, Y, ws)
    for got, w in ((G, Wg), (U, Wu)):
        want = X.float() @ w[0].float()
        # one rounding to bf16, at most 2^-9 of the value, and as much again; beside it, where the value is small, the fp32 sums
        # of d terms on both sides: sqrt(2 d) 2^-24 / sqrt(3) of a value of order one, six times that for the largest of 5e7
        assert float(((got.float() - want).abs() - want.abs() * 2 ** -8).max()) <= max(1e-5, 6 * d ** 0.5 * 2 ** -24)
    assert bool(torch.isfinite(H).all())

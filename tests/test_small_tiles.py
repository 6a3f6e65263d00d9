"""The small tiles of short bf16 calls and the full ones beyond their lines: groups at the edges of both, and plans that the
dispatch made for the other family."""
import pytest

torch = pytest.importorskip("torch")

import paper_2502_02581_amd as moe

from .helpers import small_tiles

pytestmark = pytest.mark.gpu
EDGES = [0, 1, 7, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 191, 193, 224, 255, 256, 257, 300, 0, 511, 513]
DEV = "cuda:0"


def _err(got, ref):
    return float((got.double().cpu() - ref).abs().max() / ref.abs().max())


@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("d,F", [(72, 136), (128, 64), (1032, 136), (1088, 264)])   # 3.6 thousand rows: the last two beyond the line
def test_groups_at_the_edges(d, F, gated):
    counts = EDGES + ([500] if d > 1000 else [])
    E, A = len(counts), sum(counts)
    assert small_tiles(E, A, d, F) == (d < 1000)
    r = torch.Generator().manual_seed(d + F)
    n = lambda *s: torch.randn(*s, generator=r).bfloat16()
    X, dY = n(A, d), n(A, d)
    Wg, Wu, Wd = n(E, d, F) / d ** 0.5, n(E, d, F) / d ** 0.5, n(E, F, d) / F ** 0.5
    off = torch.tensor([0] + counts).cumsum(0).int()
    shape = moe.MoEShape(A, d, E, 1, F, "bf16")
    b = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device=DEV)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=DEV)
    G, U, H, Y, dX = b(A, F), b(A, F), b(A, F), b(A, d), b(A, d)
    ids, na, dWg, dWu, dWd = i32(E), i32(1), b(E, d, F), b(E, d, F), b(E, F, d)
    ws = torch.empty(max(moe.moe_expert_fwd_workspace_bytes(shape, E, A, False), moe.moe_expert_bwd_workspace_bytes(shape, E, A, False)),
                     dtype=torch.uint8, device=DEV)
    g = lambda t: t.to(DEV)
    args = (g(off), A, g(X), g(Wg), g(Wu) if gated else None, g(Wd), G, U if gated else None, H)
    moe.moe_expert_fwd(shape, E, *args, Y, ws)
    moe.moe_expert_bwd(shape, E, *args, g(dY), dX, ids, na, dWg, dWu if gated else None, dWd, ws)
    slot = {int(e): i for i, e in enumerate(ids[: int(na)].tolist())}
    assert sorted(slot) == [e for e in range(E) if counts[e]]
    f = lambda t: t.double()
    refY, refdX = torch.zeros(A, d, dtype=torch.float64), torch.zeros(A, d, dtype=torch.float64)
    worst = 0.0
    Gc, Uc, Hc = f(G.cpu()), f(U.cpu()), f(H.cpu())
    for e in slot:
        s = slice(int(off[e]), int(off[e + 1]))
        x, dy = f(X[s]), f(dY[s])
        z = x @ f(Wg[e])
        worst = max(worst, _err(G[s], z))
        # later products from the saved activations, which are rounded to bf16
        z, h = Gc[s], Hc[s]
        dh = dy @ f(Wd[e]).T
        if gated:
            sg = torch.sigmoid(z)
            dg, du = dh * Uc[s] * sg * (1 + z * (1 - sg)), dh * z * sg
            worst = max(worst, _err(U[s], x @ f(Wu[e])), _err(H[s], z * sg * Uc[s]))
        else:
            cdf, pdf = 0.5 * (1 + torch.erf(z * 0.5 ** 0.5)), torch.exp(-0.5 * z * z) * 0.3989422804014327
            dg, du = dh * (cdf + z * pdf), None
            worst = max(worst, _err(H[s], z * cdf))
        refY[s], refdX[s] = h @ f(Wd[e]), dg @ f(Wg[e]).T + (du @ f(Wu[e]).T if gated else 0)
        worst = max(worst, _err(dWg[slot[e]], x.T @ dg), _err(dWd[slot[e]], h.T @ dy))
        if gated:
            worst = max(worst, _err(dWu[slot[e]], x.T @ du))
    # two roundings to bf16 (2^-9 each, of the value and of an operand) and the spread of the operands' errors in short sums
    assert max(worst, _err(Y, refY), _err(dX, refdX)) <= 1.2e-2


@pytest.mark.parametrize("given,used", [(8, 136), (6400, 136), (136, 6400)])
def test_plan_of_another_width(given, used):
    """A dispatch need not be told the experts' width: a plan for the other family's tiles gives the same bits, forward and backward."""
    T, d, E, k = 1500, 512, 12, 2
    assert small_tiles(E, T * k, d, used) == (used == 136) and small_tiles(E, T * k, d, given) == (given < 6400)
    r = torch.Generator().manual_seed(1)
    logits = torch.randn(T, E, generator=r)
    logits[:, 3] += 2.0
    X = torch.randn(T, d, generator=r).bfloat16().to(DEV)
    A = T * k
    W = [(torch.randn(*s, generator=r) / s[1] ** 0.5).bfloat16().to(DEV) for s in ((E, d, used), (E, d, used), (E, used, d))]
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32, device=DEV)
    b = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device=DEV)
    sd, su = moe.MoEShape(T, d, E, k, given, "bf16"), moe.MoEShape(T, d, E, k, used, "bf16")
    idx, w, counts, off, row, src, Xp = i32(T, k), torch.zeros(T, k, device=DEV), i32(E), i32(E + 1), i32(A), i32(A), b(A, d)
    plan = torch.empty(moe.moe_expert_plan_bytes(sd), dtype=torch.uint8, device=DEV)
    ids, na = i32(E), i32(1)
    ws = torch.empty(max(moe.moe_route_dispatch_workspace_bytes(sd), moe.moe_expert_fwd_workspace_bytes(su, E, A, False)), dtype=torch.uint8, device=DEV)
    moe.moe_route_dispatch_plan(sd, logits.to(DEV), X, 0.0, idx, w, counts, off, row, src, Xp, None, None, plan, ids, na, ws)
    dY = torch.randn(A, d, generator=r).bfloat16().to(DEV)
    ws = torch.empty(max(ws.numel(), moe.moe_expert_bwd_workspace_bytes(su, E, A, False)), dtype=torch.uint8, device=DEV)
    out = []
    for p in (plan, None):
        G, U, H, Y, dX, dW = b(A, used), b(A, used), b(A, used), b(A, d), b(A, d), [b(E, d, used), b(E, d, used), b(E, used, d)]
        own_ids, own_na = (ids, na) if p is not None else (i32(E), i32(1))
        both = dict(d_ff=used, n_groups=E, n_rows=A, offsets=off, Xin=Xp, Wg=W[0], Wu=W[1], Wd=W[2], G=G, U=U, H=H, ws=ws, ws_bytes=ws.numel(), plan=p)
        moe.moe_experts_fwd(su, dict(both, Yout=Y), None)
        moe.moe_experts_bwd(su, dict(both, dYin=dY, dXin=dX, active_ids=own_ids, n_active=own_na, dWg_c=dW[0], dWu_c=dW[1], dWd_c=dW[2]), None)
        out.append((G, U, H, Y, dX, *dW, own_ids, own_na))
    for x, y in zip(*out):
        assert torch.equal(x, y)

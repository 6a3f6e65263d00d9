"""moe_experts_fwd / _bwd (routed and shared experts in common launches) against the calls of either set alone."""
import pytest
import torch

from .helpers import small_tiles

pytestmark = pytest.mark.gpu

# T, d, E, k, d_ff, shared experts, their width, routed activation, shared activation, rows read in place
CASES = [
    (1, 64, 4, 2, 64, 1, 64, "swiglu", "swiglu", False),          # one token
    (16, 256, 12, 4, 192, 4, 192, "swiglu", "swiglu", True),      # a few rows an expert, long shared sums
    (257, 128, 5, 2, 200, 2, 128, "swiglu", "swiglu", False),     # only the routed width has a K tail
    (300, 192, 6, 3, 128, 1, 72, "swiglu", "swiglu", True),       # only the shared width has one
    (700, 136, 6, 2, 264, 3, 328, "gelu", "gelu", False),         # ragged everywhere, two-matrix experts
    (1500, 512, 3, 1, 320, 1, 640, "swiglu", "swiglu", False),    # tall tiles on both sides
    (130, 64, 8, 2, 64, 2, 128, "swiglu", "gelu", False),         # two activations: no common launch
    (130, 64, 8, 2, 64, 2, 128, "gelu", "swiglu", False),
    (0, 64, 4, 2, 64, 2, 64, "swiglu", "swiglu", False),          # no tokens
    (1743, 832, 8, 2, 128, 1, 64, "swiglu", "swiglu", False),     # shared sums in parts alone
    (42, 1472, 8, 2, 1024, 2, 1024, "swiglu", "swiglu", False),
]
# bf16: the cases above are short calls, with tiles of their own; these take the tall ones
TALL_CASES = [
    (1701, 1024, 5, 2, 192, 2, 192, "swiglu", "swiglu", True),    # no K tail, rows read in place
    (1700, 1024, 6, 2, 200, 2, 128, "swiglu", "swiglu", False),   # only the routed width has a K tail
    (1700, 1024, 6, 2, 128, 1, 72, "swiglu", "swiglu", True),     # only the shared width has one
    (1743, 1000, 6, 2, 264, 3, 328, "gelu", "gelu", True),        # ragged everywhere, two-matrix experts
]


@pytest.mark.parametrize("dtype,T,d,E,k,F,S,Fs,act,act_s,gather", [(t, *c) for t in ("f32", "bf16") for c in CASES] +
                         [("bf16", *c) for c in TALL_CASES])
def test_both_sets_in_one_call(dtype, T, d, E, k, F, S, Fs, act, act_s, gather):
    """Routed results are the same bits, and in fp32 shared ones are too (the same parts of their sums, so the same error);
    in bf16 shared ones differ by the order of fp32 sums and by the rounding of the output to its type."""
    import paper_2502_02581_amd as moe

    shape, sshape = moe.MoEShape(T, d, E, k, F, dtype), moe.MoEShape(T, d, E, k, Fs, dtype)
    dt, dev, A = shape.torch_dtype, "cuda", T * k
    assert dtype == "f32" or small_tiles(E, A, d, F) == ((T, d, E, k, F, S, Fs, act, act_s, gather) in CASES)
    g = torch.Generator().manual_seed(T + d + F)
    rnd = lambda *s: (torch.randn(*s, generator=g) * d ** -0.5).to(dt).to(dev)
    X, dY = rnd(T, d), rnd(T, d)
    Wg, Wu, Wd = rnd(E, d, F), rnd(E, d, F) if act == "swiglu" else None, rnd(E, F, d)
    Wsg, Wsu, Wsd = rnd(S, d, Fs), rnd(S, d, Fs) if act_s == "swiglu" else None, rnd(S, Fs, d)
    i32 = lambda *s: torch.full(s, -7, dtype=torch.int32, device=dev)
    idx, w = i32(T, k), torch.empty(T, k, device=dev)
    counts, off, row_of, src_of, Xp, dYp, dw = i32(E), i32(E + 1), i32(A), i32(A), rnd(A, d), rnd(A, d), torch.empty(T, k, device=dev)
    logits = torch.randn(T, E, generator=g).to(dev)
    size = max(moe.moe_dispatch_workspace_bytes(shape), moe.moe_expert_fwd_workspace_bytes(shape, E, A, False),
               moe.moe_expert_bwd_workspace_bytes(shape, E, A, False))
    size_s = max(moe.moe_expert_fwd_workspace_bytes(sshape, S, T, True), moe.moe_expert_bwd_workspace_bytes(sshape, S, T, True))
    ws, ws_s = (torch.empty(n, dtype=torch.uint8, device=dev) for n in (size, size_s))
    moe.moe_route(shape, logits, idx, w)
    moe.moe_dispatch(shape, X, idx, counts, off, row_of, src_of, Xp, ws)

    def bufs():
        new = lambda *s: torch.full(s, float("nan"), dtype=dt, device=dev)
        r = dict(G=new(A, F), U=new(A, F), H=new(A, F), Yout=new(A, d), dXin=new(A, d), active_ids=i32(E), n_active=i32(1),
                 dWg_c=new(E, d, F), dWu_c=new(E, d, F), dWd_c=new(E, F, d))
        s = dict(G=new(S, T, Fs), U=new(S, T, Fs), H=new(S, T, Fs), Yout=new(T, d), dXin=new(T, d), active_ids=i32(S),
                 n_active=i32(1), dWg_c=new(S, d, Fs), dWu_c=new(S, d, Fs), dWd_c=new(S, Fs, d))
        return r, s

    (r, s), (r2, s2) = bufs(), bufs()
    gr = ["dXin", "active_ids", "n_active", "dWg_c", "dWu_c", "dWd_c"]
    if gather:
        moe.moe_expert_fwd_gather(shape, off, src_of, X, Wg, Wu, Wd, r["G"], r["U"], r["H"], r["Yout"], ws)
    else:
        moe.moe_expert_fwd(shape, E, off, A, Xp, Wg, Wu, Wd, r["G"], r["U"], r["H"], r["Yout"], ws)
    moe.moe_expert_fwd(sshape, S, None, T, X, Wsg, Wsu, Wsd, s["G"], s["U"], s["H"], s["Yout"], ws_s)
    moe.moe_combine_bwd(shape, dY, r["Yout"], row_of, w, dYp, dw)
    if gather:
        moe.moe_expert_bwd_gather(shape, off, src_of, Xp, Wg, Wu, Wd, r["G"], r["U"], r["H"], dY, w, dYp, *[r[n] for n in gr], ws)
    else:
        moe.moe_expert_bwd(shape, E, off, A, Xp, Wg, Wu, Wd, r["G"], r["U"], r["H"], dYp, *[r[n] for n in gr], ws)
    moe.moe_expert_bwd(sshape, S, None, T, X, Wsg, Wsu, Wsd, s["G"], s["U"], s["H"], dY, *[s[n] for n in gr], ws_s)

    fwd = ("G", "U", "H", "Yout")
    base = dict(d_ff=F, n_groups=E, n_rows=A, offsets=off, Wg=Wg, Wu=Wu, Wd=Wd)
    base_s = dict(d_ff=Fs, n_groups=S, n_rows=T, Xin=X, Wg=Wsg, Wu=Wsu, Wd=Wsd)
    bands = []

    def workspaces(query):   # of exactly the queried sizes, filled, between bands in one buffer: one launch writes both
        n, n_s = query(shape, E, A, False), query(sshape, S, T, True)
        at = 4096 + (n + 255) // 256 * 256 + 4096
        big = torch.full((at + n_s + 4096,), 0xA5, dtype=torch.uint8, device=dev)
        bands.extend((big[:4096], big[4096 + n:at], big[at + n_s:]))
        for b, piece, m in ((base, big[4096:4096 + n], n), (base_s, big[at:at + n_s], n_s)):
            piece.fill_(255)
            b.update(ws=piece, ws_bytes=m)

    workspaces(moe.moe_expert_fwd_workspace_bytes)
    moe.moe_experts_fwd(shape, dict(base, Xin=X if gather else Xp, src_of=src_of if gather else None, **{n: r2[n] for n in fwd}),
                        dict(base_s, **{n: s2[n] for n in fwd}))
    workspaces(moe.moe_expert_bwd_workspace_bytes)
    in_place = dict(src_of=src_of, dY=dY, row_w=w) if gather else {}
    moe.moe_experts_bwd(shape, dict(base, Xin=Xp, dYin=dYp, **in_place, **{n: r2[n] for n in gr + ["G", "U", "H"]}),
                        dict(base_s, dYin=dY, **{n: s2[n] for n in gr + ["G", "U", "H"]}))
    torch.cuda.synchronize()
    assert all(bool((band == 0xA5).all()) for band in bands)
    for n in r:
        assert torch.equal(r[n].view(torch.uint8), r2[n].view(torch.uint8)), n
    for n in s:
        a, b = s[n], s2[n]
        if T == 0 or dtype == "f32" or n in ("active_ids", "n_active") or (act_s == "gelu" and n in ("U", "dWu_c")):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), n
        else:
            # half a unit in the last place of both, 2 * 2^-9, for each of the two roundings on the way to an output
            err = float((a.double() - b.double()).norm() / a.double().norm())
            assert err <= 8e-3, (n, err)


# The first three: sizes at which, without the limit in choose_direct, more room than a set asks for alone would make more parts beside
# these routed rows, of dH (2 and 1 -> 4 and 2 with 16 MiB more), dH (3 -> 4), gate/up (3 -> 4).  They take the tall tiles: with the costs of
# the small ones, the others', no size out of 350 thousand drawn ones makes more parts.
@pytest.mark.parametrize("T,d,E,k,F,S,Fs", [(997, 3968, 8, 1, 64, 2, 192), (667, 2240, 4, 3, 64, 2, 192), (1366, 3136, 6, 2, 128, 1, 384),
                                            (256, 256, 120, 2, 1024, 2, 1024), (80, 5376, 48, 1, 128, 4, 64), (85, 3840, 65, 1, 256, 1, 256)])
def test_room_beyond_the_query_changes_nothing(T, d, E, k, F, S, Fs):
    """A call gives the same bits with every workspace from the size queries' answer on."""
    import paper_2502_02581_amd as moe

    shape, sshape = moe.MoEShape(T, d, E, k, F, "bf16"), moe.MoEShape(T, d, E, k, Fs, "bf16")
    A, dev = T * k, "cuda"
    assert small_tiles(E, A, d, F) == (T < 500)
    g = torch.Generator().manual_seed(T + d)
    rnd = lambda *s: (torch.randn(*s, generator=g) * d ** -0.5).bfloat16().to(dev)
    X, dY, Xp, dYp = rnd(T, d), rnd(T, d), rnd(A, d), rnd(A, d)
    w, ws_ = dict(Wg=rnd(E, d, F), Wu=rnd(E, d, F), Wd=rnd(E, F, d)), dict(Wg=rnd(S, d, Fs), Wu=rnd(S, d, Fs), Wd=rnd(S, Fs, d))
    off = torch.arange(E + 1, dtype=torch.int32, device=dev) * (A // E)
    off[-1] = A

    def run(room):
        new, i32 = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device=dev), lambda n: torch.zeros(n, dtype=torch.int32, device=dev)
        a = dict(G=new(A, F), U=new(A, F), H=new(A, F))
        b = dict(G=new(S, T, Fs), U=new(S, T, Fs), H=new(S, T, Fs))
        grads = lambda n, f, r: dict(dXin=new(r, d), dWg_c=new(n, d, f), dWu_c=new(n, d, f), dWd_c=new(n, f, d), active_ids=i32(n), n_active=i32(1))
        outs = []
        for call, query in ((moe.moe_experts_fwd, moe.moe_expert_fwd_workspace_bytes), (moe.moe_experts_bwd, moe.moe_expert_bwd_workspace_bytes)):
            n, n_s = query(shape, E, A, False), query(sshape, S, T, True) + room
            t, t_s = torch.empty(n, dtype=torch.uint8, device=dev), torch.empty(n_s, dtype=torch.uint8, device=dev)
            more, more_s = (dict(Yout=new(A, d)), dict(Yout=new(T, d))) if call is moe.moe_experts_fwd else \
                (dict(dYin=dYp, **grads(E, F, A)), dict(dYin=dY, **grads(S, Fs, T)))
            call(shape, dict(d_ff=F, n_groups=E, n_rows=A, offsets=off, Xin=Xp, ws=t, ws_bytes=n, **w, **a, **more),
                 dict(d_ff=Fs, n_groups=S, n_rows=T, Xin=X, ws=t_s, ws_bytes=n_s, **ws_, **b, **more_s))
            outs += [*more.values(), *more_s.values()]
        return outs + [*a.values(), *b.values()]

    for x, y in zip(run(0), run(16 << 20)):
        assert torch.equal(x, y)


def test_sets_are_checked():
    import paper_2502_02581_amd as moe

    shape = moe.MoEShape(16, 64, 4, 2, 64, "bf16")
    t = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    off = torch.zeros(5, dtype=torch.int32, device="cuda")
    b = t.view(torch.bfloat16)
    names = ("Xin", "Wg", "Wu", "Wd", "G", "U", "H", "Yout")
    good = dict({n: b for n in names}, d_ff=64, ws=t, ws_bytes=t.numel())
    routed, shared = dict(good, n_groups=4, n_rows=32, offsets=off), dict(good, n_groups=1, n_rows=16)
    for r, s, msg in [(dict(routed, offsets=None), shared, "null"), (routed, dict(shared, offsets=off), "null"),
                      (dict(routed, ws_bytes=16), shared, "workspace"), (routed, dict(shared, ws_bytes=16), "workspace"),
                      (routed, dict(shared, Xin=b[1:]), "aligned"), (routed, dict(shared, d_ff=60), "multiples of 8"),
                      (dict(routed, src_of=off, n_rows=30), shared, "in place"), (routed, dict(shared, Yout=None), "null")]:
        with pytest.raises(moe.MoEError, match=msg):
            moe.moe_experts_fwd(shape, r, s)


@pytest.mark.parametrize("dtype,T,d,E,k", [(t, *s) for t in ("f32", "bf16") for s in (
    (0, 64, 5, 2), (1, 64, 1, 1), (700, 64, 6, 2), (517, 64, 64, 3), (40, 64, 300, 8), (60, 64, 1024, 4))] +
    [("bf16", 700, 2496, 6, 2), ("bf16", 1301, 1000, 64, 3)])   # the last two: the tall tiles
def test_plan_of_the_dispatch(dtype, T, d, E, k):
    """A plan that the dispatch wrote gives the bits of the calls that build their own, and the same active_ids."""
    import paper_2502_02581_amd as moe

    F, A, dev = 72, T * k, "cuda"
    assert dtype == "f32" or small_tiles(E, A, d, F) == (d == 64)
    shape = moe.MoEShape(T, d, E, k, F, dtype)
    dt = shape.torch_dtype
    g = torch.Generator().manual_seed(T + E)
    rnd = lambda *s: (torch.randn(*s, generator=g) * d ** -0.5).to(dt).to(dev)
    i32 = lambda *s: torch.full(s, -7, dtype=torch.int32, device=dev)
    logits = (torch.randn(T, E, generator=g) + 2.0 * torch.randn(E, generator=g)).to(dev)
    X, dY, Wg, Wu, Wd = rnd(T, d), rnd(A, d), rnd(E, d, F), rnd(E, d, F), rnd(E, F, d)
    idx, w, counts, off, row_of, src_of, Xp = i32(T, k), torch.empty(T, k, device=dev), i32(E), i32(E + 1), i32(A), i32(A), rnd(A, d)
    size = max(moe.moe_route_dispatch_workspace_bytes(shape), moe.moe_expert_fwd_workspace_bytes(shape, E, A, False),
               moe.moe_expert_bwd_workspace_bytes(shape, E, A, False))
    ws = torch.full((size,), 255, dtype=torch.uint8, device=dev)
    need = moe.moe_expert_plan_bytes(shape)
    big = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=dev)
    with pytest.raises(moe.MoEError, match="plan of"):
        moe.moe_route_dispatch_plan(shape, logits, X, 0.0, idx, w, counts, off, row_of, src_of, Xp, None, None, big[:need - 16], i32(E), i32(1), ws)
    outs = []
    for plan in (big[:need], None):
        ids, n_act = i32(E), i32(1)
        if plan is not None:
            moe.moe_route_dispatch_plan(shape, logits, X, 0.0, idx, w, counts, off, row_of, src_of, Xp, None, None, plan, ids, n_act, ws)
        else:
            moe.moe_route_dispatch(shape, logits, X, 0.0, idx, w, counts, off, row_of, src_of, Xp, None, None, ws)
        new = lambda *s: torch.full(s, float("nan"), dtype=dt, device=dev)
        o = dict(G=new(A, F), U=new(A, F), H=new(A, F))
        base = dict(d_ff=F, n_groups=E, n_rows=A, offsets=off, Xin=Xp, Wg=Wg, Wu=Wu, Wd=Wd, ws=ws, ws_bytes=size, plan=plan, **o)
        Y, gr = new(A, d), dict(dXin=new(A, d), dWg_c=new(E, d, F), dWu_c=new(E, d, F), dWd_c=new(E, F, d))
        moe.moe_experts_fwd(shape, dict(base, Yout=Y), None)
        ws.fill_(255)
        moe.moe_experts_bwd(shape, dict(base, dYin=dY, active_ids=ids, n_active=n_act, **gr), None)
        outs.append([Y, *o.values(), *gr.values(), ids, n_act, counts.clone(), off.clone()])
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert bool((big[need:] == 0xA5).all())


@pytest.mark.parametrize("S", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_of_a_pass_that_was_put_back(dtype, S):
    """Two micro-batches in flight on one MoEHotPath: the tensors of the first are saved, the second runs forward with another
    routing, the first ones are put back.  Its backward pass gives the bits of a backward pass right after its forward pass."""
    import paper_2502_02581_amd as moe

    T, d, E, k, F = 700, 128, 6, 2, 192
    shape = moe.MoEShape(T, d, E, k, F, dtype)
    g = torch.Generator().manual_seed(3)
    new = lambda *n: torch.randn(*n, generator=g).to("cuda", shape.torch_dtype)
    X, dY = new(T, d), new(T, d)
    w = [new(E, d, F), new(E, d, F), new(E, F, d)] + ([new(S, d, F), new(S, d, F), new(S, F, d)] if S else [])
    logits = torch.randn(2, T, E, generator=g)
    logits[0, :, 0] += 2.0   # the two routings load other experts
    logits[1, :, 4] += 2.0
    logits = logits.to("cuda")
    hp = moe.MoEHotPath(shape, S, F if S else 0, "cuda:0")
    names = ["dX", "dw", "active_ids", "n_active", "dWg_c", "dWu_c", "dWd_c"] + (["dWsg", "dWsu", "dWsd"] if S else [])
    for n in names:
        hp.b[n].zero_()
    hp.forward(logits[0], X, *w)
    saved = {n: t.clone() for n, t in hp.b.items()}
    hp.backward(dY, X, *w)
    want = {n: hp.b[n].clone() for n in names}
    hp.forward(logits[1], X, *w)
    for n, t in saved.items():
        hp.b[n].copy_(t)
    hp.backward(dY, X, *w)
    for n in names:
        assert torch.equal(hp.b[n], want[n]), n


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("S", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_forward_leaves_the_last_gradients_alone(dtype, S, fused):
    """A forward pass after a backward pass (validation, the next micro-batch) writes none of that pass's gradients, nor the ids
    that say which experts the compact slots belong to."""
    import paper_2502_02581_amd as moe

    T, d, E, k, F = 300, 128, 8, 2, 192
    shape = moe.MoEShape(T, d, E, k, F, dtype)
    g = torch.Generator().manual_seed(4)
    new = lambda *n: torch.randn(*n, generator=g).to("cuda", shape.torch_dtype)
    X, dY = new(T, d), new(T, d)
    w = [new(E, d, F), new(E, d, F), new(E, F, d)] + ([new(S, d, F), new(S, d, F), new(S, F, d)] if S else [])
    logits = torch.randn(2, T, E, generator=g)
    logits[0, :, :3] -= 100.0   # experts 3 to 7, then 0 to 4
    logits[1, :, 5:] -= 100.0
    logits = logits.to("cuda")
    hp = moe.MoEHotPath(shape, S, F if S else 0, "cuda:0", aux_alpha=0.01, fused=fused)
    names = ["dX", "dw", "dlogits", "active_ids", "n_active", "dWg_c", "dWu_c", "dWd_c"]
    names += ["dWsg", "dWsu", "dWsd", "s_active_ids", "s_n_active"] if S else []
    for n in names:
        hp.b[n].zero_()
    hp.forward(logits[0], X, *w)
    hp.backward(dY, X, *w)
    want = {n: hp.b[n].clone() for n in names}
    assert hp.b["active_ids"].tolist() == [3, 4, 5, 6, 7, -1, -1, -1] and hp.b["n_active"].item() == 5
    hp.forward(logits[1], X, *w)
    for n in names:
        assert torch.equal(hp.b[n], want[n]), n


@pytest.mark.parametrize("gated", [(True, False), (False, True)])   # the routed set, the shared set
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_overlap_where_no_common_launch_is_possible(dtype, gated, monkeypatch):
    """One set gated, the other not: with overlap_shared the shared calls go to the second stream, and eager passes, passes on a
    stream of the caller's and replays of a captured one give the bits of the order one after the other."""
    import paper_2502_02581_amd as moe
    from paper_2502_02581_amd import binding

    T, d, E, k, F, S, Fs = 700, 192, 6, 2, 256, 2, 128
    shape = moe.MoEShape(T, d, E, k, F, dtype)
    g = torch.Generator().manual_seed(6)
    new = lambda *n: (torch.randn(*n, generator=g) * 0.1).to("cuda", shape.torch_dtype)
    w = [new(E, d, F), new(E, d, F) if gated[0] else None, new(E, F, d), new(S, d, Fs), new(S, d, Fs) if gated[1] else None, new(S, Fs, d)]
    a, b = ((torch.randn(T, E, generator=g).cuda(), new(T, d), new(T, d)) for _ in range(2))
    names = ["Y", "dX", "dw", "dlogits", "dWg_c", "dWd_c", "dWsg", "dWsd"] + ["dWu_c"] * gated[0] + ["dWsu"] * gated[1]
    streams = []
    for call in ("moe_expert_fwd", "moe_expert_bwd"):
        def spy(*args, real=getattr(binding, call)):
            streams.append(args[-1].cuda_stream)
            return real(*args)
        monkeypatch.setattr(binding, call, spy)

    def layer(overlap):
        hp = moe.MoEHotPath(shape, S, Fs, "cuda:0", overlap_shared=overlap, aux_alpha=0.01)
        for n in names:
            hp.b[n].zero_()
        return hp

    def step(hp, q, stream=None):
        hp.forward(q[0], q[1], *w, stream=stream)
        hp.backward(q[2], q[1], *w, stream=stream)

    def result(hp):
        torch.cuda.synchronize()
        return {n: hp.b[n].clone() for n in names}

    hp = layer(False)
    step(hp, a)
    want = result(hp)
    assert not streams
    hp = layer(True)
    main = torch.cuda.current_stream().cuda_stream
    for _ in range(3):   # repeated passes reuse the buffers and the events
        step(hp, b)
        step(hp, a)
    got = result(hp)
    assert len(streams) == 12 and len(set(streams)) == 1 and streams[0] != main
    assert all(torch.equal(got[n], want[n]) for n in names)
    step(hp, b)
    torch.cuda.synchronize()
    own = torch.cuda.Stream()
    step(hp, a, own)
    assert all(torch.equal(v, want[n]) for n, v in result(hp).items())
    step(hp, b)
    torch.cuda.synchronize()
    step(hp, a, own.cuda_stream)
    assert all(torch.equal(v, want[n]) for n, v in result(hp).items())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(hp, a)
    for _ in range(3):
        step(hp, b)
        torch.cuda.synchronize()
        graph.replay()
        assert all(torch.equal(v, want[n]) for n, v in result(hp).items())
    # a call that is refused after the shared experts' one was queued: the main stream waits for it all the same
    joined = []
    monkeypatch.setattr(hp, "_join", lambda m, real=hp._join: (joined.append(m), real(m)))
    w[2] = w[2].double()
    with pytest.raises(moe.MoEError, match="Wd"):
        hp.forward(a[0], a[1], *w)
    with pytest.raises(moe.MoEError, match="Wd"):
        hp.backward(a[2], a[1], *w)
    torch.cuda.synchronize()
    assert len(joined) == 2

"""fp32 products at the edges of their tiles, and what a sum of bf16 products must not get wrong: few products, values that no
finite sum holds, values at the ends of the range."""
import re

import pytest

torch = pytest.importorskip("torch")

import paper_2502_02581_amd as moe

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _router(T, d, E, X, W, g, parts=True):
    """The three products; without parts: with the workspaces that the calls refuse to go below, so that each sum is one."""
    shape = moe.MoEShape(T, d, E, 1, 8, "f32")
    dev = "cuda:0"
    X, W, g = X.to(dev), W.to(dev), g.to(dev)
    ws = torch.empty(max(moe.moe_router_fwd_workspace_bytes(shape), moe.moe_router_bwd_workspace_bytes(shape)), dtype=torch.uint8,
                     device=dev)
    logits, dW, dX = torch.empty(T, E, device=dev), torch.empty_like(W), torch.empty_like(X)
    for call in (lambda ws: moe.moe_router_fwd(shape, X, W, logits, ws), lambda ws: moe.moe_router_bwd(shape, X, W, g, dW, dX, False, ws)):
        n = ws.numel()
        if not parts:
            try:
                n = 16
                call(ws[:n])
            except moe.MoEError as e:
                n = int(re.search(r"need (\d+)", str(e)).group(1))
        call(ws[:n])
    return logits.cpu(), dW.cpu(), dX.cpu()


def _check(got, a, b):
    """Any value: |got - ab| <= (roundings + 4) u |a||b|, two roundings per eight values of K (at most one per value), the parts of K, the
    dropped products (below 4 u).  All of them, of operands about zero: the 2-norm of the error against that of the result, the
    roundings as independent ones.  (Without one of the six products of parts: 40 u and more.)"""
    ref, scale = a.double() @ b.double(), a.double().abs() @ b.double().abs()
    k = a.shape[1]
    n = min(k, 2 * ((k + 7) // 8))
    err = (got.double() - ref).abs()
    assert (err <= (n + 16 + 4) * U * scale).all()
    assert err.norm() <= (1 + n ** 0.5) * U * ref.norm()


def _fp32_sum(a, b):
    """ab with one rounding per product, as the fp32 matrix instruction sums."""
    s = torch.zeros(a.shape[0], b.shape[1])
    for k in range(a.shape[1]):
        s = (s.double() + a[:, k, None].double() * b[k].double()).float()
    return s


@pytest.mark.parametrize("T", [1, 2, 8, 9, 15, 16, 17, 31, 33, 64, 65, 127, 128, 129, 300])
@pytest.mark.parametrize("d,E", [(8, 64), (24, 128), (40, 60), (136, 192), (1032, 8)])
def test_products_at_the_edges(T, d, E):
    r = torch.Generator().manual_seed(T * 1000 + d)
    X, W, g = (torch.randn(*s, generator=r) for s in ((T, d), (d, E), (T, E)))
    logits, dW, dX = _router(T, d, E, X, W, g)
    _check(logits, X, W)
    _check(dW, X.T, g)
    _check(dX, g, W.T)


@pytest.mark.parametrize("T,d,E", [(70, 136, 64), (300, 40, 128)])
def test_values_that_are_not_finite(T, d, E):
    """Infinities and NaN go where fp32 arithmetic takes them, whatever else the tile holds; sums that overflow in parts do too."""
    r = torch.Generator().manual_seed(5)
    X, W, g = (torch.randn(*s, generator=r) for s in ((T, d), (d, E), (T, E)))
    X[3, 5], X[17, 2], X[40, 7] = float("inf"), float("nan"), -float("inf")
    X[41, 7], X[42, 1] = 3.4028234e38, -3.4e38   # the largest values round to infinity in bf16
    W[1], W[9, 3] = 0.0, float("inf")
    logits, dW, dX = _router(T, d, E, X, W, g)
    for got, a, b in ((logits, X, W), (dW, X.T, g), (dX, g, W.T)):
        ref = a.double() @ b.double()
        big = ref.abs() > 3.4028235e38   # (no value lies within rounding of it)
        assert not ((ref.abs() / 3.4028235e38 - 1).abs() < 1e-5).any()
        finite = torch.isfinite(ref) & ~big
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
        assert torch.equal(torch.isinf(got) & (got > 0), (ref > 0) & (torch.isinf(ref) | big))
        assert torch.equal(torch.isinf(got) & (got < 0), (ref < 0) & (torch.isinf(ref) | big))
        z = lambda t: torch.nan_to_num(t.double(), 0.0, 0.0, 0.0)
        scale = z(a).abs() @ z(b).abs()
        assert ((got.double() - ref).abs()[finite] <= ((a.shape[1] + 20) * U * scale)[finite]).all()


@pytest.mark.parametrize("d,n", [(40, 0), (40, 17), (200, 46), (72, 63), (72, 64), (40, 95), (136, 111), (40, 127)])
def test_one_lane_asks_for_the_fp32_instruction(d, n):
    """One value of each tile of 128 x 128 overflows in the sum of its parts and not in fp32 (both operands round up to a power of two
    in bf16): it is right whichever lane and wavefront finds it."""
    T, E = 1920, 256
    r = torch.Generator().manual_seed(7)
    X, W, g = torch.randn(T, d, generator=r), torch.randn(d, E, generator=r), torch.randn(T, E, generator=r)
    rows = [128 * i + (37 * i + n) % 128 for i in range(T // 128)]
    big = 2.0 ** 64 * (1 - 2.0 ** -12)
    X[:, 3], W[3] = 0.0, 0.0
    X[rows, 3] = big
    W[3, [n, 255 - n]] = big
    logits, _, _ = _router(T, d, E, X, W, g)
    ref, scale = X.double() @ W.double(), X.double().abs() @ W.double().abs()
    assert torch.isfinite(logits).all()
    assert ((logits.double() - ref).abs() <= (d + 20) * U * scale).all()


@pytest.mark.parametrize("T,d,E,k", [(1024, 512, 64, 2), (700, 320, 256, 8), (300, 256, 128, 1), (64, 128, 8, 2), (130, 64, 60, 3)])
def test_sums_of_few_products(T, d, E, k):
    """Operands that are mostly zero (gradients of the logits outside the selected experts, sparse tokens): no further off than with
    one rounding per product."""
    r = torch.Generator().manual_seed(T + E)
    X, W, g = torch.randn(T, d, generator=r), torch.randn(d, E, generator=r), torch.zeros(T, E)
    g.scatter_(1, torch.rand(T, E, generator=r).topk(k, 1).indices, torch.randn(T, k, generator=r))
    Xs = X * (torch.rand(T, d, generator=r) < 0.03)
    _, dW, dX = _router(T, d, E, X, W, g, parts=False)
    logits, _, _ = _router(T, d, E, Xs, W, g, parts=False)
    for got, a, b in ((dW, X.T, g), (dX, g, W.T), (logits, Xs, W)):
        ref = a.double() @ b.double()
        assert (got.double() - ref).norm() <= 1.005 * (_fp32_sum(a, b).double() - ref).norm()


@pytest.mark.parametrize("scale", [1e-39, 2.0 ** -126, 1e-36, 2.0 ** -110, 2.0 ** -102, 1e-30, 1e-20, 1.0, 1e18])
def test_ends_of_the_range(scale):
    """Operands of any magnitude keep all of their bits (below 2^-102 their third part does not fit into bf16's range): sums, and single
    products with one."""
    r = torch.Generator().manual_seed(6)
    T, d, E = 65, 72, 64
    X = (torch.rand(T, d, generator=r) + 1.0) * scale   # values of one binade: none below the limit
    W, g = torch.randn(d, E, generator=r), torch.randn(T, E, generator=r)
    logits, dW, dX = _router(T, d, E, X, W, g)
    if scale >= 2.0 ** -120:   # (below, results themselves are rounded at the end of fp32's range)
        _check(logits, X, W)
        _check(dW, X.T, g)
    _check(dX, g, W.T)
    pick = torch.randperm(d, generator=r)[:E]
    one = torch.zeros(d, E)
    one[pick, torch.arange(E)] = 1.0
    logits, _, _ = _router(T, d, E, X, one, g)
    assert torch.equal(logits, X[:, pick])

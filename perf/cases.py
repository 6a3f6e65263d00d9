"""The work that is timed: MoE-layer passes through the package's public entry points.

A case is one layer on one GPU.  `op` says which part of a program it stands for:
  "train"    forward and backward of a training step (MoEHotPath.forward, .backward)
  "forward"  forward only: evaluation, prefill of a long prompt, a decode step of a few tokens
  "router"   the gating network's own GEMMs (moe_router_fwd, moe_router_bwd)
Calls are made eagerly, as a training or serving loop makes them; inputs are on the GPU beforehand.
"""
from __future__ import annotations

import math

import torch

import paper_2502_02581_amd as moe

_DEFAULTS = dict(op="train", T=0, d=0, E=0, k=1, d_ff=0, n_shared=0, d_ff_shared=0, dtype="bf16", gate="softmax",
                 renorm=True, ffn="swiglu", zipf=1.0, stress=False, gather=False, overlap=False, aux=0.001)


def _case(name=None, **kw):
    c = dict(_DEFAULTS, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a decode step: the tokens of 16 sequences through one layer, forward only (latency and launches)
        _case("decode-16", op="forward", T=16, d=2048, E=60, k=4, d_ff=1408, n_shared=4, d_ff_shared=1408, aux=0.0),
        # prefill / evaluation of a short batch with many large experts: bound by reading the weights
        _case("prefill-192", op="forward", T=192, d=7168, E=256, k=8, d_ff=2048, n_shared=1, d_ff_shared=2048,
              gate="sigmoid", zipf=1.2, overlap=True, aux=0.0),
        # the smallest training step, fp32 (the configuration that is checked to 1e-4)
        _case("train-tiny-f32", T=256, d=128, E=8, k=2, d_ff=256, dtype="f32", zipf=0.0),
        # a training step kept in fp32 at the size of a small model's layer
        _case("train-f32", T=2048, d=1024, E=16, k=2, d_ff=2816, dtype="f32", zipf=0.8),
        # sizes that are multiples of 8 only (a hidden size of 1000, a width cut for parameter parity), odd token
        # count and top-k, sigmoid gate without renormalisation, one narrow shared expert
        _case("train-ragged", T=3001, d=1000, E=24, k=3, d_ff=1368, n_shared=1, d_ff_shared=712, gate="sigmoid",
              renorm=False),
        # two-matrix GELU experts, small hidden size: short products, many launches per FLOP
        _case("train-gelu", T=8192, d=768, E=64, k=2, d_ff=3072, ffn="gelu"),
        # ordinary training step with shared experts on the second stream
        _case("train-shared", T=4096, d=2048, E=60, k=4, d_ff=1408, n_shared=4, d_ff_shared=1408, overlap=True),
        # the same layer with top-3 and the ragged last batch of an epoch, token rows read in place
        _case("train-top3-gather", T=2777, d=2048, E=60, k=3, d_ff=1408, n_shared=4, d_ff_shared=1408, gather=True),
        # extreme imbalance: one expert takes 30 % of the tokens, ten take none
        _case("train-stress", T=16384, d=2048, E=60, k=4, d_ff=1408, zipf=1.5, stress=True),
        # few wide experts, no shared ones
        _case("train-wide", T=8192, d=4096, E=16, k=2, d_ff=6400, zipf=0.8),
        # the largest layer: 256 experts, many of them with a handful of rows or none
        _case("train-256", T=8192, d=7168, E=256, k=8, d_ff=2048, n_shared=1, d_ff_shared=2048, gate="sigmoid",
              zipf=1.2, overlap=True),
        # the gating network of the largest layer, forward and backward
        _case("router-256", op="router", T=8192, d=7168, E=256, k=8, d_ff=2048, gate="sigmoid"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(x, m):
    return max(m, x // m * m)


def draw(rng):
    """Another case of the ranges above: token counts from 1 (forward) or 64 (training) to 16384, hidden sizes and
    widths from 128 to 7168 (three in four multiples of 64, the others multiples of 8 only), 4 to 256 experts,
    top-1 to top-8, every option; at most half the arithmetic and weights of the largest listed case."""
    while True:
        op = rng.choice(("train", "train", "train", "forward", "forward", "router"))
        f32 = rng.random() < 0.15
        m = 64 if rng.random() < 0.75 else 8
        c = _case(op=op, T=_log(rng, 64 if op == "train" else 1, 16384), d=_mult(_log(rng, 128, 7168), m),
                  E=_log(rng, 4, 256), d_ff=_mult(_log(rng, 128, 6400), m), dtype="f32" if f32 else "bf16",
                  gate=rng.choice(("softmax", "sigmoid")), renorm=rng.random() < 0.8)
        c["k"] = min(rng.choice((1, 2, 2, 3, 4, 4, 5, 6, 8)), c["E"])
        if op != "router":
            c["ffn"] = rng.choice(("swiglu", "swiglu", "swiglu", "gelu"))
            c["n_shared"] = rng.choice((0, 0, 1, 2, 4))
            c["d_ff_shared"] = _mult(rng.choice((c["d_ff"], c["d_ff"] // 2)), m) if c["n_shared"] else 0
            c["overlap"] = bool(c["n_shared"] and rng.random() < 0.7)
            c["zipf"] = round(rng.uniform(0.0, 1.5), 2)
            c["stress"] = c["E"] - 11 >= c["k"] and rng.random() < 0.15
            c["gather"] = rng.random() < 0.15
            c["aux"] = 0.001 if op == "train" else 0.0
        rows = c["T"] * (c["k"] + c["n_shared"])
        weights = 3 * c["d"] * (c["E"] * c["d_ff"] + c["n_shared"] * c["d_ff_shared"])
        flops = 18 * rows * c["d"] * c["d_ff"]
        if weights <= 5.5e9 and flops <= (4e11 if f32 else 1e13):
            return c


# ---------------------------------------------------------------------------------------- inputs
def _skewed_logits(c, seed, device):
    """Router logits: N(0,1) plus log p_e, p_e Zipf over a random expert order; `stress`: the first expert of the order
    is chosen by 30 % of the tokens, the next ten by none."""
    g = torch.Generator(device=device)
    g.manual_seed(seed * 977 + 5)
    T, E, k = c["T"], c["E"], c["k"]
    z = torch.randn(T, E, generator=g, device=device)
    order = torch.randperm(E, generator=g, device=device)
    first = min(11, E - k) if c["stress"] else 0
    ranks = torch.arange(1, E - first + 1, device=device, dtype=torch.float32)
    z[:, order[first:]] -= c["zipf"] * ranks.log()
    if first:
        z[:, order[:first]] = -1.0e4
        chosen = torch.randperm(T, generator=g, device=device)[: int(round(0.3 * T))]
        z[chosen, order[0]] = 4.0
    return z


def prepare(case, seed):
    c = case
    dev, dt = torch.device("cuda:0"), torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 977 + 6)

    def normal(std, *shape):
        return torch.empty(*shape, dtype=dt, device=dev).normal_(0.0, std, generator=g)

    T, d, E, F, S, Fs = c["T"], c["d"], c["E"], c["d_ff"], c["n_shared"], c["d_ff_shared"]
    shape = moe.MoEShape(T, d, E, c["k"], F, c["dtype"], c["gate"], c["renorm"])
    s = {"case": c, "shape": shape, "X": normal(1.0, T, d)}
    if c["op"] == "router":
        s["Wr"] = normal(1.0 / math.sqrt(d), d, E)
        s["dlogits"] = torch.randn(T, E, generator=g, device=dev) * 0.02
        s["logits"] = torch.empty(T, E, device=dev)
        s["dWr"], s["dX"] = torch.empty_like(s["Wr"]), torch.empty_like(s["X"])
        n = max(moe.moe_router_fwd_workspace_bytes(shape), moe.moe_router_bwd_workspace_bytes(shape))
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=dev)
        return s
    gated = c["ffn"] == "swiglu"
    s["logits"] = _skewed_logits(c, seed, dev)
    s["dY"] = normal(0.02, T, d)
    std = 1.0 / math.sqrt(d)   # pre-activations of order one
    s["w"] = [normal(std, E, d, F), normal(std, E, d, F) if gated else None, normal(std, E, F, d)]
    s["w"] += [normal(std, S, d, Fs), normal(std, S, d, Fs) if gated else None, normal(std, S, Fs, d)] if S else [None] * 3
    s["hp"] = moe.MoEHotPath(shape, S, Fs, dev, overlap_shared=c["overlap"], aux_alpha=c["aux"], gather=c["gather"])
    names = ["dWg_c", "dWd_c"] + (["dWu_c"] if gated else [])
    names += (["dWsg", "dWsd"] + (["dWsu"] if gated else [])) if S else []
    for n in names:   # gradients are written for activated experts only: the other slots are zeros
        s["hp"].b[n].zero_()
    s["grads"] = names
    return s


def run(state):
    c = state["case"]
    if c["op"] == "router":
        sh, X, Wr = state["shape"], state["X"], state["Wr"]
        moe.moe_router_fwd(sh, X, Wr, state["logits"], state["ws"])
        moe.moe_router_bwd(sh, X, Wr, state["dlogits"], state["dWr"], state["dX"], False, state["ws"])
        return {"logits": state["logits"], "dWr": state["dWr"], "dX": state["dX"]}
    hp = state["hp"]
    hp.forward(state["logits"], state["X"], *state["w"])
    names = ["Y", "topk_idx", "topk_w", "counts"]
    if c["op"] == "train":
        hp.backward(state["dY"], state["X"], *state["w"])
        names += ["dX", "dlogits", "active_ids", "n_active"] + state["grads"]
    if c["aux"] > 0:
        names += ["aux_P", "aux_loss"]
    return {n: hp.b[n] for n in names}


# ------------------------------------------------------------------------------ work and tolerance
def work(case):
    """Arithmetic of the products over the rows there are; every input read and every output written once (weights
    and weight gradients of the experts that a drawing of the routing activates)."""
    c = case
    T, d, E, F, S, Fs = c["T"], c["d"], c["E"], c["d_ff"], c["n_shared"], c["d_ff_shared"]
    b = 4 if c["dtype"] == "f32" else 2
    if c["op"] == "router":
        return {"bytes": T * d * b * 2 + 2 * d * E * b + 2 * T * E * 4, "flops": 6.0 * T * d * E}
    mats = 3 if c["ffn"] == "swiglu" else 2
    chosen = torch.topk(_skewed_logits(c, 1, "cpu"), c["k"], dim=1).indices
    weights = mats * d * (int(torch.unique(chosen).numel()) * F + S * Fs) * b
    macs = mats * d * (T * c["k"] * F + S * T * Fs)
    if c["op"] == "forward":
        return {"bytes": weights + 2 * T * d * b + T * E * 4, "flops": 2.0 * macs}
    return {"bytes": 2 * weights + 4 * T * d * b + 2 * T * E * 4, "flops": 6.0 * macs}


def tolerance(case):
    """Against a 64-bit evaluation of the same layers the outputs are off by at most 3.8e-3 of their norm in bf16 and
    1.6e-6 in fp32 (K up to 2816; the sums of the drawn cases are up to 7168 long)."""
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}

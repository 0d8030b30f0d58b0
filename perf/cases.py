"""Timed cases of the condensed MoE layer, through the package's public entry points.

Three kinds of work that a program has this package do:

  layer   MoELayer(x): route, condense, expert FFN on the representatives and
          combine, i.e. the forward of one condensed MoE layer (inference and
          the forward half of training)
  train   MoELayer(x), luffy_combine_backward and luffy_expert_ffn_backward: one
          layer's training step
  stack   MoEStack(xs): consecutive blocks over the same tokens, each
          condensing with the historical similarity of the block before it

Tokens are clustered (a centre and noise around it; `centres` = 0 draws them
i.i.d.), which is how this layer's inputs look in earnest, and the router's
bias gives the experts a Zipf load where `zipf` is set.  All inputs are drawn
on the GPU from the seed.  Same-centre cosines lie above 0.99 and others near
0, far from every threshold used here, so indices are the same for every
correct implementation.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2411_15419_amd as luffy

# Sizes of the layers below: `dtype` of activations and weights, T tokens of
# width d, E experts, top-k routing, hidden width d_ff, activation, capacity
# factor cf (0: no limit), threshold h, number of centres and noise sigma,
# Zipf exponent of the expert load (0: no bias).
_LISTED = [
    # the smallest float32 layer of this repository: 512 tokens, where launches and latency count
    dict(name="f32_small", kind="layer", dtype="f32", T=512, d=256, E=4, k=1, d_ff=1024, act="gelu", cf=0.0,
         h=0.95, centres=64, sigma=0.05, zipf=0.0),
    # an ordinary float32 layer with an odd token count, top-2, SiLU and a capacity limit
    dict(name="f32_odd", kind="layer", dtype="f32", T=3001, d=512, E=8, k=2, d_ff=2048, act="silu", cf=1.25,
         h=0.9, centres=700, sigma=0.03, zipf=0.0),
    # a serving step of a few tokens on the ordinary bf16 layer: every expert's weights for a handful of rows
    dict(name="few_tokens", kind="layer", dtype="bf16", T=61, d=1024, E=16, k=2, d_ff=4096, act="gelu", cf=0.0,
         h=0.95, centres=24, sigma=0.03, zipf=0.0),
    # the ordinary bf16 layer: 8 x 1024 tokens, top-2, capacity factor 1.25 with drops
    dict(name="ordinary", kind="layer", dtype="bf16", T=8192, d=1024, E=16, k=2, d_ff=4096, act="gelu", cf=1.25,
         h=0.95, centres=2048, sigma=0.03, zipf=0.0),
    # odd sizes throughout: prime token count, widths that are multiples of 64 only, 12 experts
    dict(name="ragged", kind="layer", dtype="bf16", T=5003, d=1088, E=12, k=2, d_ff=2880, act="silu", cf=1.1,
         h=0.9, centres=1500, sigma=0.04, zipf=0.7),
    # one GPU's share of an expert-parallel layer: 16 x 2048 tokens, Zipf(1.1) load, no capacity limit
    dict(name="expert_share", kind="layer", dtype="bf16", T=32768, d=2048, E=32, k=2, d_ff=8192, act="gelu", cf=0.0,
         h=0.9, centres=4096, sigma=0.02, zipf=1.1),
    # condensation's worst case: i.i.d. tokens, nothing merges, so every token goes through its expert
    dict(name="no_merge", kind="layer", dtype="bf16", T=16384, d=4096, E=8, k=1, d_ff=11008, act="silu", cf=0.0,
         h=0.9, centres=0, sigma=1.0, zipf=0.0),
    # many experts, skewed load, capacity factor 1.0 with drops: 32 x 2048 tokens
    dict(name="many_experts", kind="layer", dtype="bf16", T=65536, d=1024, E=64, k=1, d_ff=4096, act="gelu", cf=1.0,
         h=0.95, centres=8192, sigma=0.05, zipf=1.3),
    # a training step of the ordinary layer, float32 weight gradients
    dict(name="train_ordinary", kind="train", dtype="bf16", T=8192, d=1024, E=16, k=2, d_ff=4096, act="gelu",
         cf=1.25, h=0.95, centres=2048, sigma=0.03, zipf=0.0, dw="f32"),
    # a training step at large width, bf16 weight gradients, at a threshold as the adaptive schedule gives it
    # while the loss falls (between 1/(1+e) and 1/2)
    dict(name="train_wide", kind="train", dtype="bf16", T=16384, d=2048, E=16, k=2, d_ff=8192, act="gelu", cf=0.0,
         h=0.45, centres=2048, sigma=0.02, zipf=1.1, dw="bf16"),
    # two blocks of the expert-parallel share with the historical similarity; one token in twenty is a mixture
    # of two centres, and the router stays the same between the blocks
    dict(name="stack_share", kind="stack", dtype="bf16", T=32768, d=2048, E=32, k=2, d_ff=8192, act="gelu", cf=0.0,
         h=0.9, centres=4096, sigma=0.02, zipf=1.1, blocks=2, mix=0.05, drift=0.0, S1=0.8, S2=0.2),
    # three ordinary blocks with a router that drifts from block to block, at an adaptive threshold
    dict(name="stack_drift", kind="stack", dtype="bf16", T=8192, d=1024, E=16, k=2, d_ff=4096, act="gelu", cf=1.25,
         h=0.45, centres=2048, sigma=0.03, zipf=0.0, blocks=3, mix=0.05, drift=0.3, S1=0.8, S2=0.2),
]


def listed():
    return [dict(c) for c in _LISTED]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(v, m):
    return max(m, int(round(v / m)) * m)


def draw(rng):
    """A case of the same ranges: sizes over the logarithm of their range,
    token counts of any parity, widths any multiple of 64."""
    kind = rng.choice(["layer", "layer", "layer", "layer", "train", "stack"])
    f32 = kind == "layer" and rng.random() < 0.3
    c = dict(kind=kind, dtype="f32" if f32 else "bf16")
    c["k"] = rng.choice([1, 2])
    c["E"] = rng.choice([4, 6, 8, 12, 16, 24, 32, 48, 64] if not f32 else [4, 6, 8, 16])
    c["d"] = _multiple(_log_uniform(rng, 256, 1024 if f32 else 4096), 64)
    c["d_ff"] = _multiple(min(c["d"] * rng.uniform(2.0, 4.0), 11008), 64)
    lo, hi = (128, 4096) if f32 else ((48, 65536) if kind == "layer" else (2048, 32768))
    c["T"] = int(_log_uniform(rng, lo, hi))
    c["act"] = rng.choice(["gelu", "silu"])
    c["cf"] = rng.choice([0.0, 1.0, 1.1, 1.25, 2.0])
    c["h"] = rng.choice([0.45, 0.8, 0.9, 0.95])
    iid = kind == "layer" and rng.random() < 0.15
    c["centres"] = 0 if iid else max(4, int(c["T"] / _log_uniform(rng, 2.0, 12.0)))
    c["sigma"] = 1.0 if iid else rng.choice([0.02, 0.03, 0.04, 0.05])
    c["zipf"] = rng.choice([0.0, 0.7, 1.1, 1.3])
    if kind == "train":
        c["dw"] = rng.choice(["f32", "bf16"])
    if kind == "stack":
        c.update(blocks=rng.choice([2, 3]), mix=0.05, drift=rng.choice([0.0, 0.3]), S1=0.8, S2=0.2)
    # no dearer than the largest listed case of its kind: weights first, then
    # tokens (pairs of tokens cost the square of a bucket)
    while 2 * c["E"] * c["d"] * c["d_ff"] * (c.get("blocks", 1)) > (2 ** 31 if kind == "stack" else 2 ** 30):
        c["E"] = max(4, c["E"] // 2)
        if c["E"] == 4:
            c["d_ff"] = _multiple(c["d_ff"] / 2, 64)
    pair_cap = 2.0e12 if kind != "stack" else 1.0e12
    ffn_cap = {"layer": 2.5e12 if not f32 else 4.0e10, "train": 6.0e11, "stack": 6.0e11}[kind]
    while True:
        pairs = _pair_work(c)
        rows, _ = _rows(c)
        if pairs <= pair_cap and 4.0 * rows * c["d"] * c["d_ff"] <= ffn_cap:
            break
        c["T"] = c["T"] * 2 // 3
        if not iid:
            c["centres"] = max(4, c["centres"] * 2 // 3)
    return c


# ------------------------------------------------------------------ inputs
_W_SCALE = 0.02


def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _zipf_share(E, s):
    p = np.arange(1, E + 1, dtype=np.float64) ** (-s)
    return p / p.sum()


@functools.lru_cache(maxsize=64)
def _router_bias(E, k, s, logit_std):
    """Bias under which the top-k load of experts with independent N(0,
    logit_std^2) token logits follows Zipf(s): a fixed point on sampled
    logits, a function of the sizes alone."""
    if s <= 0.0:
        return np.zeros(E, np.float32)
    p = _zipf_share(E, s)
    z = np.random.default_rng(1).standard_normal((8192, E)) * logit_std
    b = np.log(p) * logit_std
    for _ in range(60):
        L = z + b
        if k == 1:
            cnt = np.bincount(L.argmax(1), minlength=E)
        else:
            cnt = np.bincount(np.argpartition(-L, k - 1, axis=1)[:, :k].reshape(-1), minlength=E)
        share = np.maximum(cnt, 0.25) / (8192.0 * k)
        b += 0.5 * logit_std * (np.log(p) - np.log(share))
        b -= b.mean()
    return b.astype(np.float32)


def _normal(gen, shape, scale, dtype):
    t = torch.randn(shape, generator=gen, dtype=torch.float32 if dtype == torch.float32 else torch.bfloat16,
                    device="cuda")
    return t.mul_(scale) if scale != 1.0 else t


def _inputs(case, seed):
    """Per block (one for a layer): x, w_gate, b_gate, w1, w2; and dy for a
    training step."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)
    dt = _torch_dtype(case)
    T, d, E, d_ff = case["T"], case["d"], case["E"], case["d_ff"]
    n_c, sigma = case["centres"], case["sigma"]
    if n_c > 0:
        centres = torch.randn((n_c, d), generator=gen, device="cuda")
        base = centres[torch.randint(0, n_c, (T,), generator=gen, device="cuda")]
        if case.get("mix", 0.0) > 0.0:
            other = centres[torch.randint(0, n_c, (T,), generator=gen, device="cuda")]
            mixed = torch.rand((T, 1), generator=gen, device="cuda") < case["mix"]
            base = torch.where(mixed, (base + other) * math.sqrt(0.5), base)
        std = _W_SCALE * math.sqrt(d * (1.0 + sigma * sigma))
    else:
        base = torch.zeros((T, d), device="cuda")
        std = _W_SCALE * math.sqrt(d)
    bias = torch.from_numpy(_router_bias(E, case["k"], case["zipf"], round(std, 6))).cuda()
    w_gate = _normal(gen, (E, d), _W_SCALE, torch.float32)
    blocks = []
    x = base
    for b in range(case.get("blocks", 1)):
        x = x + sigma * torch.randn((T, d), generator=gen, device="cuda")
        if b > 0 and case["drift"] > 0.0:
            w_gate = w_gate + case["drift"] * _normal(gen, (E, d), _W_SCALE, torch.float32)
        blocks.append(dict(x=x.to(dt), w_gate=w_gate.to(dt), b_gate=bias,
                           w1=_normal(gen, (E, d_ff, d), 0.02, dt), w2=_normal(gen, (E, d, d_ff), 0.02, dt)))
    dy = _normal(gen, (T, d), 1.0, dt) if case["kind"] == "train" else None
    return blocks, dy


def prepare(case, seed):
    """The layer (or stack) with its weights and buffers, and its inputs."""
    blocks, dy = _inputs(case, seed)
    history = (case["S1"], case["S2"]) if case["kind"] == "stack" else None
    layers = [luffy.MoELayer(b["w_gate"], b["b_gate"], b["w1"], b["w2"], k=case["k"], act=case["act"],
                             threshold=case["h"], capacity_factor=case["cf"], T=case["T"], history=history)
              for b in blocks]
    xs = [b["x"] for b in blocks]
    if case["kind"] == "stack":
        return dict(kind="stack", stack=luffy.MoEStack(layers), xs=xs)
    state = dict(kind=case["kind"], layer=layers[0], x=xs[0])
    if case["kind"] == "train":
        # the backward's buffers, as MoELayer.backward keeps them; rows of
        # dx_rep past the representatives in use are never written and stay 0
        T, k, d, E, d_ff = case["T"], case["k"], case["d"], case["E"], case["d_ff"]
        S, dt = T * k, torch.bfloat16
        dw = torch.float32 if case["dw"] == "f32" else torch.bfloat16
        ws_c = luffy.combine_backward_workspace_size(T, k, S)
        ws_f = luffy.expert_ffn_backward_workspace_size(S, E, d, d_ff, luffy.LUFFY_BF16)
        state.update(dy=dy, dgate=torch.empty(T, k, device="cuda"),
                     dy_rep=torch.empty(S, d, dtype=dt, device="cuda"),
                     dx_rep=torch.zeros(S, d, dtype=dt, device="cuda"),
                     dw1=torch.empty(E, d_ff, d, dtype=dw, device="cuda"),
                     dw2=torch.empty(E, d, d_ff, dtype=dw, device="cuda"),
                     ws_c=torch.empty(ws_c, dtype=torch.uint8, device="cuda"),
                     ws_f=torch.empty(ws_f, dtype=torch.uint8, device="cuda"))
    return state


def _block_outputs(layer, y):
    b = layer.buf
    return dict(y=y, gate=b.topk_gate, expert=b.topk_idx, offsets=b.offsets, rep_offsets=b.rep_offsets)


def run(state):
    if state["kind"] == "stack":
        ys = state["stack"](state["xs"])
        return [_block_outputs(layer, y) for layer, y in zip(state["stack"].layers, ys)]
    layer, x = state["layer"], state["x"]
    out = _block_outputs(layer, layer(x))
    if state["kind"] == "train":
        s, b = state, layer.buf
        luffy.luffy_combine_backward(s["dy"], b.y_rep, b.rep_row, b.perm_token, b.slot_pos, b.topk_gate, b.offsets,
                                     b.rep_offsets, s["dy_rep"], s["dgate"], s["ws_c"])
        luffy.luffy_expert_ffn_backward(x, b.rep_token, b.rep_offsets, layer.w1, layer.w2, layer.act,
                                        b.y_rep.shape[0], s["dy_rep"], s["dx_rep"], s["dw1"], s["dw2"], s["ws_f"])
        out.update(dgate=s["dgate"], dx_rep=s["dx_rep"], dw1=s["dw1"], dw2=s["dw2"])
    return out


# -------------------------------------------------------------------- work
def _load(case):
    """Expected kept slots of every expert."""
    T, E, k = case["T"], case["E"], case["k"]
    n = T * k * (_zipf_share(E, case["zipf"]) if case["zipf"] > 0 else np.full(E, 1.0 / E))
    n = np.minimum(n, T)
    C = _capacity(case)
    return np.minimum(n, C) if C else n


def _capacity(case):
    if case["cf"] <= 0:
        return 0
    return math.ceil(case["cf"] * case["k"] * case["T"] / case["E"] - 1e-9)


def _rows(case):
    """Expected representatives, and kept slots: the tokens of a centre share
    their experts, so they condense to one row in each."""
    kept = float(_load(case).sum())
    if case["centres"] <= 0:
        return kept, kept
    T, n_c = case["T"], case["centres"]
    distinct = n_c * -math.expm1(T * math.log1p(-1.0 / n_c))
    return min(kept, max(1.0, kept * distinct / T)), kept


def _pair_work(case):
    return float((_load(case) ** 2).sum()) * case["d"]


def work(case):
    """Bytes: tokens and weights (of the experts with rows) read once, the
    outputs written once.  Flops: the gate and the expert products on the
    representatives.  Neither counts the pairs of a bucket: which pairs are
    similar can be decided without every pair's full product."""
    b = 4 if case["dtype"] == "f32" else 2
    T, d, E, k, d_ff = case["T"], case["d"], case["E"], case["k"], case["d_ff"]
    rows, _ = _rows(case)
    used = min(E, rows)
    weights = 2.0 * used * d * d_ff * b + E * d * b
    nbytes = 2.0 * T * d * b + weights + 8.0 * T * k
    flops = 2.0 * T * d * E + 4.0 * rows * d * d_ff
    if case["kind"] == "train":
        # dy read, the weights read again, both weight gradients and dx written
        nbytes += T * d * b + 2.0 * E * d * d_ff * (4 if case["dw"] == "f32" else 2) + rows * d * b
        flops += 8.0 * rows * d * d_ff + 4.0 * T * k * d
    n = case.get("blocks", 1)
    return {"bytes": nbytes * n, "flops": flops * n}


def tolerance(case):
    """float32: sums of a few thousand products in another order (up to 1.1e-6
    measured against 64 bits).  bf16: the hidden rows, the expert outputs and the results are rounded to 8 bits
    each (and the backward's dZ and dY rows once more), so a result is about
    0.3% off its 64-bit value whichever order the sums take."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": 1.2e-2}


# ------------------------------------------------------------------- exact
def _act(z, act):
    if act == "gelu":
        return 0.5 * z * (1.0 + torch.erf(z * math.sqrt(0.5)))
    return z * torch.sigmoid(z)


def _act_grad(z, act):
    if act == "gelu":
        return 0.5 * (1.0 + torch.erf(z * math.sqrt(0.5))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
    s = torch.sigmoid(z)
    return s * (1.0 + z * (1.0 - s))


def _exact_route(case, blk):
    """Experts and gates of every token, kept slots bucket by bucket."""
    T, E, k = case["T"], case["E"], case["k"]
    logits = blk["x"].double() @ blk["w_gate"].double().t() + blk["b_gate"].double()
    top, idx = logits.topk(k, dim=1)
    gate = torch.softmax(logits, dim=1).gather(1, idx) if k == 1 else torch.softmax(top, dim=1)
    slot_e = idx.t().reshape(-1)                       # slot j * T + t
    order = torch.sort(slot_e, stable=True).indices
    counts = torch.bincount(slot_e, minlength=E).tolist()
    C = _capacity(case)
    buckets, at = [], 0
    for e in range(E):
        s = order[at:at + counts[e]]
        at += counts[e]
        buckets.append(s[:C] if C else s)
    return gate, buckets


def _greedy(adj):
    """Representative (position) of every position of one bucket: highest
    degree first, lower position on ties."""
    n = adj.shape[0]
    pos = torch.arange(n, device=adj.device)
    key = adj.sum(1) * (n + 1) + (n - pos)
    state = torch.zeros(n, dtype=torch.int8, device=adj.device)   # 0 undecided, 1 kept, 2 absorbed
    while bool((state == 0).any()):
        und = state == 0
        rows = und.nonzero().squeeze(1)
        best = torch.empty(rows.numel(), dtype=torch.int64, device=adj.device)
        kmask = torch.where(und, key, torch.zeros_like(key))
        for a in range(0, rows.numel(), 4096):
            r = rows[a:a + 4096]
            best[a:a + 4096] = torch.where(adj[r], kmask[None, :], torch.zeros_like(kmask)[None, :]).amax(1)
        keep = rows[best < key[rows]]
        state[keep] = 1
        hit = torch.zeros(n, dtype=torch.bool, device=adj.device)
        for a in range(0, keep.numel(), 4096):
            hit |= adj[keep[a:a + 4096]].any(0)
        state[hit & (state == 0)] = 2
    rep = pos.clone()
    kkey = torch.where(state == 1, key, torch.zeros_like(key))
    gone = (state == 2).nonzero().squeeze(1)
    for a in range(0, gone.numel(), 4096):
        r = gone[a:a + 4096]
        rep[r] = torch.where(adj[r], kkey[None, :], torch.zeros_like(kkey)[None, :]).argmax(1)
    return rep


def _exact_condense(case, blk, buckets, previous):
    """Per bucket the representative of every position; with a history also
    this block's classes (tokens, weight > S1, weight < S2) per bucket."""
    T = case["T"]
    stack = case["kind"] == "stack"
    xn = blk["x"].double()
    xn = xn / xn.norm(dim=1, keepdim=True)
    reps, record = [], []
    for slots in buckets:
        tok = slots % T
        n = tok.numel()
        if n == 0:
            reps.append(tok)
            record.append((tok, None, None))
            continue
        u = xn[tok]
        w = u @ u.t()
        if previous is not None:
            one = torch.zeros((n, n), dtype=torch.bool, device=w.device)
            zero = torch.zeros_like(one)
            for ptok, phi, plo in previous:
                if ptok.numel() == 0:
                    continue
                where = torch.full((T,), -1, dtype=torch.int64, device=w.device)
                where[ptok] = torch.arange(ptok.numel(), device=w.device)
                q = where[tok]
                here = (q >= 0).nonzero().squeeze(1)
                if here.numel() == 0:
                    continue
                q = q[here]
                one[here[:, None], here[None, :]] |= phi[q[:, None], q[None, :]]
                zero[here[:, None], here[None, :]] |= plo[q[:, None], q[None, :]]
            w = torch.where(one, torch.ones_like(w), torch.where(zero, torch.zeros_like(w), w))
        if stack:
            record.append((tok, w > case["S1"], w < case["S2"]))
        adj = w >= case["h"]
        del w
        adj.fill_diagonal_(False)
        reps.append(_greedy(adj))
    return reps, (record if stack else None)


def _exact_block(case, blk, dy, previous):
    T, k, d = case["T"], case["k"], case["d"]
    gate, buckets = _exact_route(case, blk)
    reps, record = _exact_condense(case, blk, buckets, previous)
    x = blk["x"]
    y = torch.zeros((T, d), dtype=torch.float64, device="cuda")
    train = dy is not None
    if train:
        dyd = dy.double()
        dgate = torch.zeros((T, k), dtype=torch.float64, device="cuda")
        dx, dw1, dw2 = [], torch.zeros(blk["w1"].shape, dtype=torch.float64, device="cuda"), \
            torch.zeros(blk["w2"].shape, dtype=torch.float64, device="cuda")
    for e, slots in enumerate(buckets):
        n = slots.numel()
        if n == 0:
            continue
        tok, ch, rep = slots % T, slots // T, reps[e]
        kept = (rep == torch.arange(n, device="cuda")).nonzero().squeeze(1)
        row = torch.zeros(n, dtype=torch.int64, device="cuda")
        row[kept] = torch.arange(kept.numel(), device="cuda")
        row = row[rep]
        xe = x[tok[kept]].double()
        w1, w2 = blk["w1"][e].double(), blk["w2"][e].double()
        z = xe @ w1.t()
        a = _act(z, case["act"])
        out = a @ w2.t()
        g = gate[tok, ch]
        y.index_add_(0, tok, out[row] * g[:, None])
        if train:
            dgate[tok, ch] = (dyd[tok] * out[row]).sum(1)
            dout = torch.zeros_like(out)
            dout.index_add_(0, row, dyd[tok] * g[:, None])
            dz = (dout @ w2) * _act_grad(z, case["act"])
            dx.append(dz @ w1)
            dw1[e] = dz.t() @ xe
            dw2[e] = dout.t() @ a
    out = dict(y=y, gate=gate, expert=None, offsets=None, rep_offsets=None)
    if train:
        dx_rep = torch.zeros((T * k, d), dtype=torch.float64, device="cuda")
        rows = torch.cat(dx)
        dx_rep[:rows.shape[0]] = rows
        out.update(dgate=dgate, dx_rep=dx_rep, dw1=dw1, dw2=dw2)
    return out, record


def exact(case, seed):
    """run()'s floating outputs in 64 bits, in plain torch."""
    blocks, dy = _inputs(case, seed)
    outs, record = [], None
    for blk in blocks:
        out, record = _exact_block(case, blk, dy, record)
        outs.append(out)
    return outs if case["kind"] == "stack" else outs[0]

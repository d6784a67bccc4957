"""The workloads this library is measured on: whole drains of expert layers
through the Python surface, from one decode step of a tiny layer to a
multi-layer drain.

A case is a dict of plain values.  ``kind`` says which calls a pass makes:

* ``layer``: fragments arrive and are routed into one layer's queues, the layer
  is drained (re-batch, expert FFN, combine).  Output: the layer's output rows.
* ``rows``: one GPU's share of an expert-parallel layer.  Rows routed elsewhere
  arrive grouped by expert, are re-batched and run through the experts; the
  rows of y go back to their owners.  Output: y, in expert order.
* ``pool``: a layer drained one expert at a time, the top-k rows of a token
  merged in the token pool.  Output: the released tokens' rows.
* ``drain``: several layers hold queued tokens and the layer with the most
  rows is drained next until every queue is empty.  Output: every layer's rows.

Activations are N(0, 1), weights 0.02 N(0, 1), gate logits N(0, 1) plus the
bias that makes expert popularity Zipf(s), experts in a seeded order.
"""

from __future__ import annotations

import math

import torch

import paper_2505_08944_amd as aep

TINY = dict(d=256, f=512, E=8, S=0, k=2, zipf=1.0, act="f32", wdt="f32", renorm=True)
MIXTRAL = dict(d=4096, f=14336, E=8, S=0, k=2, zipf=1.2, act="bf16", wdt="bf16", renorm=True)
FINE = dict(d=2048, f=1408, E=64, S=2, k=6, zipf=1.1, act="bf16", wdt="bf16", renorm=True)
SHARE = dict(d=4096, f=2048, E=16, S=0, k=1, zipf=1.3, act="bf16", wdt="bf16", renorm=True)


def listed():
    return [
        # the smallest call: a tiny f32 layer, all latency and launches
        dict(TINY, name="tiny_f32_256", kind="layer", T=256, frag=1),
        # one decode step of a Mixtral-style layer: four attention ranks send
        # eight tokens each; every expert's weights are streamed for a few rows
        dict(MIXTRAL, name="mixtral_decode_32", kind="layer", T=32, frag=4),
        # an ordinary ragged batch: mixed prefill and decode, odd fragments
        dict(MIXTRAL, name="mixtral_777", kind="layer", T=777, frag=3),
        # a full prefill batch (the benchmark's workload)
        dict(MIXTRAL, name="mixtral_4096", kind="layer", T=4096, frag=4),
        # one decode step of a fine-grained layer: 64 experts, two shared ones
        dict(FINE, name="fine_decode_64", kind="layer", T=64, frag=4),
        # ragged batch of a fine-grained layer, weights not renormalised
        dict(FINE, name="fine_1999", kind="layer", T=1999, frag=3, renorm=False),
        # a full prefill batch of the fine-grained layer
        dict(FINE, name="fine_8192", kind="layer", T=8192, frag=4),
        # one GPU's 16 of 128 experts, queue depths 4096 ... 111
        dict(SHARE, name="share_4096", kind="rows", depth=4096),
        # the same with fp8 weights
        dict(SHARE, name="share_fp8_4096", kind="rows", depth=4096, wdt="fp8"),
        # the same share in decode: 200 ... 38 rows per expert, fp8 weights
        dict(SHARE, name="share_fp8_cold_200", kind="rows", depth=200, zipf=0.6, wdt="fp8"),
        # experts scheduled one by one, merged through the token pool
        dict(MIXTRAL, name="pool_1024", kind="pool", T=1024, frag=2),
        # asynchronous drain of four Mixtral-style layers, most tokens first
        dict(MIXTRAL, name="drain_4_layers", kind="drain", tokens="2048,512,3072,1024", frag=4),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny", "mixtral", "mixtral", "fine", "fine", "share", "share", "pool", "drain"])
    if kind == "tiny":
        E = rng.choice([4, 8, 13, 16])
        return dict(TINY, kind="layer", T=_log(rng, 1, 1024), frag=rng.randint(1, 3), d=64 * rng.randint(2, 8),
                    f=64 * rng.randint(2, 16), E=E, k=rng.randint(1, 4), renorm=rng.random() < 0.7)
    if kind == "mixtral":
        return dict(MIXTRAL, kind="layer", T=_log(rng, 1, 4096), frag=rng.randint(1, 4), d=64 * rng.randint(32, 64),
                    f=64 * rng.randint(64, 224), k=rng.randint(1, 2), wdt=rng.choice(["bf16", "bf16", "fp8"]))
    if kind == "fine":
        return dict(FINE, kind="layer", T=_log(rng, 1, 8192), frag=rng.randint(1, 4), d=64 * rng.randint(16, 40),
                    f=64 * rng.randint(12, 28), E=rng.choice([32, 48, 60, 64]), S=rng.randint(0, 2),
                    k=rng.randint(4, 8), renorm=rng.random() < 0.5)
    if kind == "share":
        return dict(SHARE, kind="rows", depth=_log(rng, 8, 4096), zipf=rng.choice([0.3, 0.6, 1.0, 1.3]),
                    d=64 * rng.randint(32, 64), f=64 * rng.randint(16, 44), E=rng.randint(8, 24),
                    wdt=rng.choice(["bf16", "fp8"]))
    if kind == "pool":
        return dict(MIXTRAL, kind="pool", T=_log(rng, 8, 1024), frag=rng.randint(1, 3), d=64 * rng.randint(32, 64),
                    f=64 * rng.randint(64, 224))
    tokens = [_log(rng, 1, 2048) for _ in range(rng.randint(2, 4))]
    return dict(MIXTRAL, kind="drain", tokens=",".join(map(str, tokens)), frag=rng.randint(1, 4),
                d=64 * rng.randint(32, 64), f=64 * rng.randint(64, 224))


# ------------------------------------------------------------------ inputs
def _layer_tokens(c):
    if c["kind"] == "drain":
        return [int(t) for t in c["tokens"].split(",")]
    return [c["T"]]


def _depths(c):
    """Queue depths of a ``rows`` case by popularity rank."""
    return [max(1, int(c["depth"] * r ** -c["zipf"])) for r in range(1, c["E"] + 1)]


def _sizes(T, frag):
    frag = max(1, min(frag, T))
    return [T // frag + (1 if i < T % frag else 0) for i in range(frag)]


def _weights(c, gen):
    """Per expert (gate, up, down, scale_gate_up, scale_down)."""
    def mat(rows, cols):
        w = torch.randn(rows, cols, device="cuda", generator=gen,
                        dtype=torch.float32 if c["act"] == "f32" else torch.bfloat16)
        return w.mul_(0.02)

    def quant(w):
        s = (w.float().abs().amax(1) / 448.0).to(torch.bfloat16)
        q = (w.float() / s.float()[:, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
        return q.view(torch.uint8), s

    out = []
    for _ in range(c["E"] + c["S"]):
        g, u, dn = mat(c["f"], c["d"]), mat(c["f"], c["d"]), mat(c["d"], c["f"])
        if c["wdt"] != "fp8":
            out.append((g, u, dn, None, None))
            continue
        (qg, sg), (qu, su), (qd, sd) = quant(g), quant(u), quant(dn)
        out.append((qg, qu, qd, torch.cat([sg, su]), sd))
    return out


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    act = torch.float32 if c["act"] == "f32" else torch.bfloat16
    layers = []
    if c["kind"] == "rows":
        perm = torch.randperm(c["E"], device="cuda", generator=gen).tolist()
        by_rank = _depths(c)
        counts = [by_rank[perm[e]] for e in range(c["E"])]
        n = sum(counts)
        layers.append({"counts": counts, "x": torch.randn(n, c["d"], device="cuda", generator=gen, dtype=act),
                       "tok": torch.randperm(n, device="cuda", generator=gen).to(torch.int32),
                       "gate_w": torch.rand(n, device="cuda", generator=gen), "w": _weights(c, gen)})
        return layers
    for T in _layer_tokens(c):
        rank = torch.randperm(c["E"], device="cuda", generator=gen).float() + 1.0
        bias = -c["zipf"] * torch.log(rank)
        frags = [(torch.randn(t, c["d"], device="cuda", generator=gen, dtype=act),
                  torch.randn(t, c["E"], device="cuda", generator=gen) + bias) for t in _sizes(T, c["frag"])]
        layers.append({"frags": frags, "w": _weights(c, gen)})
    return layers


def prepare(case, seed):
    c = case
    layers = _inputs(c, seed)
    cap = sum(layers[0]["counts"]) if c["kind"] == "rows" else max(_layer_tokens(c))
    ctx = aep.Context(len(layers), c["E"], c["d"], c["f"], c["k"], n_shared=c["S"], renorm=c["renorm"], act=c["act"],
                      wdt=c["wdt"], max_tokens_per_layer=cap, token_pool=c["kind"] == "pool")
    for l, layer in enumerate(layers):
        for e, w in enumerate(layer["w"]):
            ctx.set_expert_weights(l, e, *w)
    st = {"case": c, "ctx": ctx, "layers": layers, "cap": cap}
    if c["kind"] == "pool":
        ids, t0 = [], 0
        for x, _ in layers[0]["frags"]:
            ids.append(torch.arange(t0, t0 + x.shape[0], device="cuda", dtype=torch.int32))
            t0 += x.shape[0]
        st["ids"] = ids
        st["out"] = torch.empty(cap, c["d"], device="cuda", dtype=layers[0]["frags"][0][0].dtype)
        st["ready"] = torch.empty(cap, device="cuda", dtype=torch.int32)
    return st


def run(state):
    c, ctx, layers = state["case"], state["ctx"], state["layers"]
    if c["kind"] == "layer":
        for x, logits in layers[0]["frags"]:
            ctx.route_enqueue(0, x, logits)
        return ctx.run_layer(0)
    if c["kind"] == "rows":
        r = layers[0]
        ctx.enqueue_rows_grouped(0, r["counts"], r["x"], r["tok"], r["gate_w"], state["cap"])
        b = ctx.rebatch(0)
        y = ctx.expert_ffn(b)
        ctx.release(b)
        return y
    if c["kind"] == "pool":
        for (x, logits), ids in zip(layers[0]["frags"], state["ids"]):
            ctx.route_enqueue_ids(0, x, logits, ids)
        for e in range(c["E"]):
            b = ctx.rebatch_expert(0, e)
            ctx.pool_accumulate(b, ctx.expert_ffn(b))
            ctx.release(b)
        ctx.pool_release(0, state["out"], state["ready"])
        return [state["out"], state["ready"]]
    for l, layer in enumerate(layers):
        for x, logits in layer["frags"]:
            ctx.route_enqueue(l, x, logits)
    outs = [None] * len(layers)
    while (l := ctx.pick_layer("mtfs")) is not None:
        outs[l] = ctx.run_layer(l)
    return outs


# ---------------------------------------------------------------- reference
def work(case):
    c = case
    asz = 4 if c["act"] == "f32" else 2
    wsz = {"f32": 4, "bf16": 2, "fp8": 1}[c["wdt"]]
    per_expert = 3 * c["d"] * c["f"] * wsz + ((2 * c["f"] + c["d"]) * 2 if c["wdt"] == "fp8" else 0)
    if c["kind"] == "rows":
        n = sum(_depths(c))
        return {"bytes": 2 * n * c["d"] * asz + 8 * n + c["E"] * per_expert, "flops": 6 * c["d"] * c["f"] * n}
    z = [r ** -c["zipf"] for r in range(1, c["E"] + 1)]
    nbytes = flops = 0
    for T in _layer_tokens(c):
        # experts that are expected to receive a row
        hit = sum(1.0 - (1.0 - v / sum(z)) ** (T * c["k"]) for v in z) + c["S"]
        nbytes += 2 * T * c["d"] * asz + 4 * T * c["E"] + int(hit * per_expert)
        flops += 6 * c["d"] * c["f"] * T * (c["k"] + c["S"])
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["act"] == "f32":
        return {"rel": 2.4e-6, "max": 2.4e-5}
    # h, y and the output are each rounded to bf16 once, sums are f32
    return {"rel": 1.2e-2, "max": 6e-2}


def _expert(c, w, x):
    """y = W_down (silu(W_gate x) * (W_up x)) in 64 bits."""
    def mat(q, s=None):
        if c["wdt"] != "fp8":
            return q.double()
        return q.view(torch.float8_e4m3fn).float().double() * s.double()[:, None]

    f = c["f"]
    sg, su = (w[3][:f], w[3][f:]) if c["wdt"] == "fp8" else (None, None)
    h = torch.nn.functional.silu(x @ mat(w[0], sg).T) * (x @ mat(w[1], su).T)
    return h @ mat(w[2], w[4]).T


def _exact_layer(c, layer):
    x = torch.cat([a for a, _ in layer["frags"]]).double()
    logits = torch.cat([b for _, b in layer["frags"]]).double()
    idx = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :c["k"]]
    p = torch.softmax(logits, 1).gather(1, idx)
    if c["renorm"]:
        p = p / p.sum(1, keepdim=True)
    out = torch.zeros_like(x)
    for e in range(c["E"]):
        t, j = (idx == e).nonzero(as_tuple=True)
        if t.numel():
            out[t] += p[t, j][:, None] * _expert(c, layer["w"][e], x[t])
    for s in range(c["S"]):
        out += _expert(c, layer["w"][c["E"] + s], x)
    return out


def exact(case, seed):
    c = case
    layers = _inputs(c, seed)
    if c["kind"] == "rows":
        r = layers[0]
        return torch.cat([_expert(c, w, x.double()) for w, x in zip(r["w"], torch.split(r["x"], r["counts"])) if x.numel()])
    outs = [_exact_layer(c, layer) for layer in layers]
    if c["kind"] == "layer":
        return outs[0]
    if c["kind"] == "pool":
        return [outs[0], torch.ones(c["T"], device="cuda", dtype=torch.int32)]
    return outs

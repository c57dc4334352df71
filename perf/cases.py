"""The calls whose speed this framework is judged by, with their inputs.

A program that serves a mixture-of-experts model on one GPU calls the
down-projection + combine stage (``combine``, ``combine_noalloc``), the
up-projection (``gemm1_swiglu``) and the whole post-router layer
(``layer_forward``).  It calls them for one token while it decodes for one
user, for tens to hundreds of tokens in batched decoding, for a few hundred
to a few thousand in chunked prefill and for ten thousand and more in a whole
prefill batch.  The cases below spread over that range.  The shapes are this
repository's configurations (one GPU's share of each model, with the split
count the configurations use), the whole Granite expert set, and odd shapes
like those of the tests.

The router is a random one: every token takes the top-k of iid Gumbel noise
plus a per-expert bias, which is zero (``uniform``) or ``-s log(rank + 1)``
over a random ranking of the experts (``zipf s``), so that a seed changes
which experts are hot as well as which tokens they get.  Gates are
renormalised softmax weights.  ``drop`` is the share of routed slots that are
dropped (tokens over an expert's capacity).
"""
import math

import numpy as np
import torch

from paper_2609_07536_amd import binding as B

# H, I, E, top-k, splits.  The first four are the repository's configurations.
SHAPES = {
    "tiny": dict(H=1024, I=512, E=8, topk=2, L=1),
    "granite": dict(H=1024, I=256, E=16, topk=8, L=1),
    "qwen": dict(H=2048, I=704, E=30, topk=4, L=2),
    "dsv2lite": dict(H=2048, I=704, E=32, topk=6, L=2),
    # Granite's whole expert set on one GPU (no tensor or expert parallelism)
    "granite_full": dict(H=1024, I=512, E=32, topk=8, L=1),
    # nothing a multiple of a tile: H, I and E as odd as the entry points take
    "odd": dict(H=1352, I=336, E=11, topk=3, L=1),
}


def _case(name, op, shape, T, routing="uniform", s=0.0, drop=0.0, mode=0):
    c = dict(name=name, op=op, shape=shape, T=T, routing=routing, s=s, drop=drop, mode=mode)
    c.update(SHAPES[shape])
    return c


def listed():
    return [
        # one user's decode step: the whole layer for one token, the smallest
        # call of serving, where launches and latencies are everything
        _case("layer_decode_1", "layer", "dsv2lite", 1),
        # a small batch of users decoding together: every call reads most of
        # the experts' weights for a few rows each
        _case("combine_decode_16", "combine", "qwen", 16),
        # a larger decode batch through the whole layer
        _case("layer_decode_64", "layer", "dsv2lite", 64, "zipf", 0.8),
        # decode inside a loop that may not allocate: the library's own scratch
        _case("noalloc_decode_48", "noalloc", "granite_full", 48),
        # the repository's tiny configuration
        _case("combine_tiny_256", "combine", "tiny", 256),
        # a ragged chunk of prefill: odd token count, odd sizes, dropped slots
        _case("layer_ragged_777", "layer", "odd", 777, "zipf", 1.0, 0.1),
        # one chunk of a chunked prefill, up-projection alone (a program that
        # fuses its own dispatch calls the two stages separately)
        _case("gemm1_chunk_1024", "gemm1", "qwen", 1024, "zipf", 0.8),
        # token bands on a prefill chunk with a skewed router
        _case("bands_chunk_4096", "combine", "dsv2lite", 4096, "zipf", 1.2, 0.0, 2),
        # the atomic scatter on a prefill chunk
        _case("scatter_chunk_2048", "combine", "granite", 2048, "uniform", 0.0, 0.0, 1),
        # the repository's Qwen-like configuration: a prefill batch
        _case("combine_prefill_8192", "combine", "qwen", 8192, "zipf", 0.8),
        # the repository's headline shape: a large prefill batch
        _case("combine_prefill_16384", "combine", "dsv2lite", 16384, "zipf", 1.2),
        # the whole layer on that batch, the largest call
        _case("layer_prefill_16384", "layer", "dsv2lite", 16384, "zipf", 1.2),
    ]


def draw(rng):
    shape = rng.choice(sorted(SHAPES))
    op = rng.choice(["combine", "combine", "layer", "gemm1", "noalloc"])
    c = dict(op=op, shape=shape)
    c.update(SHAPES[shape])
    most = 8192
    if op == "noalloc":   # what the library's scratch holds
        most = min(most, int(0.8 * B.NOALLOC_SCRATCH_BYTES / (2 * c["topk"] * (c["H"] + 256))))
    c["T"] = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    c["routing"] = rng.choice(["uniform", "zipf"])
    c["s"] = rng.choice([0.8, 1.0, 1.2]) if c["routing"] == "zipf" else 0.0
    c["drop"] = rng.choice([0.0, 0.0, 0.05, 0.2])
    c["mode"] = rng.choice([0, 0, 0, 2, 1]) if op == "combine" else 0
    return c


def _route(case, seed):
    """Expert-major rows: counts [E], token of each row, gate of each row."""
    g = np.random.default_rng([seed, case["T"], case["E"]])
    T, E, k = case["T"], case["E"], case["topk"]
    logits = g.standard_normal((T, E))
    key = g.gumbel(size=(T, E))
    if case["routing"] == "zipf":
        key -= case["s"] * np.log(g.permutation(E) + 1.0)
    sel = np.argpartition(-key, k - 1, axis=1)[:, :k]
    p = np.exp(np.take_along_axis(logits, sel, 1))
    p /= p.sum(1, keepdims=True)
    keep = np.ones(T * k, dtype=bool)
    keep[g.permutation(T * k)[:int(case["drop"] * T * k)]] = False
    keep = keep.reshape(T, k)
    tok = np.broadcast_to(np.arange(T)[:, None], (T, k))[keep]
    exp, gate = sel[keep], p[keep]
    order = np.lexsort((tok, exp))
    counts = np.bincount(exp, minlength=E)
    return counts, tok[order].astype(np.int32), gate[order].astype(np.float32)


def _normal(shape, scale, gen):
    return (torch.randn(shape, generator=gen, device="cuda") * scale).to(torch.bfloat16)


def prepare(case, seed):
    T, H, I, E, k = (case[n] for n in ("T", "H", "I", "E", "topk"))
    counts, tok, gate = _route(case, seed)
    rows = int(counts.sum())
    off = np.zeros(E + 1, dtype=np.int32)
    off[1:] = np.cumsum(counts)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    st = dict(case, rows=rows, off=torch.from_numpy(off).cuda(), tok=torch.from_numpy(tok).cuda(),
              gate=torch.from_numpy(gate).cuda())
    if case["op"] in ("layer", "gemm1"):
        st["hidden"] = _normal((T, H), 1.0, gen)
        w = _normal((E, H, 2 * I), 1.0 / math.sqrt(H), gen)
        st["w1"] = B.pack_w1(w)   # the weights a program lays out once
        st["w1_plain"] = w
    else:
        st["x"] = _normal((rows, I), 1.0, gen)
    if case["op"] != "gemm1":
        st["w2"] = _normal((E, I, H), 1.0 / math.sqrt(I), gen)
        st["out"] = torch.empty((T, H), dtype=torch.float32, device="cuda")
    else:
        st["out"] = torch.empty((max(rows, 1), I), dtype=torch.bfloat16, device="cuda")
    # the workspace a program allocates once for its layer
    wl, _ = B.make_workload(T, H, I, E, k, case["L"], rows=rows)
    if case["op"] == "layer":
        st["ws"] = B.Workspace(B.layer_workspace_size(wl))
    elif case["op"] == "combine":
        st["ws"] = B.Workspace(B.workspace_size(wl))
    elif case["op"] == "gemm1":
        st["ws"] = B.Workspace(512)
    return st


def run(st):
    op = st["op"]
    if op == "combine":
        B.combine(st["x"], st["w2"], st["off"], st["tok"], st["gate"], T=st["T"], splits=st["L"],
                  topk=st["topk"], out=st["out"], workspace=st["ws"],
                  mode=st["mode"] if st["mode"] else None)
    elif op == "noalloc":
        B.combine_noalloc(st["x"], st["w2"], st["off"], st["tok"], st["gate"], st["out"], T=st["T"],
                          splits=st["L"], topk=st["topk"])
    elif op == "gemm1":
        B.gemm1_swiglu(st["hidden"], st["w1"], st["off"], st["tok"], st["topk"], st["rows"],
                       out=st["out"], workspace=st["ws"])
    else:
        B.layer_forward(st["hidden"], st["w1"], st["w2"], st["off"], st["tok"], st["gate"],
                        st["topk"], splits=st["L"], out=st["out"], workspace=st["ws"])
    return st["out"]


def work(case):
    T, H, I = case["T"], case["H"], case["I"]
    counts, tok, _ = _route(case, 0)
    rows, experts, tokens = int(counts.sum()), int((counts > 0).sum()), len(np.unique(tok))
    w1, w2 = experts * H * 2 * I * 2, experts * I * H * 2   # the experts that have rows
    up, down = 2 * rows * H * 2 * I, 2 * rows * I * H
    idx = 4 * (case["E"] + 1) + 4 * rows
    if case["op"] == "gemm1":
        return {"bytes": w1 + tokens * H * 2 + idx + rows * I * 2, "flops": up}
    if case["op"] == "layer":
        return {"bytes": w1 + w2 + tokens * H * 2 + idx + 4 * rows + T * H * 4, "flops": up + down}
    return {"bytes": w2 + rows * I * 2 + idx + 4 * rows + T * H * 4, "flops": down}


def tolerance(case):
    # About four times the distance from 64-bit arithmetic that one bf16
    # rounding of Y (combine) or of the activations (gemm1), 1.7e-3, or both
    # (layer), 2.3e-3, leaves.
    return {"rel": 1e-2 if case["op"] == "layer" else 7e-3}


def exact(case, seed):
    st = prepare(case, seed)
    off = st["off"].tolist()
    T, H, I = case["T"], case["H"], case["I"]
    tok = st["tok"].long()
    out = torch.zeros((max(st["rows"], 1), I) if case["op"] == "gemm1" else (T, H),
                      dtype=torch.float64, device="cuda")
    for e in range(case["E"]):
        a, b = off[e], off[e + 1]
        if a == b:
            continue
        if case["op"] in ("layer", "gemm1"):
            h = st["hidden"][tok[a:b]].double() @ st["w1_plain"][e].double()
            act = torch.nn.functional.silu(h[:, :I]) * h[:, I:]
            del h
            if case["op"] == "gemm1":
                out[a:b] = act
                continue
        else:
            act = st["x"][a:b].double()
        out.index_add_(0, tok[a:b], st["gate"][a:b].double()[:, None] * (act @ st["w2"][e].double()))
    return out

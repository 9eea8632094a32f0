"""The calls whose speed is measured, as a serving program makes them.

A program that serves requests from document caches holds a pool of compiled K/V, a rotary table
and a plan; per request batch it composes a cache, prefills the suffix tokens layer by layer and
then decodes.  The cases are those calls over their real range: one small float32 request (the
exact-check shape), a lone 32-layer request from plan to second token, and single layers of every
call at the sizes of the workloads in synth/configs.py (Llama-3-8B and Qwen2.5-7B shaped
attention, head_dim 64 and 128).

Kinds of case:
  request    plan -> blocks to the device -> compose -> prefill of every layer -> decode steps
  compose    composition of a batch's caches (per block, or grouped by shared source runs)
  rerotate   standalone re-rotation of a key set
  prefill    one layer's suffix prefill (tokens already rotated, or rotated by the call)
  frontier   one layer's prefill of inline spans between documents
  paged      slot map -> tiles composed ahead -> prefill of the layers straight from the pool
  decode     one layer's decode step (tokens already rotated, or rotated by the call)
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2607_28069_amd as pic

DEV = "cuda"
# (query heads, kv heads, head_dim, rope theta)
SHAPES = {
    "llama8b": (32, 8, 128, 5e5),
    "qwen7b": (28, 4, 128, 1e6),
    "llama_hd64": (32, 8, 64, 5e5),
    "small": (16, 4, 64, 1e4),
    "tiny": (4, 2, 64, 1e4),
}


def listed():
    return [
        # the tiny exact-check request: every launch is latency, in float32
        dict(name="request_tiny_f32", kind="request", shape="tiny", dtype="f32", layers=1, batch=1, docs=2,
             pool_docs=2, doc_lo=128, doc_hi=128, prefix=16, suffix=16, steps=1),
        # one user waiting for the first two tokens of a 32-layer model: time to first token at batch 1
        dict(name="request_llama_lone", kind="request", shape="llama8b", dtype="bf16", layers=32, batch=1, docs=10,
             pool_docs=16, doc_lo=1024, doc_hi=1024, prefix=128, suffix=128, steps=1),
        # a batch of 16 requests sharing a pool of 64 documents: four of the 32 layers
        dict(name="compose_llama_batch", kind="compose", shape="llama8b", dtype="bf16", layers=4, batch=16, docs=10,
             pool_docs=64, doc_lo=1024, doc_hi=1024, prefix=128, shared=True, pairing="half"),
        # a stored key set moved to new positions, two layers' worth of the batch above
        dict(name="rerotate_keys", kind="rerotate", dtype="bf16", tokens=331776, heads=8, head_dim=128,
             pairing="half"),
        # one layer of the batch above: 128 suffix tokens over about 10K of context
        dict(name="prefill_llama_batch", kind="prefill", shape="llama8b", dtype="bf16", batch=16, ctx=10368, ragged=0.0,
             suffix=128, rope=False, pairing="half"),
        # long contexts of uneven length, 256 suffix tokens, 7 query heads per kv head
        dict(name="prefill_qwen_32k", kind="prefill", shape="qwen7b", dtype="bf16", batch=8, ctx=32749, ragged=0.25,
             suffix=256, rope=False, pairing="half"),
        # a small batch at head_dim 64, suffix tokens rotated by the call: a short launch
        dict(name="prefill_hd64_rope", kind="prefill", shape="llama_hd64", dtype="bf16", batch=4, ctx=4160, ragged=0.0,
             suffix=64, rope=True, pairing="half"),
        # a small float32 model
        dict(name="prefill_small_f32", kind="prefill", shape="small", dtype="f32", batch=4, ctx=2077, ragged=0.25,
             suffix=61, rope=False, pairing="half"),
        # inline prefix and spans between documents: 576 inline tokens per request
        dict(name="frontier_llama_batch", kind="frontier", shape="llama8b", dtype="bf16", batch=16, docs=10, doc=1024,
             prefix=128, span=32, query=128),
        # zero-copy first token: two 32K requests of documents with uneven lengths, four layers
        dict(name="paged_qwen_32k", kind="paged", shape="qwen7b", dtype="bf16", layers=4, batch=2, docs=32, pool_docs=32,
             doc_lo=768, doc_hi=1280, prefix=0, suffix=256, tiles=True, pairing="half"),
        # a full decode batch: 64 requests at 16K, one layer
        dict(name="decode_llama_64x16k", kind="decode", shape="llama8b", dtype="bf16", batch=64, ctx=16384, ragged=0.0,
             step=100, rope=False, pairing="half"),
        # a small decode batch of long, uneven contexts, the new token rotated by the call
        dict(name="decode_qwen_32k_rope", kind="decode", shape="qwen7b", dtype="bf16", batch=8, ctx=33001, ragged=0.5,
             step=7, rope=True, pairing="half"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["request", "compose", "rerotate", "prefill", "prefill", "frontier", "paged", "decode"])
    f32 = kind in ("request", "compose", "rerotate", "prefill", "decode") and rng.random() < 0.2
    dtype = "f32" if f32 else "bf16"
    pairing = rng.choice(["half", "half", "interleaved"])
    shape = rng.choice(["tiny", "small"]) if f32 else rng.choice(["llama8b", "llama8b", "qwen7b", "llama_hd64"])
    hq, hkv, d, _ = SHAPES[shape]
    if kind == "rerotate":
        return dict(kind=kind, dtype=dtype, tokens=_log(rng, 64, 331776 // (2 if f32 else 1)), heads=rng.choice([1, 2, 4, 8]),
                    head_dim=rng.choice([64, 128]), pairing=pairing)
    if kind in ("request", "compose", "paged"):
        docs = rng.randint(2, 16)
        doc_lo = _log(rng, 64, 1024)
        doc_hi = doc_lo + rng.choice([0, rng.randint(1, doc_lo)])
        c = dict(kind=kind, shape=shape, dtype=dtype, layers=rng.randint(1, 4), batch=_log(rng, 1, 8), docs=docs,
                 pool_docs=docs + rng.randint(0, 48), doc_lo=doc_lo, doc_hi=doc_hi, prefix=rng.choice([0, 16, 128]))
        if f32:   # float32 serves small models and short contexts
            c.update(layers=1, batch=rng.randint(1, 2), docs=min(docs, 4), doc_lo=min(doc_lo, 256), doc_hi=min(doc_hi, 384))
        if kind == "request":
            c.update(suffix=_log(rng, 1, 256), steps=rng.randint(1, 2))
        elif kind == "paged":
            c.update(suffix=_log(rng, 1, 256), tiles=rng.random() < 0.7, pairing=pairing)
        else:
            c.update(shared=rng.random() < 0.7, pairing=pairing)
        if kind != "compose":   # no more work than the largest listed case
            pairs = 2e9 / 4 if f32 else 9e11 / 4
            while c["layers"] * c["batch"] * hq * d * c["suffix"] * docs * doc_hi > pairs and c["batch"] > 1:
                c["batch"] -= 1
            while c["layers"] * c["batch"] * hq * d * c["suffix"] * docs * doc_hi > pairs and c["suffix"] > 1:
                c["suffix"] //= 2
        return c
    if kind == "frontier":
        docs, doc, span, batch = rng.randint(2, 10), _log(rng, 64, 1024), rng.randint(1, 48), _log(rng, 1, 16)
        return dict(kind=kind, shape=shape, dtype=dtype, batch=batch, docs=docs, doc=doc, prefix=rng.choice([0, 48, 128]),
                    span=span, query=_log(rng, 8, 128))
    ragged = rng.choice([0.0, 0.0, 0.25, 0.5])
    rope = not f32 and rng.random() < 0.4
    if kind == "prefill":
        batch, suffix = (_log(rng, 1, 4), _log(rng, 1, 64)) if f32 else (_log(rng, 1, 16), _log(rng, 1, 256))
        top = min(2048 if f32 else 32768, int((2e9 if f32 else 9e11) / (4 * hq * d * batch * suffix)))
        return dict(kind=kind, shape=shape, dtype=dtype, batch=batch, ctx=_log(rng, 64, max(top, 65)), ragged=ragged,
                    suffix=suffix, rope=rope, pairing=pairing)
    batch = _log(rng, 1, 4 if f32 else 64)
    top = min(4096 if f32 else 33000, int(4e9 / (hkv * d * 4 * batch)))
    return dict(kind=kind, shape=shape, dtype=dtype, batch=batch, ctx=_log(rng, 64, top), ragged=ragged,
                step=rng.randint(0, 255), rope=rope, pairing=pairing)


# ------------------------------------------------------------------------------------------
# layouts: fixed by the case, so that the work does not depend on the seed; only the order of a
# request's documents does
# ------------------------------------------------------------------------------------------

def _pool(case):
    """(entry lengths, entry offsets, per request the entries it composes, unordered)"""
    r = random.Random(1)
    lens = [r.randint(case["doc_lo"], case["doc_hi"]) for _ in range(case["pool_docs"])]
    picks = [r.sample(range(case["pool_docs"]), case["docs"]) for _ in range(case["batch"])]
    if case["prefix"]:
        lens.append(case["prefix"])
    lens = np.asarray(lens, np.int32)
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    return lens, offs, picks


def _ctx_of(case):
    lens, _, picks = _pool(case)
    return [int(lens[p].sum()) + case["prefix"] for p in picks]


def _ragged(case):
    """Context lengths of a batch: the longest is case["ctx"], the others up to a share `ragged` shorter."""
    r = random.Random(2)
    return [case["ctx"]] + [case["ctx"] - int(r.random() * case["ragged"] * case["ctx"]) for _ in range(case["batch"] - 1)]


def _spans(case):
    """Inline positions of a frontier request and its length: prefix, then a span after every document, then the query."""
    pos, at = list(range(case["prefix"])), case["prefix"]
    for i in range(case["docs"]):
        at += case["doc"]
        n = case["span"] + (case["query"] if i == case["docs"] - 1 else 0)
        pos += range(at, at + n)
        at += n
    return pos, at


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------

class _Gen:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) + 12345)
        self.dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def __call__(self, *shape):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=self.dt)


def _table(model, mad):
    t = torch.empty(pic.pic_rope_table_bytes(model, mad) // 4, dtype=torch.float32, device=DEV)
    pic.pic_rope_table_init(model, mad, t)
    return t


def _bytes(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device=DEV)


def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int32).reshape(-1).copy()).to(DEV)


def prepare(case, seed):
    kind, g = case["kind"], _Gen(seed, case["dtype"])
    s = dict(case=dict(case), kind=kind)
    if kind == "rerotate":
        n, h, d = case["tokens"], case["heads"], case["head_dim"]
        m = s["model"] = pic.Model.of(1, h, h, d, case["dtype"], 5e5, case["pairing"])
        s["k"] = g(n, h, d)
        s["out"] = torch.empty_like(s["k"])
        s["mad"] = 16384
        # documents of 1024 tokens, each moved by one shift
        r = np.random.default_rng(seed)
        s["delta"] = _i32(np.repeat(r.integers(-16384, 16385, -(-n // 1024)), 1024)[:n].astype(np.int32))
        s["table"] = _table(m, s["mad"])
        return s
    hq, hkv, d, theta = SHAPES[case["shape"]]
    L, B = case.get("layers", 1), case["batch"]
    s["model"] = pic.Model.of(L, hq, hkv, d, case["dtype"], theta, case.get("pairing", "half"))
    s["m1"] = s["model"].with_layers(1)
    if kind in ("request", "compose", "paged"):
        lens, offs, picks = _pool(case)
        r = random.Random(seed)
        picks = [r.sample(p, len(p)) for p in picks]
        s["requests"] = [([len(lens) - 1] if case["prefix"] else []) + p for p in picks]
        s["lens"], s["offs"], s["cpos"] = lens, offs, np.zeros_like(lens)
        T = s["T"] = int(lens.sum())
        ctx = _ctx_of(case)
        ls, steps = case.get("suffix", 0), case.get("steps", 0)
        s["max_ctx"], s["cap"] = max(ctx), max(ctx) + ls + steps
        s["mad"] = s["cap"]
        s["table"] = _table(s["model"], s["mad"])
        s["pool_k"], s["pool_v"] = g(L, hkv, T, d), g(L, hkv, T, d)
        s["cache_k"] = torch.zeros((L, B, hkv, s["cap"], d), dtype=g.dt, device=DEV)
        s["cache_v"] = torch.zeros_like(s["cache_k"])
        s["ctx"] = _i32(np.asarray(ctx, np.int32))
        blocks, _ = pic.pic_plan_layout(s["requests"], offs, lens, s["cpos"], T)
        s["host_blocks"] = blocks
        if kind != "request":
            if case.get("shared"):
                blocks, starts = pic.pic_plan_shared(blocks)
                s["starts"], s["n_groups"] = _i32(starts), len(starts) - 1
            s["blocks"], s["n_blocks"] = _i32(blocks), len(blocks)
        if kind == "compose":
            return s
        s["q"], s["k"], s["v"] = g(L, B, ls, hq, d), g(L, B, ls, hkv, d), g(L, B, ls, hkv, d)
        s["out"] = torch.zeros((L, B, ls, hq, d), dtype=g.dt, device=DEV)
        s["ws"] = _bytes(pic.pic_prefill_workspace_bytes(s["m1"], B, ls, s["max_ctx"]))
        if kind == "request":
            s["dq"], s["dk"], s["dv"] = g(steps, L, B, hq, d), g(steps, L, B, hkv, d), g(steps, L, B, hkv, d)
            s["dout"] = torch.zeros((steps, L, B, hq, d), dtype=g.dt, device=DEV)
            s["base"] = _i32(np.asarray(ctx, np.int32) + ls)
            s["max_base"] = s["max_ctx"] + ls
            s["dws"] = _bytes(pic.pic_decode_workspace_bytes(s["m1"], B, s["max_base"] + steps, 0))
        else:
            s["slot_src"] = torch.zeros((B, s["max_ctx"]), dtype=torch.int32, device=DEV)
            s["slot_delta"] = torch.zeros_like(s["slot_src"])
            s["tile_map"] = torch.zeros((B, pic.pic_slot_map_tiles(s["max_ctx"]), 2), dtype=torch.int32, device=DEV)
        return s
    if kind == "frontier":
        pos, total = _spans(case)
        n = s["n"] = len(pos)
        s["cap"] = s["max_len"] = total
        s["pos"] = _i32(np.tile(np.asarray(pos, np.int32), B))
        s["n_valid"] = _i32(np.full(B, n, np.int32))
        s["ws"] = _bytes(pic.pic_frontier_workspace_bytes(s["m1"], B, n, total))
        s["q"], s["k"], s["v"] = g(B, n, hq, d), g(B, n, hkv, d), g(B, n, hkv, d)
        s["out"] = torch.zeros_like(s["q"])
    else:
        ctx = _ragged(case)
        s["ctx"], s["max_ctx"] = _i32(np.asarray(ctx, np.int32)), max(ctx)
        n = case["suffix"] if kind == "prefill" else case["step"] + 1
        s["cap"] = s["max_ctx"] + n
        s["mad"] = s["cap"]
        if case["rope"]:
            s["table"] = _table(s["m1"], s["mad"])
        if kind == "prefill":
            s["ws"] = _bytes(pic.pic_prefill_workspace_bytes(s["m1"], B, n, s["max_ctx"]))
            s["q"], s["k"], s["v"] = g(B, n, hq, d), g(B, n, hkv, d), g(B, n, hkv, d)
        else:
            s["ws"] = _bytes(pic.pic_decode_workspace_bytes(s["m1"], B, s["cap"], 0))
            s["q"], s["k"], s["v"] = g(B, hq, d), g(B, hkv, d), g(B, hkv, d)
        s["out"] = torch.zeros_like(s["q"])
    s["cache_k"], s["cache_v"] = g(B, hkv, s["cap"], d), g(B, hkv, s["cap"], d)
    return s


# ------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------

def _run_request(s):
    c, m1, L, B = s["case"], s["m1"], s["case"]["layers"], s["case"]["batch"]
    blocks, _ = pic.pic_plan_layout(s["requests"], s["offs"], s["lens"], s["cpos"], s["T"])
    if B > 1:
        blocks, starts = pic.pic_plan_shared(blocks)
        dev_blocks = torch.from_numpy(blocks.view(np.int32)).to(DEV)
        dev_starts = torch.from_numpy(starts).to(DEV)
        pic.pic_compose_shared(s["model"], s["pool_k"], s["pool_v"], s["T"], dev_blocks, len(blocks), dev_starts,
                               len(starts) - 1, s["table"], s["mad"], s["cache_k"], s["cache_v"], B, s["cap"])
    else:
        dev_blocks = torch.from_numpy(blocks.view(np.int32)).to(DEV)
        pic.pic_compose(s["model"], s["pool_k"], s["pool_v"], s["T"], dev_blocks, len(blocks), s["table"], s["mad"],
                        s["cache_k"], s["cache_v"], B, s["cap"])
    for l in range(L):
        pic.pic_suffix_prefill_attn(m1, s["q"][l], s["k"][l], s["v"][l], s["cache_k"][l], s["cache_v"][l], B, s["cap"],
                                    s["ctx"], s["max_ctx"], c["suffix"], s["out"][l], s["ws"])
    for t in range(c["steps"]):
        for l in range(L):
            pic.pic_decode_attn(m1, s["dq"][t, l], s["dk"][t, l], s["dv"][t, l], s["cache_k"][l], s["cache_v"][l], B,
                                s["cap"], s["base"], t, s["max_base"], s["dout"][t, l], s["dws"])
    return {"out": s["out"], "dout": s["dout"], "cache_k": s["cache_k"], "cache_v": s["cache_v"]}


def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "request":
        return _run_request(s)
    if kind == "rerotate":
        pic.pic_rerotate_keys(s["model"], s["k"], s["out"], c["tokens"], c["heads"], s["delta"], s["table"], s["mad"])
        return s["out"]
    B = c["batch"]
    if kind == "compose":
        if c["shared"]:
            pic.pic_compose_shared(s["model"], s["pool_k"], s["pool_v"], s["T"], s["blocks"], s["n_blocks"], s["starts"],
                                   s["n_groups"], s["table"], s["mad"], s["cache_k"], s["cache_v"], B, s["cap"])
        else:
            pic.pic_compose(s["model"], s["pool_k"], s["pool_v"], s["T"], s["blocks"], s["n_blocks"], s["table"], s["mad"],
                            s["cache_k"], s["cache_v"], B, s["cap"])
        return {"cache_k": s["cache_k"], "cache_v": s["cache_v"]}
    if kind == "paged":
        tiles, cap = s["tile_map"] if c["tiles"] else None, s["max_ctx"]
        src, delta = s["slot_src"], s["slot_delta"]
        pic.pic_build_slot_map(s["blocks"], s["n_blocks"], B, cap, src, delta, tiles)
        if tiles is not None:
            pic.pic_compose_tiles(s["model"], s["pool_k"], s["pool_v"], s["T"], src, delta, cap, tiles, s["table"], s["mad"],
                                  s["ctx"], s["max_ctx"], s["cache_k"], s["cache_v"], B, s["cap"])
            src = delta = None
        for l in range(c["layers"]):
            pic.pic_paged_prefill_attn(s["m1"], s["pool_k"][l], s["pool_v"][l], s["T"], src, delta, cap, s["table"], s["mad"],
                                       s["q"][l], s["k"][l], s["v"][l], s["cache_k"][l], s["cache_v"][l], B, s["cap"],
                                       s["ctx"], s["max_ctx"], c["suffix"], s["out"][l], s["ws"], tile_map=tiles)
        return s["out"]
    args = (s["m1"], s["q"], s["k"], s["v"], s["cache_k"], s["cache_v"], B, s["cap"])
    if kind == "frontier":
        pic.pic_frontier_prefill_attn(*args, s["pos"], s["n_valid"], s["n"], s["max_len"], s["out"], s["ws"])
    elif kind == "prefill" and c["rope"]:
        pic.pic_suffix_prefill_attn_rope(*args, s["ctx"], s["max_ctx"], c["suffix"], s["table"], s["mad"], s["out"], s["ws"])
    elif kind == "prefill":
        pic.pic_suffix_prefill_attn(*args, s["ctx"], s["max_ctx"], c["suffix"], s["out"], s["ws"])
    elif c["rope"]:
        pic.pic_decode_attn_rope(*args, s["ctx"], c["step"], s["max_ctx"], s["table"], s["mad"], s["out"], s["ws"])
    else:
        pic.pic_decode_attn(*args, s["ctx"], c["step"], s["max_ctx"], s["out"], s["ws"])
    return {"out": s["out"], "cache_k": s["cache_k"], "cache_v": s["cache_v"]}


# ------------------------------------------------------------------------------------------
# the work a pass cannot do without, and how far a correct result may be off
# ------------------------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    e = 4 if case["dtype"] == "f32" else 2
    if kind == "rerotate":
        n = case["tokens"] * case["heads"] * case["head_dim"]
        return {"bytes": 2 * n * e + 4 * case["tokens"], "flops": 3 * n}
    hq, hkv, d, _ = SHAPES[case["shape"]]
    L, B = case.get("layers", 1), case["batch"]
    row, qrow = hkv * d * e * 2, hq * d * e   # one token's K and V; one token's q or out
    if kind in ("request", "compose", "paged"):
        lens, _, picks = _pool(case)
        ctx = _ctx_of(case)
        used = sum(int(lens[i]) for i in set().union(*picks)) + case["prefix"]
        moved = L * row * (used + sum(ctx))            # every document run read once, every slot written
        rot = 3 * L * hkv * d * sum(ctx)
        if kind == "compose":
            return {"bytes": moved, "flops": rot}
        ls = case["suffix"]
        pairs = sum(c * ls + ls * (ls + 1) // 2 for c in ctx)
        flops = 4 * L * hq * d * pairs
        io = L * B * ls * (2 * qrow + 2 * row)
        if kind == "paged":
            return {"bytes": L * row * used + io, "flops": flops}
        for t in range(case["steps"]):
            n = sum(c + ls + t + 1 for c in ctx)
            flops += 4 * L * hq * d * n
            io += L * (row * n + B * (2 * qrow + 2 * row))
        return {"bytes": moved + L * row * sum(ctx) + io, "flops": flops + rot}
    if kind == "frontier":
        pos, total = _spans(case)
        return {"bytes": B * (row * total + len(pos) * (2 * qrow + 2 * row)), "flops": 4 * hq * d * B * sum(p + 1 for p in pos)}
    ctx = _ragged(case)
    if kind == "prefill":
        ls = case["suffix"]
        return {"bytes": row * sum(ctx) + B * ls * (2 * qrow + 2 * row),
                "flops": 4 * hq * d * sum(c * ls + ls * (ls + 1) // 2 for c in ctx)}
    n = sum(c + case["step"] + 1 for c in ctx)
    return {"bytes": row * n + B * (2 * qrow + 2 * row), "flops": 4 * hq * d * n}


def tolerance(case):
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind in ("rerotate", "compose"):
        # one rotation in float32 (angles up to 2^15 rounded once to float32 cos/sin); in bf16 a
        # rounding that falls the other way moves a value by one unit in its last place
        return {"rel": 5e-7, "max": 1e-5} if f32 else {"rel": 1e-4, "max": 1.6e-2}
    if f32:   # 32-bit sums over up to a few thousand keys: 3.5e-7 off 64 bits
        return {"rel": 2e-6, "max": 4e-5}
    # bf16: probabilities and outputs rounded once each (2^-9 at most); composed paths round the
    # turned keys or queries too: 1.9e-3 to 3.3e-3 off 64 bits
    return {"rel": 1e-2, "max": 1e-1}


# ------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------

def _turned(x, pos, theta, pairing):
    """Rows x [..., n, D] turned to positions pos [n], in 64 bits."""
    d = x.shape[-1]
    inv = float(theta) ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    ang = pos.to(torch.float64)[:, None] * inv
    c, s = ang.cos(), ang.sin()
    x = x.double()
    y = torch.empty_like(x)
    a, b = (slice(0, d // 2), slice(d // 2, d)) if pairing == "half" else (slice(0, d, 2), slice(1, d, 2))
    y[..., a] = x[..., a] * c - x[..., b] * s
    y[..., b] = x[..., a] * s + x[..., b] * c
    return y


def _attend(q, k, v, pos):
    """q [n, Hq, D] at positions pos [n] over slots k, v [Hkv, S, D] (64 bits): each query sees slots 0 .. its position."""
    n, hq, d = q.shape
    rep = hq // k.shape[0]
    out = torch.empty_like(q)
    slots = torch.arange(k.shape[1], device=q.device)
    for h in range(k.shape[0]):
        s = (q[:, h * rep:(h + 1) * rep].reshape(n * rep, d) @ k[h].t().contiguous()) / math.sqrt(d)
        s.masked_fill_(slots[None, :] > pos.repeat_interleave(rep)[:, None], -math.inf)
        out[:, h * rep:(h + 1) * rep] = (torch.softmax(s, -1) @ v[h]).reshape(n, rep, d)
    return out


def _exact_composed(s, l, b):
    """K, V [Hkv, ctx, D] of request b's composed context on layer l."""
    c = s["case"]
    theta, K, V = SHAPES[c["shape"]][3], [], []
    at = 0
    for e in s["requests"][b]:
        o, n = int(s["offs"][e]), int(s["lens"][e])
        shift = torch.full((n,), at, device=DEV)
        K.append(_turned(s["pool_k"][l, :, o:o + n], shift, theta, c.get("pairing", "half")))
        V.append(s["pool_v"][l, :, o:o + n].double())
        at += n
    return torch.cat(K, 1), torch.cat(V, 1)


def exact(case, seed):
    s, kind = prepare(case, seed), case["kind"]
    if kind == "rerotate":
        return _turned(s["k"].transpose(0, 1), s["delta"], 5e5, case["pairing"]).transpose(0, 1).contiguous()
    hq, hkv, d, theta = SHAPES[case["shape"]]
    L, B = case.get("layers", 1), case["batch"]
    if kind in ("request", "compose", "paged"):
        ls, steps = case.get("suffix", 0), case.get("steps", 0)
        ck = torch.zeros((L, B, hkv, s["cap"], d), dtype=torch.float64, device=DEV)
        cv = torch.zeros_like(ck)
        out = s["out"].double() if ls else None
        dout = s["dout"].double() if steps else None
        ctx = _ctx_of(case)
        for l in range(L):
            for b in range(B):
                n = ctx[b]
                ck[l, b, :, :n], cv[l, b, :, :n] = _exact_composed(s, l, b)
                if not ls:
                    continue
                ck[l, b, :, n:n + ls], cv[l, b, :, n:n + ls] = s["k"][l, b].double().transpose(0, 1), s["v"][l, b].double().transpose(0, 1)
                out[l, b] = _attend(s["q"][l, b].double(), ck[l, b, :, :n + ls], cv[l, b, :, :n + ls], n + torch.arange(ls, device=DEV))
                for t in range(steps):
                    p = n + ls + t
                    ck[l, b, :, p], cv[l, b, :, p] = s["dk"][t, l, b].double(), s["dv"][t, l, b].double()
                    dout[t, l, b] = _attend(s["dq"][t, l, b].double()[None], ck[l, b, :, :p + 1], cv[l, b, :, :p + 1],
                                            torch.tensor([p], device=DEV))[0]
        if kind == "compose":
            return {"cache_k": ck, "cache_v": cv}
        return out if kind == "paged" else {"out": out, "dout": dout, "cache_k": ck, "cache_v": cv}
    ck, cv = s["cache_k"].double(), s["cache_v"].double()
    out = s["out"].double()
    for b in range(B):
        if kind == "frontier":
            pos = s["pos"].view(B, -1)[b].long()
        else:
            n = int(s["ctx"][b])
            pos = n + (torch.arange(case["suffix"], device=DEV) if kind == "prefill" else torch.tensor([case["step"]], device=DEV))
        q, k, v = (x[b].double() if kind != "decode" else x[b].double()[None] for x in (s["q"], s["k"], s["v"]))
        if case.get("rope"):
            q = _turned(q.transpose(0, 1), pos, theta, case["pairing"]).transpose(0, 1).contiguous()
            k = _turned(k.transpose(0, 1), pos, theta, case["pairing"]).transpose(0, 1).contiguous()
        ck[b, :, pos], cv[b, :, pos] = k.transpose(0, 1), v.transpose(0, 1)
        top = int(pos.max()) + 1
        y = _attend(q, ck[b, :, :top], cv[b, :, :top], pos)
        out[b] = y if kind != "decode" else y[0]
    return {"out": out, "cache_k": ck, "cache_v": cv}

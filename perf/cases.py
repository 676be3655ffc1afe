"""The calls whose speed this repository cares about: one token's decode attention, through the entry
points a program calls, from a single 4K layer to a whole 36-layer step at 128K.

A case is a dict of sizes and options:
  call      "layer"   one lychee_decode_attn (its index sets complete when the call's work is)
            "static"  lychee_decode_attn_static: the same on the library's own scratch
            "loop"    the model loop: one lychee_decode_attn_deferred per layer, then a flush
            "step"    lychee_decode_step (lychee_decode_step_append if `append`), in either order
            "dense"   lychee_dense_decode_attn: every head over the whole cache
  phased    "step" only: all layers pooled per phase (the library's default) or layer after layer
  batch, q_heads, kv_heads, layers, k   as in lychee_shape (k counts blocks when `block` is 64)
  len_lo, len_hi   the sequences' lengths are spread over this range
  cap       rows the cache holds per sequence (>= len_hi; also the host-known bound of the lengths)
  retrieval retrieval heads per layer; `first_dense`: every head of layer 0 is one
  rule, param      "topk", "ratio" (share kept), "threshold" or "top_p" (on probabilities)
  block     1: sets name positions; 64: blocks of 64 positions
  planted, zipf    query-aligned rows per KV head and the exponent of their heavy tail (0: equal)
  token_major      cache layout [B][L][H_kv][128] instead of [B][H_kv][L][128]

Head types and lengths belong to the case (a model's assignment and a batch's lengths are fixed before a
call); values come from the seed: N(0,1) in bf16 with planted query-aligned keys, so that the selection is
not a choice among equals, and inherited sets that an independent query picked on the same cache.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2602_04541_amd import binding as lb

D = 128
DEV = "cuda"
RULES = {"topk": 0, "ratio": 0, "threshold": lb.RULE_THRESHOLD, "top_p": lb.RULE_TOP_P}


def _case(name=None, **kw):
    c = dict(call="layer", phased=False, batch=1, q_heads=32, kv_heads=8, layers=1, len_lo=0, len_hi=32768, cap=0,
             k=2048, retrieval=4, first_dense=False, append=False, rule="topk", param=0.0, block=1, planted=512,
             zipf=0.0, token_major=False)
    c.update(kw)
    c["len_lo"] = c["len_lo"] or c["len_hi"]
    c["cap"] = c["cap"] or c["len_hi"]
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one layer of a small model at 4K (two KV heads), launches and latency
        _case("layer_4k", q_heads=8, kv_heads=2, len_hi=4096, k=256, retrieval=2, planted=32),
        # an ordinary layer of an 8B-class model at 32K, called alone by code that needs its sets at once
        _case("layer_32k", len_hi=32768, k=2048),
        # a batch of long conversations of unequal lengths
        _case("layer_b8_16k_96k", batch=8, len_lo=16411, len_hi=98304, k=2048, planted=256),
        # a serving batch of many short sequences in a paged-allocator style cache (token-major, room to grow)
        _case("layer_b64_short", batch=64, len_lo=61, len_hi=3001, cap=4096, k=512, planted=24, token_major=True),
        # a wide budget at an odd long context, on the entry point that allocates nothing
        _case("static_100k_k8192", call="static", len_hi=100003, k=8192, planted=1024, zipf=1.2),
        # the Top-p rule (a set as large as the attention mass asks for) at 128K
        _case("layer_128k_top_p", len_hi=131072, k=4096, rule="top_p", param=0.9, planted=1024, zipf=1.2),
        # block-granular sets, batch 8 at 128K, two of eight KV groups dense, a tenth of the blocks kept
        _case("blocks_b8_128k", batch=8, len_hi=131072, k=204, retrieval=8, block=64, planted=256),
        # the model loop at a middling context: one call per layer, the select inside the next call
        _case("loop_8x32k", call="loop", layers=8, len_hi=32768, k=4096, retrieval=3, planted=1024, zipf=1.2),
        # a whole decode step early in a conversation: appends, 36 layers one after the other
        _case("step_36x4k", call="step", layers=36, len_hi=4099, cap=8192, k=1024, retrieval=3, first_dense=True,
              append=True, planted=256, zipf=1.2),
        # a whole decode step in the library's default order (pooled phases), appends inside
        _case("step_phased_36x32k", call="step", phased=True, layers=36, len_hi=33333, cap=33408, k=4096, retrieval=3,
              first_dense=True, append=True, planted=1024, zipf=1.2),
        # the headline: the 36-layer step at 128K, layer after layer as a model has to run it
        _case("step_36x128k", call="step", layers=36, len_hi=131072, k=4096, retrieval=3, first_dense=True,
              planted=1024, zipf=1.2),
        # a layer that keeps every head dense, at 128K
        _case("dense_128k", call="dense", len_hi=131072, k=1, retrieval=32, planted=1024, zipf=1.2),
    ]


# The most cache rows (K and V, 512 bytes a row) a drawn case streams or holds.
MOST_ROWS = 14_000_000


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any entry point, 1K to 128K of context, budgets from 64 rows to 8192,
    groups of 1 to 4 query heads, batches up to 64, either layout, every rule; sizes mostly odd."""
    call = rng.choice(["layer", "layer", "layer", "static", "loop", "loop", "step", "step", "step", "dense"])
    kv = rng.choice([2, 4, 8, 8, 8])
    group = rng.choice([1, 2, 3, 4, 4, 4])
    q_heads = kv * group
    layers = rng.randint(2, 8) if call == "loop" else rng.randint(4, 36) if call == "step" else 1
    batch = rng.choice([1, 1, 1, 1, 2, 5, 8]) if call in ("loop", "step") else rng.choice([1, 1, 1, 2, 3, 8, 17, 64])
    if call == "static":
        batch = 1
    most = max(2048, min(131072, MOST_ROWS // (batch * kv * layers)))
    len_hi = _log(rng, 1024, most)
    len_lo = len_hi if batch == 1 else max(1, int(len_hi * rng.uniform(0.1, 0.9)))
    block = 64 if call not in ("static", "dense") and rng.random() < 0.2 else 1
    k = _log(rng, 64, max(65, min(8192, len_hi // 4)))
    if block == 64:
        k = max(1, k // 64)
    rule, param = "topk", 0.0
    if block == 1 and call in ("layer", "static") and rng.random() < 0.3:
        rule, param = rng.choice([("threshold", 1e-4), ("top_p", 0.9), ("top_p", 0.5)])
    elif call != "dense" and rng.random() < 0.15:
        rule, param = "ratio", round(rng.uniform(0.01, 0.25), 3)
    return _case(call=call, phased=call == "step" and rng.random() < 0.5, batch=batch, q_heads=q_heads, kv_heads=kv,
                 layers=layers, len_lo=len_lo, len_hi=len_hi, cap=len_hi + rng.choice([0, 0, 1, 63, 200]), k=k,
                 retrieval=q_heads if call == "dense" else rng.randint(1, max(1, q_heads // 4)),
                 first_dense=call == "step", append=call == "step" and rng.random() < 0.5, rule=rule, param=param,
                 block=block, planted=max(8, min(1024, len_lo // 32)), zipf=rng.choice([0.0, 1.2]),
                 token_major=rng.random() < 0.2)


# ------------------------------------------------------------------ what belongs to the case


def _lengths(c):
    n = c["batch"]
    lens = [c["len_hi"] if n == 1 else c["len_lo"] + (c["len_hi"] - c["len_lo"]) * i // (n - 1) for i in range(n)]
    random.Random(7).shuffle(lens)
    return lens


def _masks(c):
    r = random.Random(11)
    out = np.zeros((c["layers"], c["q_heads"]), np.uint8)
    for l in range(c["layers"]):
        if c["call"] == "dense" or (c["first_dense"] and l == 0):
            out[l] = 1
        elif c["block"] == 64:  # whole KV groups
            g = c["q_heads"] // c["kv_heads"]
            for j in r.sample(range(c["kv_heads"]), max(1, min(c["kv_heads"] - 1, c["retrieval"] // g))):
                out[l, j * g:(j + 1) * g] = 1
        else:
            out[l, r.sample(range(c["q_heads"]), c["retrieval"])] = 1
    return out


def _units(c, length):
    return -(-length // c["block"])


def _budget(c, length):
    """Entries a set of the Top-k or Ratio rule holds for a sequence of this length."""
    n = min(c["k"], _units(c, length))
    if c["rule"] == "ratio":
        ppm = int(round(c["param"] * 1e6))
        n = min(n, max(1, -(-_units(c, length) * ppm // 1000000)))
    return n


def _set_rows(c, length):
    """Cache rows a sparse KV head reads (probability rules: up to the budget)."""
    return min(_budget(c, length) * c["block"], length)


def work(case):
    G = case["q_heads"] // case["kv_heads"]
    masks = _masks(case)
    rows = pairs = 0
    for m in masks:
        m = m.reshape(case["kv_heads"], G)
        for length in _lengths(case):
            n_set = _set_rows(case, length)
            rows += int(m.any(1).sum()) * length + int((m == 0).any(1).sum()) * n_set
            pairs += int(m.sum()) * length + int((m == 0).sum()) * n_set
    sets = 0 if case["call"] == "dense" else 2 * 4 * case["batch"] * case["kv_heads"] * case["k"]
    per_layer = 2 * 2 * case["batch"] * case["q_heads"] * D + sets
    if case["append"]:
        per_layer += 2 * 2 * 2 * case["batch"] * case["kv_heads"] * D
    return {"bytes": rows * 2 * 2 * D + case["layers"] * per_layer, "flops": pairs * 4 * D}


def tolerance(case):
    # out: bf16, fp32 sums (two correct implementations differ in the last bit of some values); sets: whole
    # numbers, the same unless two scores tie within rounding
    return {"rel": 4e-3, "max": 2e-2, "differ": 0.0}


# ------------------------------------------------------------------ values


def _view(cache, c):
    """[..., B, H_kv, L, 128] of a cache in either layout."""
    return cache.transpose(-3, -2) if c["token_major"] else cache


def _plant(c, kc, q, mask, lens, gen):
    """Adds query-aligned key rows at `planted` positions of every (sequence, KV head), in place."""
    B, H, P = c["batch"], c["kv_heads"], min(c["planted"], min(_lengths(c)))
    G = c["q_heads"] // H
    m = torch.from_numpy(mask.reshape(H, G).argmax(1)).to(DEV)  # the first retrieval head, else head 0
    qs = q.view(B, H, G, D)[:, torch.arange(H, device=DEV), m].float()
    qn = qs.norm(dim=-1, keepdim=True)
    r = torch.arange(1, P + 1, device=DEV, dtype=torch.float32)
    a = (3.0 * math.sqrt(D) - c["zipf"] * r.log()) / qn if c["zipf"] > 0 else torch.full((B, H, P), 3.0, device=DEV)
    u = torch.rand((B, H, c["len_hi"]), device=DEV, generator=gen)
    u.masked_fill_(torch.arange(c["len_hi"], device=DEV) >= lens.view(B, 1, 1), -1.0)
    pos = u.topk(P, dim=-1).indices
    b = torch.arange(B, device=DEV).view(B, 1, 1)
    h = torch.arange(H, device=DEV).view(1, H, 1)
    kc[b, h, pos] = (kc[b, h, pos].float() + (a * math.sqrt(D)).unsqueeze(-1) * (qs / qn).unsqueeze(2)).to(kc.dtype)


def _inherited(c, kc, gen):
    """Sets that an independently drawn query selects on this cache, ascending, -1 padded."""
    B, H, k = c["batch"], c["kv_heads"], c["k"]
    out = torch.full((B, H, k), -1, dtype=torch.int32, device=DEV)
    q = torch.randn((B, H, D, 1), device=DEV, generator=gen)
    for b, length in enumerate(_lengths(c)):
        n = _budget(c, length)
        for h in range(H):
            s = (kc[b, h, :length].float() @ q[b, h]).squeeze(-1)
            if c["block"] == 64:
                s = torch.nn.functional.pad(s, (0, -length % 64), value=-math.inf).view(-1, 64).amax(1)
            out[b, h, :n] = s.topk(n).indices.sort().values.to(torch.int32)
    return out


def prepare(case, seed):
    c = case
    B, H, n = c["batch"], c["kv_heads"], c["layers"]
    gen = torch.Generator(DEV)
    gen.manual_seed(seed)
    masks = _masks(c)
    lens = torch.tensor(_lengths(c), dtype=torch.int32, device=DEV)
    dims = (n, B, c["cap"], H, D) if c["token_major"] else (n, B, H, c["cap"], D)
    k_cache, v_cache = (torch.empty(dims, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    q = torch.randn((n, B, c["q_heads"], D), dtype=torch.bfloat16, device=DEV, generator=gen)
    for l in range(n):
        k_cache[l].normal_(generator=gen)
        v_cache[l].normal_(generator=gen)
        _plant(c, _view(k_cache[l], c), q[l], masks[l], lens, gen)
    s = {"case": c, "masks": masks, "lens": lens, "q": q, "k": k_cache, "v": v_cache, "idx_in": None}
    if not masks[0].all():
        s["idx_in"] = _inherited(c, _view(k_cache[0], c), gen)
    if c["append"]:
        s["k_new"], s["v_new"] = (torch.randn((n, B, H, D), dtype=torch.bfloat16, device=DEV, generator=gen)
                                  for _ in range(2))
    if torch.cuda.is_available():
        kv = _view(k_cache[0], c)
        s["shape"] = lb.make_shape(B, c["q_heads"], H, c["cap"], c["k"], kv=kv,
                                   keep_ppm=int(round(c["param"] * 1e6)) if c["rule"] == "ratio" else 0,
                                   block_size=c["block"], prob_rule=RULES[c["rule"]],
                                   prob_param=c["param"] if RULES[c["rule"]] else 0.0)
        s["ctx"] = lb.Context(0)
        if c["call"] == "step":
            s["ctx"].set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if c["phased"] else lb.STEP_LAYERWISE)
        if c["call"] != "static":
            s["ws"] = lb.alloc_workspace(s["shape"], DEV, n_layers={"loop": 2, "step": n}.get(c["call"], 1))
        s["out"] = torch.zeros_like(q)
        s["idx"] = torch.zeros((n if c["call"] == "loop" else 1, B, H, c["k"]), dtype=torch.int32, device=DEV)
        for key in ("q", "k", "v", "k_new", "v_new", "out", "idx"):  # what the calls take: one tensor per layer
            if key in s:
                s[key + "s"] = list(s[key].unbind(0))
    return s


def run(state):
    s, c, ctx = state, state["case"], state["ctx"]
    if c["call"] == "layer":
        ctx.decode_attn(s["shape"], s["qs"][0], s["ks"][0], s["vs"][0], s["masks"][0], s["idx_in"], s["outs"][0],
                        s["idxs"][0], s["lens"], s["ws"])
    elif c["call"] == "static":
        ctx.decode_attn_static(s["shape"], s["qs"][0], s["ks"][0], s["vs"][0], s["masks"][0], s["idx_in"], s["outs"][0],
                               s["idxs"][0], s["lens"])
    elif c["call"] == "loop":
        idx = s["idx_in"]
        for l in range(c["layers"]):
            ctx.decode_attn_deferred(s["shape"], s["qs"][l], s["ks"][l], s["vs"][l], s["masks"][l], idx, s["outs"][l],
                                     s["idxs"][l], s["lens"], s["ws"])
            idx = s["idxs"][l]
        ctx.select_flush()
    elif c["call"] == "step" and c["append"]:
        ctx.decode_step_append(s["shape"], s["qs"], s["k_news"], s["v_news"], s["ks"], s["vs"], s["masks"], s["idx_in"],
                               s["outs"], s["idxs"][0], s["lens"], s["ws"])
    elif c["call"] == "step":
        ctx.decode_step(s["shape"], s["qs"], s["ks"], s["vs"], s["masks"], s["idx_in"], s["outs"], s["idxs"][0],
                        s["lens"], s["ws"])
    else:
        ctx.dense_decode_attn(s["shape"], s["qs"][0], s["ks"][0], s["vs"][0], s["outs"][0], s["lens"], s["ws"])
        return {"out": s["out"]}
    if c["append"]:  # the caches are updated state
        return {"out": s["out"], "idx": s["idx"], "k_cache": s["k"], "v_cache": s["v"]}
    return {"out": s["out"], "idx": s["idx"]}


# ------------------------------------------------------------------ the same in 64 bits


def _select(c, score, length):
    """The set of one (sequence, KV head) from its pooled logits: ascending, -1 padded."""
    if c["block"] == 64:
        rank = torch.nn.functional.pad(score, (0, -length % 64), value=-math.inf).view(-1, 64).amax(1)
    else:
        rank = score
    order = rank.sort(descending=True, stable=True)  # ties: the lower position first
    n = _budget(c, length)
    if c["rule"] == "threshold":
        n = min(n, max(1, int((score.softmax(0) > c["param"]).sum())))
    elif c["rule"] == "top_p":
        mass = score.softmax(0)[order.indices].cumsum(0)
        n = min(n, int((mass < c["param"]).sum()) + 1)
    out = torch.full((c["k"],), -1, dtype=torch.int32, device=DEV)
    out[:n] = order.indices[:n].sort().values.to(torch.int32)
    return out


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    H, G = c["kv_heads"], c["q_heads"] // c["kv_heads"]
    lens, out, sets = _lengths(c), torch.zeros(s["q"].shape, dtype=torch.float64, device=DEV), s["idx_in"]
    every = []
    for l in range(c["layers"]):
        kl, vl = _view(s["k"][l], c), _view(s["v"][l], c)
        if c["append"]:
            for b, length in enumerate(lens):
                kl[b, :, length - 1] = s["k_new"][l, b]
                vl[b, :, length - 1] = s["v_new"][l, b]
        new = sets.clone() if sets is not None else torch.empty_like(s["idx"][0])
        for b, length in enumerate(lens):
            for h in range(H):
                heads = range(h * G, (h + 1) * G)
                dense = [i for i in heads if s["masks"][l, i]]
                sparse = [i for i in heads if not s["masks"][l, i]]
                if dense:
                    logit = (kl[b, h, :length].double() @ s["q"][l, b, dense].double().T) / math.sqrt(D)
                    out[l, b, dense] = logit.softmax(0).T @ vl[b, h, :length].double()
                    if c["call"] != "dense":
                        new[b, h] = _select(c, logit.mean(1), length)
                if sparse:
                    at = sets[b, h][sets[b, h] >= 0].long()
                    if c["block"] == 64:
                        at = (at.view(-1, 1) * 64 + torch.arange(64, device=DEV)).view(-1)
                        at = at[at < length]
                    logit = (kl[b, h, at].double() @ s["q"][l, b, sparse].double().T) / math.sqrt(D)
                    out[l, b, sparse] = logit.softmax(0).T @ vl[b, h, at].double()
        sets = new
        every.append(new)
    if c["call"] == "dense":
        return {"out": out}
    got = {"out": out, "idx": torch.stack(every) if c["call"] == "loop" else sets.unsqueeze(0)}
    if c["append"]:
        got.update(k_cache=None, v_cache=None)
    return got

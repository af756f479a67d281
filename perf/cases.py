"""What a serving program has this library do, as measurable cases.

A case is one call sequence of the public binding over a stack of attention layers:

  step "turn"    a new conversation turn: rebase, then per layer load the kept history from the tier, append the new
                 turn and save it to the tier, attend the new tokens over [kept history | new]; join at the end
  step "decode"  one decoding step of a running batch: rebase with one new token per conversation, then per layer
                 append, attend over the whole context, write the token's keys and values back to the tier

Model shapes and length mixes are those of the repository's five configurations, of its benchmark's decode leg and of
its tests; a case holds as many layers as keep a pass and three resident copies of its tensors affordable (every layer
has buffers of its own).  Values are ~N(0, 1) in bf16 and come from the seed; lengths and page tables are part of the
case, so that every seed has the same amount of work.  The context (ca_ctx), the pools, the tier and the pointer arrays
are what a serving program keeps between turns.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2403_19708_amd as ca

PAGE = 16

_BASE = dict(step="turn", layers=1, batch=1, q_heads=32, kv_heads=32, head_dim=128, rope_style=0, window=4096, tier="hbm",
             overflow="none", hist_lo=0, hist_hi=0, hist_mid=0, new_lo=1, new_hi=1, new_mid=0, lengths=0)


def _case(name: str, **kw) -> dict:
    return dict(_BASE, name=name, **kw)


def listed() -> list:
    return [
        # the smallest turn the configurations name: one conversation, four heads, 256 saved tokens and 32 new ones,
        # tier in pinned host memory; all latency
        _case("tiny_turn", q_heads=4, kv_heads=4, head_dim=64, hist_lo=256, hist_hi=256, new_lo=32, new_hi=32, tier="pinned"),
        # decoding on the 7B-shaped multi-head stack (the benchmark's decode leg): 16 conversations, whole stack
        _case("decode_mha_b16", step="decode", layers=32, batch=16, hist_lo=1000, hist_hi=1600),
        # decoding on the 70B-shaped grouped-query stack: a full batch at the lengths of configuration 5
        _case("decode_gqa_b64", step="decode", layers=8, batch=64, q_heads=64, kv_heads=8, window=8192, hist_lo=1024, hist_hi=4096),
        # one user waiting for tokens on the 70B-shaped stack, whole stack: few bytes per layer, many calls
        _case("decode_gqa_b1", step="decode", layers=80, batch=1, q_heads=64, kv_heads=8, window=8192, hist_lo=2777, hist_hi=2777),
        # configuration 2: an ordinary batch of turns, multi-head, tier in HBM
        _case("turn_mha_b16", layers=4, batch=16, hist_lo=512, hist_hi=2048, new_lo=32, new_hi=256),
        # configuration 3: 40 heads, many ragged conversations with mostly short new turns
        _case("turn_mha_b32_ragged", layers=4, batch=32, q_heads=40, kv_heads=40, hist_lo=64, hist_hi=3800, hist_mid=1097,
              new_lo=8, new_hi=512, new_mid=90),
        # configuration 4: every conversation overflows its window and keeps the most recent half
        _case("turn_overflow_b8", layers=4, batch=8, hist_lo=4700, hist_hi=5500, new_lo=64, new_hi=512, overflow="recent"),
        # configuration 5, tier in HBM: grouped-query attention, compute-bound, the largest batch
        _case("turn_gqa_b64", layers=2, batch=64, q_heads=64, kv_heads=8, window=8192, hist_lo=1024, hist_hi=4096, new_lo=64, new_hi=512),
        # configuration 5 with the tier where the method keeps it, pinned host memory: bound by the host link
        _case("turn_gqa_b64_pinned", layers=2, batch=64, q_heads=64, kv_heads=8, window=8192, hist_lo=1024, hist_hi=4096, new_lo=64,
              new_hi=512, tier="pinned"),
        # one conversation with a long document behind it
        _case("turn_gqa_b1_long", layers=8, batch=1, q_heads=64, kv_heads=8, window=65536, hist_lo=31003, hist_hi=31003, new_lo=301, new_hi=301),
        # first turns: nothing saved yet, prompts of very different length; 64-wide heads, interleaved rotary pairs
        _case("first_turn_b16_d64", layers=4, batch=16, q_heads=32, kv_heads=4, head_dim=64, rope_style=1, new_lo=128, new_hi=2048),
        # a small batch whose discarding lists keep the first tokens and the most recent ones; tier in pinned host memory
        _case("turn_sinks_b4_pinned", layers=4, batch=4, window=2048, hist_lo=2000, hist_hi=2600, new_lo=48, new_hi=200,
              overflow="sinks", tier="pinned"),
    ]


# largest work of a drawn case, in seconds at rates the card and the host link sustain (what the largest listed cases take)
_MOST_SECONDS = {"hbm": 4.0e-3, "pinned": 2.0e-2}
_MODELS = ((32, 32, 128), (40, 40, 128), (64, 8, 128), (32, 4, 64), (8, 2, 128), (4, 4, 64))


def _log_int(rng, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    q_heads, kv_heads, head_dim = rng.choice(_MODELS)
    c = dict(_BASE, q_heads=q_heads, kv_heads=kv_heads, head_dim=head_dim, rope_style=rng.randrange(2), window=8192,
             batch=_log_int(rng, 1, 64), lengths=rng.randrange(1 << 20))
    kind = rng.choice(("turn", "turn", "turn", "overflow", "first", "long", "decode", "decode"))
    hist = _log_int(rng, 100, 4000)
    c["hist_lo"], c["hist_hi"] = hist, _log_int(rng, hist, 4100)
    if kind == "decode":
        c.update(step="decode")
    else:
        new = _log_int(rng, 8, 400)
        c["new_lo"], c["new_hi"] = new, _log_int(rng, new, 520)
        c["tier"] = "pinned" if rng.random() < 0.2 else "hbm"
        if kind == "overflow":
            c.update(window=4096, hist_lo=4000, hist_hi=_log_int(rng, 4000, 5500), overflow=rng.choice(("recent", "sinks")))
        elif kind == "first":
            c.update(hist_lo=0, hist_hi=0, new_hi=_log_int(rng, new, 2048))
        elif kind == "long":
            c.update(batch=rng.choice((1, 2)), window=65536, hist_lo=_log_int(rng, 4000, 31000), hist_hi=31003)
    while _seconds(c) > _MOST_SECONDS[c["tier"]] and c["batch"] > 1:
        c["batch"] = (c["batch"] + 1) // 2
    c["layers"] = max(1, min(_log_int(rng, 1, 32), int(_MOST_SECONDS[c["tier"]] / _seconds(c))))
    return c


def _seconds(case: dict) -> float:
    w = work(case)
    return max(w["bytes"] / (4e10 if case["tier"] == "pinned" else 4e12), w["flops"] / 0.7e15)


def _lengths(case: dict):
    """hist_len, keep (keep_start array or list of kept ranges), kept tokens, new_len of every conversation"""
    rng = np.random.default_rng([case["lengths"], 77])
    b = case["batch"]

    def lens(lo, hi, mid, sigma):
        if mid:
            return np.clip(np.rint(rng.lognormal(math.log(mid), sigma, b)), lo, hi).astype(np.int32)
        return rng.integers(lo, hi + 1, b).astype(np.int32)

    hist = lens(case["hist_lo"], case["hist_hi"], case["hist_mid"], 0.6)
    new = lens(case["new_lo"], case["new_hi"], case["new_mid"], 0.8)
    over = hist.astype(np.int64) + new > case["window"]
    budget = np.where(over, np.maximum(0, case["window"] // 2 - new), hist).astype(np.int64)
    return hist, new, np.minimum(budget, hist)


def work(case: dict) -> dict:
    """Turn: kept history, new keys/values and queries in; pool, tier rows and outputs out.  Decode: the context (which is
    in the pool already), the new token and its query in; its pool slot, tier row and output out."""
    _, new, kept = _lengths(case)
    n, k = float(new.sum()), float(kept.sum())
    kv = 2.0 * case["kv_heads"] * case["head_dim"] * 2
    qo = 2.0 * case["q_heads"] * case["head_dim"] * 2
    moved = kv * (k + 3 * n) if case["step"] == "decode" else kv * (2 * k + 3 * n)
    newf, keptf = new.astype(np.float64), kept.astype(np.float64)
    flops = 4.0 * case["head_dim"] * case["q_heads"] * float(np.sum(newf * keptf + newf * (newf + 1) / 2))
    return {"bytes": case["layers"] * (moved + qo * n), "flops": case["layers"] * flops}


def tolerance(case: dict):
    # attention outputs are bf16 with bf16 operands in both products; pool and tier contents are whole numbers and exact
    return {"rel": 1e-2, "max": 0.2}


def prepare(case: dict, seed: int) -> dict:
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    bf = torch.bfloat16
    L, B, D, Hq, Hkv = case["layers"], case["batch"], case["head_dim"], case["q_heads"], case["kv_heads"]
    decode = case["step"] == "decode"

    def normal(*shape):
        return torch.empty(shape, dtype=bf, device=dev).normal_(generator=gen)

    hist, new, kept = _lengths(case)
    keep_start, keep_ranges = np.zeros(B, np.int32), None
    if case["overflow"] == "sinks":
        keep_ranges = ca.truncate_plan_sinks(hist, new, case["window"], 0.5, n_sink=4)
    elif case["overflow"] == "recent":
        keep_start = ca.truncate_plan(hist, new, case["window"], 0.5)
    context = kept + new
    pages = (context + PAGE - 1) // PAGE
    num_pages = int(pages.sum()) + 8
    perm = np.random.default_rng([case["lengths"], 78]).permutation(num_pages).astype(np.int32)
    table = np.full((B, int(pages.max())), -1, np.int32)
    at = 0
    for c in range(B):
        table[c, :pages[c]] = perm[at:at + pages[c]]
        at += int(pages[c])

    total_q = int(new.sum())
    pool = (L, num_pages, Hkv, PAGE, D)
    # decoding finds its context in the pool; a turn finds its history in the tier
    k_pool, v_pool = (normal(*pool), normal(*pool)) if decode else (torch.zeros(pool, dtype=bf, device=dev) for _ in range(2))
    rows = np.ones(B, np.int64) if decode else hist.astype(np.int64) + new
    shape = (L, int(rows.sum()), Hkv, D)
    tier_k, tier_v = normal(*shape), normal(*shape)
    if case["tier"] == "pinned":
        host = [torch.empty(shape, dtype=bf, pin_memory=True) for _ in range(2)]
        for h, t in zip(host, (tier_k, tier_v)):
            h.copy_(t)
        tier_k, tier_v = host
    first = np.concatenate([[0], np.cumsum(rows)[:-1]]) * (Hkv * D * 2)

    def pointers(t):
        return [ca.pointer_array([t[l].data_ptr() + int(o) for o in first]) for l in range(L)]

    ctx = ca.Context(ca.Config(n_layers=L, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, max_positions=case["window"], rope_style=case["rope_style"],
                               pipeline_depth=2, max_seqs=B, max_batch_kv_tokens=int(context.sum()) + 64, max_batch_q_tokens=total_q + 16,
                               require_load=0 if decode else 1))
    return dict(decode=decode, ctx=ctx, layers=L, hist=hist, keep_start=keep_start, keep_ranges=keep_ranges, new=new, table=table, num_pages=num_pages,
                k_pool=k_pool, v_pool=v_pool, tier_k=tier_k, tier_v=tier_v, ptr_k=pointers(tier_k), ptr_v=pointers(tier_v),
                pools=[(k_pool[l], v_pool[l]) for l in range(L)], q=list(normal(L, total_q, Hq, D)), new_k=list(normal(L, total_q, Hkv, D)),
                new_v=list(normal(L, total_q, Hkv, D)), out=torch.zeros((L, total_q, Hq, D), dtype=bf, device=dev), scale=1.0 / math.sqrt(D),
                end=hist + 1, offset=np.zeros(B, np.int64))


def run(state: dict):
    s, ctx = state, state["ctx"]
    stream = torch.cuda.current_stream()
    layers, out = s["layers"], s["out"]
    ctx.rope_rebase(s["hist"], s["keep_start"], s["new"], s["table"], s["num_pages"], stream, keep_ranges=s["keep_ranges"])
    if s["decode"]:
        for l in range(layers):
            k_pool, v_pool = s["pools"][l]
            ctx.kv_append_layer(l, s["new_k"][l], s["new_v"][l], k_pool, v_pool, stream)
            ctx.cached_prefill_attn(l, s["q"][l], k_pool, v_pool, out[l], s["scale"], stream)
            ctx.kv_save_layer(l, k_pool, v_pool, s["ptr_k"][l], s["ptr_v"][l], tok_begin=s["hist"], tok_end=s["end"],
                              dst_tok_offset=s["offset"], after_stream=stream)
    else:
        for l in range(layers):
            ctx.kv_load_layer(l, s["ptr_k"][l], s["ptr_v"][l], *s["pools"][l])
        for l in range(layers):
            k_pool, v_pool = s["pools"][l]
            ctx.kv_append_save_layer(l, s["new_k"][l], s["new_v"][l], k_pool, v_pool, s["ptr_k"][l], s["ptr_v"][l], stream)
            ctx.cached_prefill_attn(l, s["q"][l], k_pool, v_pool, out[l], s["scale"], stream)
    ctx.join(stream)
    return {"out": out, "k_pool": s["k_pool"].view(torch.int16), "v_pool": s["v_pool"].view(torch.int16),
            "tier_k": s["tier_k"].view(torch.int16), "tier_v": s["tier_v"].view(torch.int16)}

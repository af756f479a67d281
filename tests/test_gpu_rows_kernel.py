"""The kernel for few stacked query rows per (conversation, kv head) (3 to 32: grouped-query decode steps, very short
turns): outputs against the oracle where it can go wrong -- one and two 16-row blocks, contexts that end anywhere in a page
or have fewer pages than a workgroup has wavefronts, rows that see different ends, both head sizes and pair conventions,
key splitting on and off, runs of pages that cover many units and units cut into many runs -- and repeatedly on one plan
(the merge counters must be back at zero)."""
import numpy as np
import pytest
import torch

import oracle
from harness import Case, GpuRun, torch_to_bits
from synth import bf16_bits_to_f64, f32_to_bf16_bits
from test_gpu_parity import check_contract, check_tight

pytestmark = pytest.mark.gpu


def run_case(case, calls=1, tight=True, **knobs):
    run = GpuRun(case, tier="device", **knobs)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        bits = []
        for _ in range(calls):
            run.out[0].zero_()
            run.attn(0)
            run.finish()
            bits.append(torch_to_bits(run.out[0]).copy())
        for c in range(case.B):
            check_contract(run.out_f64(0, c), case.oracle_out(0, c), c)
            if tight:
                check_tight(run.out_f64(0, c), case.oracle_out(0, c), int(case.n_keep[c]), c)
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        return items, bits
    finally:
        run.close()


SHAPES = [  # Hq, Hkv, D, style, new tokens: rows = new * Hq / Hkv
    (8, 1, 128, 0, 1), (8, 2, 128, 1, 1), (16, 1, 64, 0, 1), (32, 1, 128, 0, 1), (4, 4, 128, 0, 32), (4, 4, 64, 1, 17),
    (3, 1, 64, 1, 1), (8, 1, 128, 0, 4), (6, 2, 64, 0, 3),
]


@pytest.mark.parametrize("split", [0, 1], ids=["split", "whole"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "hq%d-hkv%d-d%d-style%d-new%d" % s)
def test_ends_and_rows(shape, split):
    Hq, Hkv, D, style, new = shape
    hist = [0, 1, 15, 16, 17, 63, 200, 333, 1000, 1027]
    keep = [0, 0, 3, 0, 16, 0, 77, 0, 500, 0]
    lens = [max(1, new - c % 3) for c in range(len(hist))]
    case = Case(hist, lens, keep, Hq, Hkv, D, seed=60 + D + style, style=style, window=2048)
    run_case(case, attn_split=split)


@pytest.mark.parametrize("shape", [(8, 1, 128, 0, 1), (16, 2, 64, 1, 4)], ids=["one-block", "two-blocks"])
def test_units_cut_into_many_runs(shape):
    Hq, Hkv, D, style, new = shape
    case = Case([9000, 700, 4100], [new] * 3, [0, 0, 37], Hq, Hkv, D, seed=62, style=style, window=16384)
    items, bits = run_case(case, calls=3)
    assert (items[:, 6] >= 0).sum() >= 8
    assert np.array_equal(bits[0], bits[1]) and np.array_equal(bits[0], bits[2])


@pytest.mark.parametrize("pages, shares", [(3, 0), (19, 0), (20, 5), (21, 6), (250, 16), (272, 17), (600, 25), (1100, 35)])
@pytest.mark.parametrize("shape", [(8, 1, 128, 0, 1), (16, 2, 64, 1, 4)], ids=["one-block", "two-blocks"])
def test_shares_of_one_conversation(shape, pages, shares):
    """Units below and above the least that is cut, shares that end in the middle of a wavefront's turn, and merges of one batch of
    eight shares, two, and more than the two in flight at once."""
    Hq, Hkv, D, style, new = shape
    case = Case([16 * pages - new - 5], [new], [0], Hq, Hkv, D, seed=66 + pages, style=style, window=32768)
    items, bits = run_case(case, calls=2)
    assert (items[:, 6] >= 0).sum() == shares * Hkv
    assert np.array_equal(bits[0], bits[1])


@pytest.mark.parametrize("split", [0, 1], ids=["split", "whole"])
@pytest.mark.parametrize("shape", [(64, 16, 64, 0, 1), (64, 8, 64, 1, 3), (64, 8, 128, 0, 1), (64, 8, 128, 1, 1), (32, 4, 128, 0, 4), (24, 8, 128, 1, 6)],
                         ids=lambda s: "hq%d-hkv%d-d%d-style%d-new%d" % s)
def test_runs_over_many_units(shape, split):
    """Enough to stream for two workgroups of four wavefronts per compute unit (16384 pages over all kv heads): most runs
    cover a whole unit and a share on either side.  Sampled conversations and heads against the oracle; the static entry
    point gives the same bits."""
    Hq, Hkv, D, style, new = shape
    pages, hist, rng = 0, [], np.random.default_rng(63)
    while pages * Hkv < 16500:
        hist.append(int(rng.integers(100, 2000 if D == 128 else 700)))
        pages += (hist[-1] + 15) // 16
    lens = [max(1, new - c % 3) for c in range(len(hist))]
    case = Case(hist, lens, [0] * len(hist), Hq, Hkv, D, seed=63, style=style, window=2048)
    run = GpuRun(case, tier="device", attn_split=split)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        bits = []
        s = 1.0 / np.sqrt(D)
        for call in (run.ctx.cached_prefill_attn, run.ctx.cached_prefill_attn, run.ctx.cached_prefill_attn_static):
            run.out[0].view(torch.int16).fill_(0x7FC0)          # NaN pattern: every element must be rewritten
            call(0, run.q[0], run.k_pool[0], run.v_pool[0], run.out[0], s)
            run.finish()
            bits.append(torch_to_bits(run.out[0]).copy())
        assert np.array_equal(bits[0], bits[1]) and np.array_equal(bits[0], bits[2])
        assert not np.any(bits[0] == 0x7FC0)
        shares = run.ctx.rebase_read(6).reshape(-1, 8)[:, 6]
        assert (shares < 0).any() and (shares >= 0).any() == (split == 0)
        ends = [int(np.argmax(hist)), int(np.argmin(hist)), 0, case.B - 1]
        for c in ends + [int(x) for x in rng.choice(case.B, 4, replace=False)]:
            heads = [int(h) for h in rng.choice(Hq, 6, replace=False)]
            got, want = run.out_f64(0, c)[:, heads], case.oracle_out(0, c, heads=heads)
            check_contract(got, want, c)
            check_tight(got, want, int(case.n_keep[c]), c)
    finally:
        run.close()


def test_peaky_scores():
    case = Case([500, 77], [1, 1], [0, 0], 8, 1, 128, seed=64, window=1024, q_scale=2.0)
    run_case(case, tight=False)      # (softmax on a few keys: the rounding of the rotated operands is over the tighter bar)


def test_the_two_entry_points_at_once():
    """an ordinary and a static call of one context on two streams, again and again: scratch and counters are their own"""
    case = Case([9000, 700, 4100], [1] * 3, [0, 0, 37], 8, 1, 128, seed=65, window=16384)
    run = GpuRun(case, tier="device")
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        run.attn(0)
        run.finish()
        want = torch_to_bits(run.out[0]).copy()
        streams = torch.cuda.Stream(), torch.cuda.Stream()
        outs = [[torch.zeros_like(run.out[0]) for _ in range(50)] for _ in streams]
        torch.cuda.synchronize()
        s = 1.0 / np.sqrt(case.head_dim)
        for a, b in zip(*outs):
            run.ctx.cached_prefill_attn(0, run.q[0], run.k_pool[0], run.v_pool[0], a, s, streams[0])
            run.ctx.cached_prefill_attn_static(0, run.q[0], run.k_pool[0], run.v_pool[0], b, s, streams[1])
        torch.cuda.synchronize()
        for out in outs[0] + outs[1]:
            assert np.array_equal(torch_to_bits(out), want)
    finally:
        run.close()


@pytest.mark.parametrize("hist, batch, D, style", [(2777, 1, 128, 0), (6000, 1, 64, 1), (600, 8, 128, 1), (250, 8, 128, 0)], ids=["shares", "long", "batch", "whole"])
def test_every_new_maximum_of_a_row_has_an_exact_probability(hist, batch, D, style):
    """In 64 bits over the operands the kernel rounds (rotated keys, rotated and scaled queries, probabilities against the maximum so far
    of the pages a wavefront has seen), the kernel's output differs by the rounding of the output alone: relative, 2^-8 / sqrt(3) times
    the root mean square 0.74 of 1 / mantissa, 0.00166.  A tenth is for probabilities that fp32 scores round the other way.
    Against a maximum that stands still the probabilities would be rounded at other places, by 0.00166 each."""
    G = 8
    case = Case([hist + 3 * c for c in range(batch)], [1] * batch, [0] * batch, G, 1, D, seed=69 + D, style=style, window=8192)
    run = GpuRun(case, tier="device")
    w = bf16_bits_to_f64
    diff = total = 0.0
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        run.attn(0)
        run.finish()
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        fold = np.float32(1.0 / np.sqrt(D)) * np.float32(1.4426950408889634)
        for c in range(batch):
            n = int(case.n_keep[c])
            K, V = (np.concatenate([w(case.tensor(0, x + "_hist", c)), w(case.tensor(0, x + "_new", c))])[:, 0] for x in "kv")
            Kr = w(f32_to_bf16_bits(np.array([oracle.rope(K[t], t, style=style) for t in range(n + 1)]).astype(np.float32)))
            Qr = np.array([oracle.rope(q, n, style=style) for q in w(case.tensor(0, "q", c))[0]])
            S = w(f32_to_bf16_bits(Qr.astype(np.float32) * fold)) @ Kr.T
            P = np.zeros_like(S)
            for begin, end, part in items[items[:, 0] == c][:, 4:7]:
                waves = 4 if part >= 0 else 8
                for wave in range(waves):
                    top = np.full(G, -np.inf)
                    for at in range(int(begin) + 16 * wave, min(int(end), n + 1), 16 * waves):
                        s = S[:, at:min(at + 16, int(end), n + 1)]
                        top = np.maximum(top, s.max(1))
                        p = w(f32_to_bf16_bits(np.exp2(s - top[:, None]).astype(np.float32)))
                        P[:, at:at + s.shape[1]] = p * np.exp2(top - S.max(1))[:, None]
            want = P @ V / P.sum(1, keepdims=True)
            diff += np.sum((run.out_f64(0, c)[0] - want) ** 2)
            total += np.sum(want ** 2)
    finally:
        run.close()
    assert (items[:, 6] >= 0).any() == (hist > 300)
    assert np.sqrt(diff / total) < 1.1 * 0.00166

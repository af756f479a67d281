"""The matrix-core tile kernel where its schedule can go wrong: contexts that end around the edges of key tiles and of the
rings (one to six tiles, one key more or less), both groups of wavefronts live or only the first, contexts that move the window
of page ids, keys that are not finite, and rows whose scores rise so fast along the context that the reference has to move
inside interior tiles, by more than a probability could hold."""
import numpy as np
import pytest
import torch

import oracle
from harness import Case, GpuRun, torch_to_bits
from test_gpu_parity import check_contract, check_tight
from synth import bf16_bits_to_f64, f32_to_bf16_bits

pytestmark = pytest.mark.gpu

SHAPES = [(128, 0), (128, 1), (64, 0), (64, 1)]


def outputs(case, **knobs):
    run = GpuRun(case, tier="device", attn_variant=2, **knobs)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        run.attn(0)
        run.finish()
        return [run.out_f64(0, c) for c in range(case.B)]
    finally:
        run.close()


@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "d%d-style%d" % s)
def test_tile_edges(shape, rows, prerotate):
    D, style = shape
    hist = [0, 1, 31, 32, 63, 64, 95, 127, 128, 191, 192, 193, 255, 256, 257, 319, 320, 383, 385]
    new = [1 + (37 * c) % 70 for c in range(len(hist))]                 # 4 to 280 stacked rows
    case = Case(hist, new, [0] * len(hist), 8, 2, D, seed=70 + D + style, style=style, window=1024)
    got = outputs(case, attn_tile_rows=rows, attn_prerotate=prerotate, attn_split=1)
    for c in range(case.B):
        check_contract(got[c], case.oracle_out(0, c), c)
        check_tight(got[c], case.oracle_out(0, c), int(case.n_keep[c]), c)


@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "d%d-style%d" % s)
@pytest.mark.parametrize("G", [1, 3, 5, 40])
def test_rows_of_odd_groups(G, shape, rows, prerotate):
    """The 32 query rows of a wavefront start and end inside a token's group of heads, or lie in one or two of them"""
    D, style = shape
    new = [300 // G + 1, 7, 1]
    case = Case([70, 0, 130], new, [0, 0, 0], G, 1, D, seed=80 + D + style, style=style, window=1024)
    got = outputs(case, attn_tile_rows=rows, attn_prerotate=prerotate, attn_split=1)
    for c in range(case.B):
        check_contract(got[c], case.oracle_out(0, c), c)
        check_tight(got[c], case.oracle_out(0, c), int(case.n_keep[c]), c)


@pytest.mark.parametrize("steps", [[1.0, 40.0], [40.0, 1.0], [1.0, 4.0, 16.0, 64.0, 1.0]], ids=["jump", "fall", "stairs"])
@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("D", [64, 128])
def test_reference_moves(D, rows, prerotate, steps):
    """Keys whose length changes along the context by powers of four and more.  The largest scores are in the hundreds, so
    the rounding of the rotated operands decides between the largest of them: the oracle gets the rotated and rounded
    operands, the query with the softmax scale folded in (as in test_attention_peaky_softmax), and every element is compared."""
    case = Case([1500], [40], [0], 8, 1, D, seed=75, window=2048)
    w = bf16_bits_to_f64
    k = w(case.tensor(0, "k_hist", 0))
    factor = np.repeat(np.asarray(steps), -(-1500 // len(steps)))[:1500]
    scaled = (k * factor[:, None, None]).astype(np.float32)            # (times a power of two or 40: rounded once more below)
    case.data[(0, "k_hist", 0)] = (scaled.view(np.uint32) >> 16).astype(np.uint16)
    got = outputs(case, attn_tile_rows=rows, attn_prerotate=prerotate, attn_split=1)[0]
    K, V = (np.concatenate([w(case.tensor(0, f"{n}_hist", 0)), w(case.tensor(0, f"{n}_new", 0))]) for n in "kv")
    Q = w(case.tensor(0, "q", 0))
    Kr = w(f32_to_bf16_bits(np.array([[oracle.rope(K[t, 0], t)] for t in range(1540)]).astype(np.float32)))
    scale = np.float32(1.0 / np.sqrt(D))
    fold = scale * np.float32(1.4426950408889634)
    Qr = w(f32_to_bf16_bits(np.array([[oracle.rope(Q[j, h], 1500 + j) for h in range(8)] for j in range(40)]).astype(np.float32) * fold)) / np.float64(fold)
    want = oracle.attention_positions(Kr, V, Qr, np.zeros(1540), np.zeros(40), 1500)
    # Rotated in 32 bits and not in 64 an element that lies between two bf16 values may be rounded to the other one, which moves a
    # score by at most `shift`, the largest elements' product times 2^-8; the outputs then by that share of how far the values
    # lie from them.  (One element in 2^14 where the table rotates, one in 2^9 after fifty steps of the recurrence: most keys
    # have none, and it is hardly ever the largest.)  On the CPU, rows taken from the next token are over the bound in nine of
    # ten elements and more of every 32 rows.
    score = np.einsum("jhd,td->jht", Qr, Kr[:, 0]) * np.float64(scale)
    score = np.where(np.arange(1540) <= 1500 + np.arange(40)[:, None, None], score, -np.inf)
    p = np.exp(score - score.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    shift = 2.0 ** -8 * np.abs(Kr).max() * np.abs(Qr).max() * float(scale)
    spread = np.stack([np.einsum("ht,htd->hd", p[j], np.abs(V[None, :, 0] - want[j][:, None])) for j in range(40)])
    excess = np.abs(got - want) - (2.0 ** -7 * np.abs(want) + 6e-3 + shift * spread)
    assert (excess <= 0).all(), (excess.max(), shift, np.unravel_index(excess.argmax(), excess.shape))
    assert np.abs(got - want).mean() <= 2e-3 + shift * spread.mean() / 8


@pytest.mark.parametrize("split", [0, 1], ids=["split", "whole"])
@pytest.mark.parametrize("D, rows, heads, new", [(128, 256, (2, 1), 150), (128, 128, (2, 1), 80), (64, 128, (8, 1), 20), (64, 256, (8, 1), 36)])
def test_the_page_id_window_moves(D, rows, heads, new, split):
    """Contexts of 70000 tokens, keys rotated beforehand: a workgroup that walks all of them moves its window of page ids
    (2048, 32768 tokens) twice.  The last tile of rows leaves wavefronts (of the eight, the whole second group) without rows."""
    case = Case([70000, 300], [new, 9], [0, 7], *heads, D, seed=28, window=1 << 17, style=split)
    got = outputs(case, attn_tile_rows=rows, attn_prerotate=2, attn_split=split)
    sampled = [0, heads[0] - 1]
    for c in range(2):
        want = case.oracle_out(0, c, heads=sampled)
        check_contract(got[c][:, sampled], want, c)
        check_tight(got[c][:, sampled], want, int(case.n_keep[c]), c)


@pytest.mark.parametrize("bits", [0x7fc0, 0xffc0, 0x7f80, 0xff80], ids=["nan", "minus-nan", "inf", "minus-inf"])
@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("D, rows", [(128, 256), (128, 128), (64, 128)])
def test_keys_that_are_not_finite(D, rows, prerotate, bits):
    """One element of a key inside the history of one conversation and of a new key of another: what the rows that see it get is
    what the oracle gets (not a number, or the other keys' average where the score is minus infinity), and nobody else notices."""
    case = Case([700, 700, 700], [50, 50, 50], [0, 0, 0], 8, 2, D, seed=77, window=1024)
    for name, conv, token in (("k_hist", 0, 333), ("k_new", 1, 20)):
        t = case.tensor(0, name, conv).copy()
        t[token, 1, 5] = bits
        case.data[(0, name, conv)] = t
    got = outputs(case, attn_tile_rows=rows, attn_prerotate=prerotate, attn_split=1)
    for c in range(3):
        want = case.oracle_out(0, c)
        assert (np.isnan(got[c]) == np.isnan(want)).all()
        assert np.isnan(want).any() == (c < 2)
        check_contract(got[c][~np.isnan(want)], want[~np.isnan(want)], c)


@pytest.mark.parametrize("new, rows", [([256, 256], 128), ([256, 224], 256)], ids=["128", "256"])
def test_tiles_of_grouped_heads_of_64(new, rows):
    """The planner's own choice for keys rotated beforehand, on both sides of it: 32 row tiles of 256 for eight kv heads take
    128-row ones, 31 do not; either has its keys cut."""
    case = Case([6000, 2000], new, [0, 0], 64, 8, 64, seed=79, window=8192)
    run = GpuRun(case, tier="device")
    try:
        run.rebase()
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        items = items[items[:, 0] >= 0]
        assert items[:, 3].max() == rows and (items[:, 6] >= 0).any()
        run.load(0)
        run.append(0)
        run.attn(0)
        run.finish()
        sampled = [0, 29, 63]
        for c in range(2):
            got, want = run.out_f64(0, c)[:, sampled], case.oracle_out(0, c, heads=sampled)
            check_contract(got, want, c)
            check_tight(got, want, int(case.n_keep[c]), c)
    finally:
        run.close()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "d%d-style%d" % s)
@pytest.mark.parametrize("new", [[20] * 15 + [129], [20] * 14 + [128] * 2, [129] * 16, [20] * 11 + [129]],
                         ids=["mixed", "short", "long", "few"])
def test_tile_rows_of_a_batch(shape, new):
    """128-row tiles for a batch with a longer turn among short ones, 256-row tiles where all are longer or the 128-row ones
    would not fill two places of every compute unit (12 conversations of 32 heads: 416 tiles)."""
    D, style = shape
    hist = [(53 * c) % 200 for c in range(len(new))]
    case = Case(hist, new, [0] * len(new), 32, 32, D, seed=90 + D + style, style=style, window=512)
    run = GpuRun(case, tier="device", attn_variant=2, attn_prerotate=1)
    try:
        run.rebase()
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        most = items[items[:, 0] >= 0][:, 3].max()          # rows of the largest item
        run.load(0)
        run.append(0)
        run.attn(0)
        run.finish()
        got = [run.out_f64(0, c) for c in range(case.B)]
    finally:
        run.close()
    full = 2 * torch.cuda.get_device_properties(0).multi_processor_count <= 32 * sum(-(-n // 128) for n in new)
    assert most == (128 if min(new) < 128 and full else 129)
    for c in (0, len(new) - 1):
        check_contract(got[c], case.oracle_out(0, c), c)
        check_tight(got[c], case.oracle_out(0, c), int(case.n_keep[c]), c)


@pytest.mark.parametrize("D, heads, batch, new", [(128, 32, 9, 140), (64, 40, 8, 200), (128, 48, 12, 60)], ids=["rows256", "heads64", "rows128"])
def test_only_the_last_round_is_cut(D, heads, batch, new):
    """A few more row tiles than workgroups fit the compute units: whole tiles first, the ones left over in shares.  Sampled heads
    against the oracle; the entry point that allocates nothing takes the plan and gives the same bits."""
    hist = [1500 + 37 * c for c in range(batch)]
    case = Case(hist, [new - c for c in range(batch)], [0] * batch, heads, heads, D, seed=90 + D, window=4096)
    run = GpuRun(case, tier="device")
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        items = items[items[:, 0] >= 0]
        shares = items[items[:, 6] >= 0]
        assert 0 < len(shares) < len(items) and len(items) - len(shares) >= 256
        assert (shares[:, 4] % 64 == 0).all() and (shares[:, 5] - shares[:, 4] >= 256).all()
        bits = []
        for call in (run.ctx.cached_prefill_attn, run.ctx.cached_prefill_attn_static):
            run.out[0].view(torch.int16).fill_(0x7FC0)
            call(0, run.q[0], run.k_pool[0], run.v_pool[0], run.out[0], 1.0 / np.sqrt(D))
            run.finish()
            bits.append(torch_to_bits(run.out[0]).copy())
        assert np.array_equal(bits[0], bits[1]) and not np.any(bits[0] == 0x7FC0)
        cut = {(int(s[0]), int(s[1])) for s in shares}
        some = sorted(cut)[:: max(1, len(cut) // 4)] + [(0, 0), (batch - 1, heads - 1)]
        for c, h in some:
            got, want = run.out_f64(0, c)[:, [h]], case.oracle_out(0, c, heads=[h])
            check_contract(got, want, c)
            check_tight(got, want, int(case.n_keep[c]), c)
    finally:
        run.close()


@pytest.mark.parametrize("batch", [4, 12], ids=["three", "four"])
@pytest.mark.parametrize("style", [0, 1])
def test_heads_of_64_on_either_side_of_four_workgroups(batch, style):
    """Fewer than 1024 row tiles of 128 rows, and more: plans of three and of four workgroups to a compute unit.  A context that moves the smaller
    window of page ids, and sampled heads against the oracle."""
    case = Case([0] * (batch - 1) + [17000], [512] * (batch - 1) + [40], [0] * batch, 32, 4, 64, seed=95 + style, style=style,
                window=32768)
    run = GpuRun(case, tier="device", attn_prerotate=2, attn_tile_rows=128, attn_split=1)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        assert (len(items) > 1024) == (batch == 12)
        run.out[0].view(torch.int16).fill_(0x7FC0)
        run.attn(0)
        run.finish()
        assert not np.any(torch_to_bits(run.out[0]) == 0x7FC0)
        for c, heads in [(0, [0, 31]), (batch - 1, [5, 16])]:
            got, want = run.out_f64(0, c)[:, heads], case.oracle_out(0, c, heads=heads)
            check_contract(got, want, c)
            check_tight(got, want, int(case.n_keep[c]), c)
    finally:
        run.close()


@pytest.mark.parametrize("heads, batch, hist, new, kw, n_shares, whole",
                         [((32, 32, 128), 5, (1053, 1053), (291, 320), {}, 256, 256),
                          ((64, 8, 128), 4, (2426, 2668), (262, 288), {}, 256, 256),
                          ((64, 8, 128), 4, (2426, 2668), (262, 288), {"attn_schedule": 1}, 256, 256),
                          ((64, 4, 64), 2, (4366, 5675), (578, 1000), {}, 384, 768),
                          ((64, 4, 64), 8, (4113, 5346), (156, 365), {}, 512, 1024)],
                         ids=["rotary", "rotated", "pipelined", "three", "four"])
def test_last_round_shares_of_every_tile_kernel(heads, batch, hist, new, kw, n_shares, whole):
    """As above, in the kernels over keys rotated beforehand and with grouped heads; 256 shares of 256 rows are the most there can be, and
    more than 32 MiB; heads of 64 with three and with four workgroups to a compute unit."""
    Hq, Hkv, D = heads
    case = Case(*(list(np.linspace(*lens, batch).round().astype(int)) for lens in (hist, new)), [0] * batch, Hq, Hkv, D, seed=97 + D, window=8192)
    run = GpuRun(case, tier="device", **kw)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        items = items[items[:, 0] >= 0]
        shares = items[items[:, 6] >= 0]
        assert len(shares) == n_shares and len(items) - len(shares) == whole
        assert D == 64 or n_shares * 256 * (D + 2) * 4 > 32 << 20
        bits = []
        for call in (run.ctx.cached_prefill_attn, run.ctx.cached_prefill_attn_static):
            run.out[0].view(torch.int16).fill_(0x7FC0)
            call(0, run.q[0], run.k_pool[0], run.v_pool[0], run.out[0], 1.0 / np.sqrt(D))
            run.finish()
            bits.append(torch_to_bits(run.out[0]).copy())
        assert np.array_equal(bits[0], bits[1]) and not np.any(bits[0] == 0x7FC0)
        cut = sorted({(int(s[0]), int(s[1])) for s in shares})
        for c, g in cut[:: max(1, len(cut) // 4)]:
            h = g * (Hq // Hkv) + 1 % (Hq // Hkv)
            got, want = run.out_f64(0, c)[:, [h]], case.oracle_out(0, c, heads=[h])
            check_contract(got, want, c)
            check_tight(got, want, int(case.n_keep[c]), c)
    finally:
        run.close()


@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("hist, n_shares", [(1000, 3), (1050, 4), (1850, 5), (2000, 7), (2050, 8), (3650, 9), (4050, 15), (4100, 16)])
def test_merges_of_three_to_sixteen_shares(hist, n_shares, D, prerotate):
    """Shares are merged in batches of four; three row tiles, the last one of 24 rows"""
    case = Case([hist], [7], [0], 40, 1, D, seed=99 + hist, style=hist // 50 % 2, window=8192)
    run = GpuRun(case, tier="device", attn_prerotate=prerotate, attn_tile_rows=128)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        items = run.ctx.rebase_read(6).reshape(-1, 8)
        items = items[items[:, 0] >= 0]
        assert np.unique(items[items[:, 6] >= 0][:, 2], return_counts=True)[1].max() == n_shares
        run.attn(0)
        run.finish()
        check_contract(run.out_f64(0, 0), case.oracle_out(0, 0), 0)
        check_tight(run.out_f64(0, 0), case.oracle_out(0, 0), hist, 0)
    finally:
        run.close()


@pytest.mark.parametrize("offset", [1, 4], ids=["2-bytes", "8-bytes"])
@pytest.mark.parametrize("heads, new, kw", [((8, 8, 128), 150, {}), ((8, 1, 64), 200, {"attn_prerotate": 2}), ((8, 1, 128), 1, {}), ((8, 1, 128), 20, {})],
                         ids=["rotary", "rotated", "few-rows", "shares"])
def test_queries_and_outputs_at_any_element(heads, new, kw, offset):
    """Queries and outputs that are aligned to their elements only; nothing is written beside the outputs, and the bits are those of aligned ones."""
    case = Case([900, 40], [new, max(1, new // 3)], [0, 0], *heads, seed=120 + new, window=2048)
    run = GpuRun(case, tier="device", **kw)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        run.attn(0)
        n = run.q[0].numel()
        room = [torch.zeros(n + 16, dtype=torch.bfloat16, device=run.dev) for _ in range(2)]
        q, out = (t[offset:offset + n].view(run.q[0].shape) for t in room)
        q.copy_(run.q[0])
        run.ctx.cached_prefill_attn(0, q, run.k_pool[0], run.v_pool[0], out, 1.0 / np.sqrt(heads[2]))
        run.finish()
        assert np.array_equal(torch_to_bits(out), torch_to_bits(run.out[0]))
        assert not room[1][:offset].any() and not room[1][offset + n:].any()
        check_contract(run.out_f64(0, 0), case.oracle_out(0, 0), 0)
    finally:
        run.close()

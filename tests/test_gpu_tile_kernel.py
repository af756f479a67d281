"""The matrix-core tile kernel where its schedule can go wrong: contexts that end around the edges of key tiles and of the
rings (one to six tiles, one key more or less), both groups of wavefronts live or only the first, and rows whose scores rise
so fast along the context that the reference has to move inside interior tiles, by more than a probability could hold."""
import numpy as np
import pytest
import torch

from harness import Case, GpuRun
from test_gpu_parity import check_contract, check_tight
from synth import bf16_bits_to_f64

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


@pytest.mark.parametrize("steps", [[1.0, 40.0], [40.0, 1.0], [1.0, 4.0, 16.0, 64.0, 1.0]], ids=["jump", "fall", "stairs"])
@pytest.mark.parametrize("prerotate", [1, 2], ids=["rotary", "rotated"])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("D", [64, 128])
def test_reference_moves(D, rows, prerotate, steps):
    """Keys whose length changes along the context by powers of four and more.  The largest scores are in the hundreds, so
    the rounding of the rotated operands decides between the largest of them: outputs are compared with the oracle where
    the two largest probabilities are clear of that, and everywhere against the range of the values."""
    case = Case([1500], [40], [0], 8, 1, D, seed=75, window=2048)
    k = bf16_bits_to_f64(case.tensor(0, "k_hist", 0))
    factor = np.repeat(np.asarray(steps), -(-1500 // len(steps)))[:1500]
    scaled = (k * factor[:, None, None]).astype(np.float32)            # (times a power of two or 40: rounded once more below)
    case.data[(0, "k_hist", 0)] = (scaled.view(np.uint32) >> 16).astype(np.uint16)
    case.data[(0, "v_hist", 0)] = case.tensor(0, "v_hist", 0)
    got, want = outputs(case, attn_tile_rows=rows, attn_prerotate=prerotate, attn_split=1)[0], case.oracle_out(0, 0)
    assert np.isfinite(got).all()
    v = np.concatenate([bf16_bits_to_f64(case.tensor(0, n, 0)) for n in ("v_hist", "v_new")])
    lo, hi = v.min(axis=0)[0], v.max(axis=0)[0]
    assert (got >= lo - 0.02).all() and (got <= hi + 0.02).all()       # a convex combination, rounded
    # rotated operands are rounded to 2^-9 of themselves: a score s moves by about |s| 2^-9 sqrt(2 / D) * 2 (independent
    # errors of D products), 0.2 for the hundreds here; a softmax over few keys then moves by that share of the values
    err = np.abs(got - want)
    assert np.median(err) < 0.05, np.median(err)
    assert err.mean() < 0.15, err.mean()


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

"""The attention work list of a plan, on the model of the HIP runtime (no GPU): which batches have their keys cut."""
import numpy as np
import pytest

from hip_model import Turn, in_model


def plan(m, hist, new, heads, **cfg):
    """live items of the plan: rows (conversation, kv head, first row, rows, first key, end of keys, share, 0)"""
    t = Turn(m, hist, new, heads=heads, **cfg)
    t.rebase()
    items = t.ctx.rebase_read(6).reshape(-1, 8)
    t.ctx.close()
    return items[items[:, 0] >= 0]


def check_cover(items, hist, new, heads):
    """every (conversation, kv head, row tile) is covered once, its shares end to end"""
    G = heads[0] // heads[1]
    tiles = {}
    for seq, head, row0, rows, begin, end, part, _ in items.tolist():
        tiles.setdefault((seq, head, row0, rows), []).append((begin, end, part))
    rows = np.zeros((len(hist), heads[1]), np.int64)
    for (seq, head, row0, n), shares in tiles.items():
        rows[seq, head] += n
        shares.sort()
        assert shares[0][0] == 0 and shares[-1][1] == hist[seq] + (row0 + n - 1) // G + 1
        assert all(a[1] == b[0] for a, b in zip(shares, shares[1:]))
        assert all((p >= 0) == (len(shares) > 1) for _, _, p in shares)
    assert (rows == np.asarray(new)[:, None] * G).all()


# Batches with fewer (conversation, kv head) units than compute units: whole, they leave the others without work.
@pytest.mark.parametrize("batch, heads, tokens", [(3, (32, 32, 128), 2000), (4, (32, 32, 128), 1000), (4, (32, 32, 128), 1500), (2, (40, 40, 128), 1000),
                                                  (4, (40, 40, 128), 2000), (6, (32, 32, 128), 3000), (12, (16, 8, 64), 2000), (28, (8, 8, 128), 3000)])
@in_model
def test_a_small_decode_batch_is_cut(m, batch, heads, tokens):
    hist = [tokens - 1 - 7 * c for c in range(batch)]
    items = plan(m, hist, [1] * batch, heads)
    check_cover(items, hist, [1] * batch, heads)
    assert len(items) >= min(256, 2 * batch * heads[1]) and (items[:, 6] >= 0).all()


# Turns on the tile kernels (four and more stacked rows; few enough for the few-rows kernel only in the first conversation of
# some).  Times are us of one attention call, cut and whole.
CUT = [(13, (16, 8, 64), 2134, 2392, 9, 45),           # 38, 72
       (33, (4, 4, 64), 3209, 3355, 5, 128),           # 60, 102
       (28, (4, 4, 64), 2184, 2335, 24, 197),          # 47, 62
       (46, (8, 2, 128), 2217, 2409, 5, 39),           # 64, 80
       (3, (16, 8, 64), 2048, 2048, 399, 416)]         # 47, 52
WHOLE = [(6, (64, 8, 128), 423, 586, 113, 134),        # 68, 41
         (3, (40, 40, 128), 284, 671, 423, 483),       # 90, 56
         (9, (32, 4, 64), 1024, 1024, 97, 151),        # 56, 35
         (5, (32, 32, 128), 1500, 1563, 75, 258),      # 102, 74
         (4, (32, 4, 64), 0, 0, 300, 703),             # 26, 22
         (8, (32, 32, 128), 2048, 2048, 64, 512)]      # 160, 150


@pytest.mark.parametrize("batch, heads, hist_lo, hist_hi, new_lo, new_hi", CUT + WHOLE)
@in_model
def test_items_stay_whole_where_shares_cost_more(m, batch, heads, hist_lo, hist_hi, new_lo, new_hi):
    hist, new = (np.linspace(lo, hi, batch).round().astype(np.int32) for lo, hi in ((hist_lo, hist_hi), (new_lo, new_hi)))
    np.random.default_rng(3).shuffle(new)
    items = plan(m, hist, new, heads)
    check_cover(items, hist, new, heads)
    whole = (batch, heads, hist_lo, hist_hi, new_lo, new_hi) in WHOLE
    assert (items[:, 6] >= 0).any() != whole


# Rows of the tiles of mixed batches; times are us of one attention call with tiles of 256 and of 128 rows.
@pytest.mark.parametrize("batch, heads, hist_lo, hist_hi, new_lo, new_hi, rows",
                         [(16, (32, 32, 128), 1536, 1536, 19, 178, 256),        # 116, 137
                          (32, (32, 32, 128), 3080, 3206, 41, 168, 256),        # 399, 460
                          (14, (32, 32, 128), 608, 612, 164, 370, 256),         # 127, 136
                          (64, (4, 4, 64), 343, 417, 279, 344, 256),            # 47, 56
                          (17, (32, 32, 128), 0, 0, 303, 311, 128),             # 103, 80
                          (40, (40, 40, 128), 0, 0, 80, 137, 128),              # 100, 70
                          (52, (32, 4, 64), 0, 0, 18, 114, 128)])               # 27, 23
@in_model
def test_tile_rows_of_mixed_batches(m, batch, heads, hist_lo, hist_hi, new_lo, new_hi, rows):
    hist, new = (np.linspace(lo, hi, batch).round().astype(np.int32) for lo, hi in ((hist_lo, hist_hi), (new_lo, new_hi)))
    items = plan(m, hist, new, heads)
    check_cover(items, hist, new, heads)
    assert (items[:, 3].max() <= 128) == (rows == 128)


# Grouped heads of 64 with 128-row tiles: as many shares as the partial-result buffer holds would be more than the static scratch
# array does (992 of 128 rows), and 256-row tiles need fewer.
@pytest.mark.parametrize("batch, heads, hist_lo, hist_hi, new_lo, new_hi", [(3, (64, 8, 64), 19538, 35752, 327, 444), (3, (32, 4, 64), 8287, 29283, 304, 389),
                                                                            (3, (64, 8, 64), 9000, 30000, 300, 500)])
@in_model
def test_the_static_entry_point_takes_plans_with_smaller_tiles(m, batch, heads, hist_lo, hist_hi, new_lo, new_hi):
    hist, new = (np.linspace(lo, hi, batch).round().astype(np.int32) for lo, hi in ((hist_lo, hist_hi), (new_lo, new_hi)))
    t = Turn(m, hist, new, heads=heads, require_load=0)
    t.rebase()
    items = t.ctx.rebase_read(6).reshape(-1, 8)
    items = items[items[:, 0] >= 0]
    check_cover(items, hist, new, heads)
    assert items[:, 3].max() <= 128
    t.attn(static=True)


# Heads of 64, keys rotated beforehand: the launch has the workgroups to a compute unit that the plan was laid out for, three, or four
# where there are more row tiles than that many places.
@pytest.mark.parametrize("batch, heads, hist_lo, hist_hi, new_lo, new_hi, per_cu, last_round",
                         [(2, (64, 4, 64), 4366, 5675, 578, 1000, 3, True),        # 792 tiles, 1152 items with the shares
                          (12, (32, 4, 64), 4167, 5417, 243, 291, 3, True),        # 824, 1496
                          (8, (64, 4, 64), 4113, 5346, 156, 365, 4, True),         # 1056, 1536
                          (12, (32, 4, 64), 0, 0, 200, 250, 3, False),
                          (16, (64, 8, 64), 0, 0, 105, 183, 4, False)])
@in_model
def test_the_launch_has_the_workgroups_that_were_planned(m, batch, heads, hist_lo, hist_hi, new_lo, new_hi, per_cu, last_round):
    hist, new = (np.linspace(lo, hi, batch).round().astype(np.int32) for lo, hi in ((hist_lo, hist_hi), (new_lo, new_hi)))
    t = Turn(m, hist, new, heads=heads, require_load=0)
    t.rebase()
    items = t.ctx.rebase_read(6).reshape(-1, 8)
    live, die = items[:, 0] >= 0, np.arange(len(items)) % 8
    check_cover(items[live], hist, new, heads)
    cut = live & (items[:, 6] >= 0)
    tiles = sum((int(n) * (heads[0] // heads[1]) + 127) // 128 for n in new) * heads[1]
    assert (tiles > 1024) == (per_cu == 4)
    if last_round:                          # whole rounds of workgroups on every die
        whole = [int((live & ~cut & (die == d)).sum()) for d in range(8)]
        assert cut.any() and all(w > 0 and w % (32 * per_cu) == 0 for w in whole)
    assert m.named(m.queued(t.attn), "attn_prerot_kernelILi64ELi0ELi4ELi32ELi%dEE" % per_cu)


# Few rows: however many compute units there are to spread the shares over, no more cuts than there is room for.
@pytest.mark.parametrize("cus", [256, 1024])
@pytest.mark.parametrize("batch, pages", [(2, 1500), (15, 500), (40, 24), (1, 4000)])
@in_model
def test_cuts_of_a_few_rows_plan_are_bounded(m, cus, batch, pages):
    m.lib.model_cus(cus)
    heads = (64, 8, 128)
    hist = [16 * pages - 3 - c for c in range(batch)]
    items = plan(m, hist, [1] * batch, heads)
    check_cover(items, hist, [1] * batch, heads)
    assert len(items) <= batch * heads[1] + 512 and (items[:, 6] >= 0).sum() <= 1024


# Plans of many rounds of workgroups: the tiles of a unit follow each other on their die, so that its L2 has their keys, up to the die's last items,
# which are longest first.
@pytest.mark.parametrize("batch, heads, hist_lo, hist_hi, new_lo, new_hi, last",
                         [(64, (64, 8, 128), 2500, 2600, 256, 260, 128), (64, (32, 32, 128), 300, 3000, 100, 900, 128),
                          (40, (32, 4, 64), 500, 4000, 200, 1500, 512), (16, (32, 4, 64), 0, 0, 128, 2048, 512)])
@in_model
def test_tiles_of_a_unit_follow_each_other(m, batch, heads, hist_lo, hist_hi, new_lo, new_hi, last):
    hist, new = (np.linspace(lo, hi, batch).round().astype(np.int32) for lo, hi in ((hist_lo, hist_hi), (new_lo, new_hi)))
    t = Turn(m, hist, new, heads=heads, require_load=0)
    t.rebase()
    all_items = t.ctx.rebase_read(6).reshape(-1, 8)
    check_cover(all_items[all_items[:, 0] >= 0], hist, new, heads)
    assert (all_items[:, 6] < 0).all()
    for die in range(8):
        items = all_items[die::8]
        items = items[items[:, 0] >= 0]
        units = [tuple(u) for u in items[:-last, :2].tolist()]
        changes = sum(a != b for a, b in zip(units, units[1:]))
        assert changes == max(len(set(units)) - 1, 0)
        full = items[-last:]
        full = full[full[:, 3] == full[:, 3].max()]
        tiles64 = (full[:, 5] + 63) // 64
        assert (np.diff(tiles64) <= 0).all()

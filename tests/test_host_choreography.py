"""What the library queues where, and what waits for it, on a model of the HIP runtime in which nothing is done before
something waits for it (hip_model.py): the host code of the C ABI, without a GPU."""
import ctypes as C

import pytest

from hip_model import PER_THREAD, Turn, in_model


@in_model
def test_a_whole_turn_runs_on_the_model(m):
    """the model itself: a pinned and a device tier, every load and save done after sync, joined work in front of the stream"""
    for tier in (0, 1):
        t = Turn(m, [4000, 30], [200, 1], tier=tier)
        s = m.stream()
        ops = m.queued(lambda: (t.rebase(s), t.load(), t.append(s), t.attn(s), t.save(s)))
        moves = m.named(ops, "link_kernel") + m.named(ops, "move_kernel")
        assert len(moves) == 2 and not any(m.done(op) for op in ops)
        attn, = m.named(ops, "attn_dma_kernel")
        assert m.behind(attn, moves[0]) and m.behind(moves[1], m.named(ops, "append_kernel")[0])
        other = m.stream()
        t.ctx.join(other)
        assert all(m.stream_behind(other, op) for op in moves)
        t.ctx.sync()
        assert all(m.done(op) for op in moves)
        t.ctx.close()


# ---- ca_sync and ca_join with another GPU current ---------------------------------------------------------------
@in_model
def test_sync_covers_a_short_save_with_another_gpu_current(m):
    t = Turn(m, [0], [2], tier=1, device=1)
    t.rebase()
    t.append()
    save, = m.queued(t.save)
    m.device(0)
    t.ctx.sync()
    assert m.done(save) and m.current() == 0


@in_model
def test_join_covers_a_short_save_with_another_gpu_current(m):
    t = Turn(m, [0], [2], tier=1, device=1)
    t.rebase()
    t.append()
    save, = m.queued(t.save)
    s1 = m.stream()
    m.device(0)
    s0 = m.stream()
    for s in (s0, s1, None):
        t.ctx.join(s)
        assert m.current() == 0 and m.stream_behind(s, save)


@in_model
def test_a_plan_waits_for_the_last_one_after_a_join_with_another_gpu_current(m):
    t = Turn(m, [4000], [200], tier=1, device=1)
    t.rebase()
    load, = m.queued(t.load)
    m.device(0)
    t.ctx.join(None)
    plan, = m.queued(t.rebase)
    assert m.behind(plan, load)


# ---- a tier that is too small --------------------------------------------------------------------------------
def refused(m, call):
    import paper_2403_19708_amd as ca
    at = m.lib.model_ops()
    with pytest.raises(ca.CaError) as e:
        call()
    assert e.value.status_name == "CA_ERR_INVALID_ARG" and m.lib.model_ops() == at       # nothing was queued


@pytest.mark.parametrize("tier", [0, 1], ids=["device", "pinned"])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("hist,new", [(40, 2), (4000, 200)], ids=["short", "long"])
@in_model
def test_a_tier_that_is_too_small_is_refused(m, hist, new, mode, tier):
    fits = Turn(m, [5, hist], [3, new], tier=tier, load_mode=mode, save_mode=mode)
    fits.rebase()
    fits.load(); fits.append(); fits.save(); fits.append_save()
    t = Turn(m, [5, hist], [3, new], tier=tier, tier_rows=[8, hist + new - 1], load_mode=mode, save_mode=mode)
    t.rebase()
    t.load()
    refused(m, t.save)
    refused(m, t.append_save)
    t = Turn(m, [5, hist], [3, new], tier=tier, tier_rows=[8, hist - 1], load_mode=mode)
    t.rebase()
    refused(m, t.load)


@in_model
def test_a_pinned_tier_has_to_hold_what_is_read(m):
    """the end of the history is discarded: its rows need not be there in pinned memory (device memory holds the history)"""
    for tier in (1, 0):
        t = Turn(m, [4000], [200], tier=tier, tier_rows=[3000])
        t.rebase(keep_ranges=[[(0, 4), (1000, 3000)]])
        if tier:
            assert len(m.queued(t.load)) == 1
        else:
            refused(m, t.load)


REGISTERED = 2          # host memory the GPU addresses 2^40 bytes further on; the runtime does not know its extent


@pytest.mark.parametrize("hist,new", [(40, 2), (4000, 200)], ids=["short", "long"])
@in_model
def test_kernels_reach_registered_memory_where_the_gpu_has_it(m, hist, new):
    t = Turn(m, [5, hist], [3, new], tier=REGISTERED)
    t.rebase()
    for call in (t.load, t.save, t.append_save):
        op = m.queued(call)[-1]
        for c in range(2):
            at = int(t.hist[c]) * t.row if "append_save" in m.what(op) else 0
            assert m.lib.model_move_pointer(op, c, 0) == t.tk[c] + (1 << 40) + at, m.what(op)
            assert m.lib.model_move_pointer(op, c, 1) == t.tv[c] + (1 << 40) + at


# ---- scratch of the two attention entry points -----------------------------------------------------------------
@in_model
def test_the_two_attention_entry_points_share_no_scratch(m):
    """a plan of the few-rows kernel that splits keys: partial results and merge counters are an entry point's own"""
    t = Turn(m, [9000, 50], [1, 1], heads=(8, 1, 128), require_load=0)
    t.rebase()
    ordinary, static = m.queued(lambda: (t.attn(), t.attn(static=True)))
    assert "attn_rows_kernel" in m.what(ordinary)
    for which in range(2):
        a, b = m.lib.model_attn_pointer(ordinary, which), m.lib.model_attn_pointer(static, which)
        assert a and b and a != b


# ---- one stream handle, several streams -------------------------------------------------------------------------
@pytest.mark.parametrize("fused", [False, True], ids=["save", "append-save"])
@in_model
def test_short_moves_of_two_threads_on_their_own_default_streams(m, fused):
    """hipStreamPerThread is one handle for a stream in each thread: a context handed on keeps track of both"""
    import threading
    t = Turn(m, [0], [2], tier=1)
    t.rebase(PER_THREAD)
    t.append(PER_THREAD)
    call = (lambda: t.append_save(PER_THREAD)) if fused else (lambda: t.save(PER_THREAD))
    saves = []
    for _ in range(2):
        thread = threading.Thread(target=lambda: saves.append(m.queued(call)[-1]))
        thread.start()
        thread.join()
    s = m.stream()
    t.ctx.join(s)
    assert all(m.stream_behind(s, op) for op in saves)
    t.ctx.sync()
    assert all(m.done(op) for op in saves)


# ---- ca_sync and ca_join cover a save by the append kernel ------------------------------------------------------
@pytest.mark.parametrize("tier,mode", [(0, 0), (1, 2), (1, 0)], ids=["device", "pinned-mode2", "pinned"])
@pytest.mark.parametrize("new", [2, 20000], ids=["short", "long"])
@pytest.mark.parametrize("own", [False, True], ids=["default-stream", "own-stream"])
@in_model
def test_sync_and_join_cover_append_save(m, own, new, tier, mode):
    t = Turn(m, [0], [new], tier=tier, save_mode=mode)
    s, s2, other = (m.stream() if own else None), m.stream(), m.stream()
    t.rebase(s)
    saves = [m.queued(lambda: t.append_save(x))[-1] for x in (s, s, s2)]        # (the third while the others are under way)
    t.ctx.join(other)
    assert all(m.stream_behind(other, op) for op in saves)
    t.ctx.sync()
    assert all(m.done(op) for op in saves)


@in_model
def test_append_save_can_be_captured(m):
    """the caller orders a graph it launches: nothing queued into one may be waited for by the calls outside"""
    t = Turn(m, [0], [2])
    s, s2 = m.stream(), m.stream()
    t.rebase(s)
    t.append_save(s2)
    m.lib.model_capture(s, 1)
    assert len(m.queued(lambda: (t.append_save(s), t.attn(s, static=True)))) == 2
    assert m.lib.model_capture(s, 0)
    t.ctx.join(s2)
    t.ctx.sync()
    t.rebase(s)


@pytest.mark.parametrize("tier", [0, 1], ids=["device", "pinned"])
@in_model
def test_a_load_stays_out_of_a_capture_of_the_plans_stream(m, tier):
    """the next job's read buffer fills while the current job's step is captured on the stream both plans were made on"""
    t = Turn(m, [40], [2], tier=tier)
    s = m.stream()
    t.rebase(s)
    m.lib.model_capture(s, 1)
    load, = m.queued(t.load)
    assert not m.stream_behind(s, load) and m.lib.model_capture(s, 0)
    t.ctx.join(s)
    assert m.stream_behind(s, load)


@pytest.mark.parametrize("tier", [0, 1], ids=["device", "pinned"])
@pytest.mark.parametrize("hist,new", [(40, 2), (4000, 200)], ids=["short", "long"])
@pytest.mark.parametrize("plan", ["default", "own", "captured"])
@in_model
def test_moves_of_another_job_leave_a_capture_whole(m, plan, hist, new, tier):
    """a step is captured on one stream (in global mode) while another job's layers are loaded and saved on others, with short
    moves and saves of that job under way on further streams"""
    t = Turn(m, [hist], [new], tier=tier, layers=4)
    captured, own, other = m.stream(), m.stream(), m.stream()
    s = {"default": None, "own": own, "captured": captured}[plan]
    after = own if plan == "own" else None
    t.rebase(s)
    ops = m.queued(lambda: (t.load(0), t.append(after), t.save(other), t.save(after, tok_begin=[0], tok_end=[hist], dst_tok_offset=[0])))
    load0, saves = ops[0], [ops[2], ops[3]]

    def during_capture(call):
        m.lib.model_capture(captured, 1)
        op = (m.queued(call) or [None])[-1]
        assert m.lib.model_capture(captured, 0)
        return op
    load1 = during_capture(lambda: t.load(1))
    during_capture(lambda: t.append(after, 1))
    for call in (lambda: t.save(after), lambda: t.save(other), lambda: t.append_save(after), lambda: t.append_save(other)):
        saves.append(during_capture(call))
    for layer, load in ((0, load0), (1, load1)):
        for x in (after, other):
            attn = during_capture(lambda: t.attn(x, layer))
            assert m.behind(attn, load) or m.done(load)
    t.rebase(s)
    t.load(0); t.append_save(s)
    during_capture(lambda: t.ctx.join(other))
    assert all(m.stream_behind(other, op) or m.done(op) for op in saves)


# ---- the order of saves ---------------------------------------------------------------------------------------------
@pytest.mark.parametrize("streams", ["one", "two"])
@pytest.mark.parametrize("sizes", [(4000, 2), (2, 4000), (2, 2, 4000), (4000, 2, 2)], ids=str)
@in_model
def test_saves_of_a_plan_are_done_in_the_order_they_were_asked_for(m, sizes, streams):
    """also where a short one, on the caller's stream, meets a long one on the save stream: both may write the same rows"""
    t = Turn(m, [0], [4000], tier=1)
    s = [m.stream()] * 3 if streams == "one" else [m.stream() for _ in range(3)]
    t.rebase(s[0])
    saves = [m.queued(lambda: t.save(x, tok_begin=[4000 - n], tok_end=[4000], dst_tok_offset=[0]))[-1] for n, x in zip(sizes, s)]
    assert all(m.behind(b, a) for a, b in zip(saves, saves[1:]))


# ---- what the binding takes as an argument ----------------------------------------------------------------------------
class _Holder:
    """an object with an address or a stream that is a numpy integer"""

    def __init__(self, value):
        import numpy as np
        self.cuda_stream = np.int64(value)

    def data_ptr(self):
        return self.cuda_stream


def _padded(np, kind, p):
    wide = np.zeros((len(p), 3), kind)
    wide[:, 1] = p
    return wide[:, 1]


POINTERS = {
    "list": lambda np, p: p,
    "tensors": lambda np, p: [_Holder(x) for x in p],
    "c_void_p": lambda np, p: (C.c_void_p * len(p))(*p),
    "uint64": lambda np, p: np.array(p, np.uint64),
    "int64-strided": lambda np, p: _padded(np, np.int64, p),
    "int64-swapped": lambda np, p: np.array(p, ">i8"),
    "objects": lambda np, p: np.array(p, object),
    "float64": lambda np, p: np.array(p, np.float64),
    "column": lambda np, p: np.array(p).reshape(-1, 1),
}


@pytest.mark.parametrize("form", POINTERS)
@in_model
def test_pointers_reach_the_library_in_every_form(m, form):
    import numpy as np
    t = Turn(m, [40, 50, 60], [2, 3, 4], tier=1)
    want = [list(t.tk), list(t.tv)]
    t.rebase()
    t.tk, t.tv = (POINTERS[form](np, p) for p in want)
    for call in (t.load, t.save, t.append_save):
        op = m.queued(call)[-1]
        for c in range(3):
            at = int(t.hist[c]) * t.row if "append_save" in m.what(op) else 0
            assert [m.lib.model_move_pointer(op, c, v) for v in range(2)] == [want[v][c] + at for v in range(2)], (form, m.what(op))


@in_model
def test_pointer_arrays_that_are_refused(m):
    import numpy as np
    t = Turn(m, [40, 50], [2, 3], tier=1)
    t.rebase()
    tk = list(t.tk)
    for bad, error in (((C.c_uint64 * 2)(*tk), C.ArgumentError), ((C.c_int32 * 2)(1, 2), C.ArgumentError), (iter(tk), TypeError),
                       (None, TypeError), (np.array(tk[:1]), ValueError), (tk + tk, ValueError)):
        t.tk = bad
        for call in (t.load, t.save, t.append_save):
            with pytest.raises(error):
                call()
    t.tk = tk
    with pytest.raises(ValueError):
        t.save(tok_begin=np.zeros((1, 1, 2)))


@in_model
def test_numbers_reach_the_library_in_every_form(m):
    import numpy as np
    t = Turn(m, [40], [2], layers=2)
    s = m.stream()
    t.num_pages = float(t.num_pages)
    plan, = m.queued(lambda: t.rebase(_Holder(s)))
    assert m.lib.model_stream(plan) == s
    t.nk = _Holder(t.nk)
    for layer in (1.0, np.int16(1)):
        op, = m.queued(lambda: t.append(_Holder(s), layer))
        assert m.lib.model_stream(op) == s


# ---- internal streams of several contexts ---------------------------------------------------------------------------
MODES = pytest.mark.parametrize("load_mode,save_mode", [(0, 0), (1, 1), (2, 2)], ids=["kernel", "staged", "in-place"])


@MODES
@in_model
def test_contexts_behind_different_streams_do_not_wait_for_each_other(m, load_mode, save_mode):
    a, b = (Turn(m, [4000], [200], tier=1, load_mode=load_mode, save_mode=save_mode) for _ in range(2))
    sa, sb = m.stream(), m.stream()

    def turn(t, s):
        t.rebase(s); t.load(); t.append(s); t.attn(s); t.save(s); t.append_save(s)
        t.ctx.join(s)
    for _ in range(2):
        first = m.queued(lambda: turn(a, sa))
        second = m.queued(lambda: turn(b, sb))
        assert not any(m.behind(y, x) for x in first for y in second)


@in_model
def test_contexts_planned_on_one_stream_that_save_behind_different_ones(m):
    a, b = (Turn(m, [0], [4000], tier=1) for _ in range(2))
    sa, sb = m.stream(), m.stream()
    a.rebase(); b.rebase()
    m.queued(lambda: (a.append(sa), a.save(sa)))
    append_a, = m.queued(lambda: a.append(sa))
    a.save(sa)
    save = m.queued(lambda: (b.append(sb), b.save(sb)))[-1]
    assert not m.behind(save, append_a)


@MODES
@in_model
def test_contexts_behind_one_stream_share_the_internal_ones(m, load_mode, save_mode):
    def turn(t, s):
        t.rebase(s); t.load(); t.append_save(s); t.save(s)
        t.ctx.join(s)
    before = m.lib.model_streams_alive()
    turns = [Turn(m, [4000], [200], tier=1, load_mode=load_mode, save_mode=save_mode) for _ in range(3)]
    per_set = 3 if load_mode == 1 else 2
    s = m.stream()
    for t in turns:
        turn(t, None)
    assert m.lib.model_streams_alive() == before + 1 + per_set
    for t in turns:
        turn(t, s)
    for t in turns:                 # (one set was left for the first context's change)
        turn(t, None)
    assert m.lib.model_streams_alive() <= before + 1 + 2 * per_set
    for t in turns:
        t.ctx.close()
    assert m.lib.model_streams_alive() == before + 1


@MODES
@in_model
def test_moves_keep_their_order_when_the_callers_stream_changes(m, load_mode, save_mode):
    """a second context keeps the first internal streams in use, so that the first one has to change them"""
    t, other = (Turn(m, [4000], [4000], tier=1, load_mode=load_mode, save_mode=save_mode) for _ in range(2))
    streams = [None, m.stream(), m.stream(), None]
    moves = []
    for s in streams:
        other.rebase(None); other.append_save(None)
        plan, = m.queued(lambda: t.rebase(s))
        assert all(m.behind(plan, op) for op in moves)
        new = m.queued(t.load)
        for x in streams:
            new += [op for op in m.queued(lambda: t.save(x)) if m.lib.model_stream(op) != x]
        assert all(m.behind(op, plan) for op in new)
        moves += new
        saves = new[1:] if load_mode != 1 else new[3:]
        assert len(saves) >= 4 and all(m.behind(y, x) for x, y in zip(saves, saves[1:]))
    t.ctx.join(streams[1])
    assert all(m.stream_behind(streams[1], op) for op in moves)
    t.ctx.sync()
    assert all(m.done(op) for op in moves)


# ---- staging rings ------------------------------------------------------------------------------------------------------
@in_model
def test_only_staged_moves_have_a_staging_ring(m):
    def bytes_of(**modes):
        before = m.lib.model_device_bytes()
        t = Turn(m, [4000], [200], tier=1, pipeline_depth=4, **modes)
        made = m.lib.model_device_bytes() - before
        t.rebase(); t.load(); t.append(); t.save(); t.append_save()
        t.ctx.close()
        return made
    ring = 4 * 2 * (4200 + 64) * 2 * 128 * 2        # slots x (keys, values) x tokens x row
    bytes_of()                                      # (the first context finds the library's static memory)
    least = bytes_of()
    assert bytes_of(load_mode=2, save_mode=2) == least
    for modes, rings in ((dict(load_mode=1), 1), (dict(save_mode=1), 1), (dict(load_mode=1, save_mode=1), 2)):
        assert bytes_of(**modes) - least == rings * ring


# ---- both directions of the host link at once ----------------------------------------------------------------------------
@pytest.mark.parametrize("fused", [False, True], ids=["save", "append-save"])
@pytest.mark.parametrize("hist, new, prerotate, beside", [(4000, 100, 2, 2), (4000, 100, 1, 4), (150, 100, 2, 4), (0, 100, 2, 4)],
                         ids=["rotated", "rotary", "short-history", "first-turn"])
@in_model
def test_few_workgroups_write_back_beside_loads_and_attention_over_rotated_keys(m, hist, new, prerotate, beside, fused):
    """the last layer's write-back, which runs beside no load, and write-backs as large as half the loads keep four"""
    t = Turn(m, [hist] * 4, [new] * 4, tier=1, layers=3, heads=(8, 8, 128), attn_prerotate=prerotate)
    t.rebase()
    for layer in range(3):
        t.load(layer=layer)
    got = []
    for layer in range(3):
        if not fused:
            t.append(layer=layer)
        ops = m.queued(lambda: t.append_save(layer=layer) if fused else t.save(layer=layer))
        got.append(m.lib.model_workgroups(m.named(ops, "link_kernel")[0]))
        t.attn(layer=layer)
    assert got == [beside, beside, 4]

"""Append and save of one token per conversation (decode steps) by the kernels that get the slots in their arguments: as
many conversations as these hold and one more, first and last slots of a page, rows of less and more than one workgroup,
both tiers; against the oracle's pool and the rows themselves, bit for bit.  A captured append follows the plan of the replay."""
import numpy as np
import pytest
import torch

from harness import Case, GpuRun, torch_to_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tier", ["device", "pinned"])
@pytest.mark.parametrize("B", [1, 16, 64, 65])
@pytest.mark.parametrize("heads", [(1, 1, 64), (4, 2, 128), (40, 40, 128), (24, 3, 64)], ids=lambda h: "hq%d-hkv%d-d%d" % h)
def test_one_token_each(heads, B, tier):
    Hq, Hkv, D = heads
    hist = [(c * 7) % 33 for c in range(B)]                # slots 0 to 15 of first, second and third pages
    case = Case(hist, [1] * B, [0] * B, Hq, Hkv, D, seed=80 + B, window=64)
    run = GpuRun(case, tier=tier)
    try:
        run.rebase()
        run.load(0)
        run.append(0)
        run.save(0)
        run.finish()
        for which, pool in (("k", run.k_pool[0]), ("v", run.v_pool[0])):
            assert np.array_equal(torch_to_bits(pool), case.oracle_pool(0, which))
        for c in range(B):
            for which, rows in (("k", run.host_k[0][c]), ("v", run.host_v[0][c])):
                want = np.concatenate([case.tensor(0, which + "_hist", c), case.tensor(0, which + "_new", c)])
                assert np.array_equal(torch_to_bits(rows), want), (c, which)
    finally:
        run.close()


def test_captured_append_follows_the_plan():
    case = Case([5, 13, 16], [1] * 3, [0] * 3, 4, 2, 128, seed=85, window=64)
    run = GpuRun(case, tier="device")
    try:
        stream = torch.cuda.Stream()
        run.rebase(stream)
        run.append(0, stream)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            run.append(0, stream)
        for step in range(3):
            hist = case.hist_len + step
            run.ctx.rope_rebase(hist, case.keep_start, case.new_len, case.block_table, case.num_pages, stream)
            with torch.cuda.stream(stream):
                run.k_pool[0].zero_()
            graph.replay()
            torch.cuda.synchronize()
            pool = torch_to_bits(run.k_pool[0])
            want = np.zeros_like(pool)
            for c in range(case.B):
                want[case.block_table[c][hist[c] // 16], :, hist[c] % 16] = case.tensor(0, "k_new", c)[0]
            assert np.array_equal(pool, want), step
    finally:
        run.close()

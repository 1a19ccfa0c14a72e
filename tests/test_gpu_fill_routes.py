"""The routes of a plan's fill: plans without misses between plans that have some (the mapped
fill enqueues nothing for them, the staged one an empty job), victims that were never used
(nothing is written back), write-back copies small and large with sorts handed over ahead,
and a flush of several 2 MiB pieces with a remainder."""
import pytest

from paper_2205_04702_amd import scratchpipe as sp
from paper_2205_04702_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harness():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("flags", [0, sp.SP_FLAG_EVENT_WAITS])
@pytest.mark.parametrize("fill,prefetch,hold_past", [("mapped", 0, 0), ("mapped", 1, 0),
                                                     ("mapped", 0, 2), ("staged", 0, 0),
                                                     ("staged", 1, 2)])
def test_plans_without_misses_between_others(harness, fill, prefetch, hold_past, flags):
    """Every batch comes three times: its second and third plan miss nothing (with prefetch
    its first misses nothing of its own either).  The slots fill up after some plans."""
    w = wl.custom(rows=[3000, 2000], dim=32, batch=48, pooling=[4, 2], slots=[1400, 800],
                  lookahead=2, steps=30, dist=("uniform",), seed=11)
    print(f"case {fill} prefetch {prefetch} hold_past {hold_past} flags {flags}", flush=True)
    batches = [wl.batch(w, s // 3) for s in range(w.steps)]
    r = harness.run_parity(w, batches, fill=fill, prefetch=prefetch, hold_past=hold_past,
                           flags=flags, prepare_ahead=1, sync_each_step=False,
                           check_fwd_steps=[0, 1, 2, 3, 15, 28, 29])
    assert r["stats"]["evictions"] > 0


@pytest.mark.parametrize("fill", ["mapped", "staged"])
def test_only_never_used_slots(harness, fill):
    """A slot for every row: plans miss for a while and never evict."""
    w = wl.custom(rows=[2500, 1500], dim=16, batch=32, pooling=3, slots=[2500, 1500],
                  lookahead=2, steps=20, dist=("zipf", 0.9), seed=12)
    print(f"case never-used slots {fill}", flush=True)
    r = harness.run_parity(w, fill=fill, sync_each_step=False, check_fwd_steps=[0, 9, 19])
    assert r["stats"]["evictions"] == 0 and r["stats"]["misses"] > 0


@pytest.mark.parametrize("device_ids", [False, True])
@pytest.mark.parametrize("batch", [150, 400])  # about 4 MB and 11 MB of evicted rows a plan
def test_sorts_ahead_of_small_and_large_writebacks(harness, batch, device_ids):
    """Beside a write-back copy above 8 MiB the batches handed over ahead are sorted on the
    plan stream, at or below it on the ingest stream; the flush takes 7 and 17 pieces."""
    ids = batch * 40
    w = wl.custom(rows=[ids * 15 // 2], dim=256, batch=batch, pooling=40, slots=[ids * 17 // 8 + 1],
                  lookahead=1, steps=7, dist=("uniform",), seed=batch)
    print(f"case sorts ahead, batch {batch}, device_ids {device_ids}", flush=True)
    r = harness.run_parity(w, fill="staged", device_ids=device_ids, prepare_ahead=2,
                           sync_each_step=False, check_fwd_steps=[0, 4, 6])
    assert r["stats"]["evictions"] > 3 * ids // 2


@pytest.mark.parametrize("fill", ["mapped", "staged"])
def test_flush_of_a_nearly_empty_scratchpad(harness, fill):
    """Slots for a million rows, a few used: the pieces of the flush (8 slots, as the largest
    batch has 8 IDs) that hold no row take no call of the runtime.  Such a call takes some
    5 us, 125k of them over half a second; the bound leaves a scan of the keys 50 ms."""
    import time
    import numpy as np
    import torch
    rows, dim = 1_000_000, 16
    host = sp.host_tables([rows], dim, fill)
    host[0][:] = 1.0
    ctx = sp.ScratchPipe([rows], dim, [rows], 0, host, 4, 8, fill=fill)
    print(f"case sparse flush {fill}", flush=True)
    try:
        ids = np.array([5, 999_999, 7, 7, 123_456, 0, 31, 64], np.int32)
        out = torch.zeros((4, dim), device="cuda:0")
        grad = torch.ones((4, dim), device="cuda:0")
        want = np.ones(rows, np.float32)
        for step in range(3):
            mine = (ids.astype(np.int64) + 1000 * step) % rows
            t = ctx.plan([(mine.astype(np.int32), np.array([0, 2, 4, 6, 8], np.int32))])
            ctx.forward(t, out)
            ctx.backward_update(t, grad, 0.25)
            np.subtract.at(want, mine, np.float32(0.25))
        took = []
        for _ in range(3):
            t0 = time.perf_counter()
            ctx.flush()
            took.append(time.perf_counter() - t0)
        assert np.array_equal(host[0], np.repeat(want, dim).reshape(rows, dim))
        assert min(took) < 0.05, took
    finally:
        ctx.close()
        host.close()

"""The Hit-Map's two forms (an entry per table row where that takes no more memory than the
hash, else the hash), queries of one, four and eight keys per thread, and slots taken from a
batch's entry into the window rather than looked up again."""
import numpy as np
import pytest

from paper_2205_04702_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def harness():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("rows", [900, 60_000])  # dense, hash
@pytest.mark.parametrize("policy,prefetch,hold_past", [("lru", 0, 0), ("lfu", 0, 2),
                                                       ("random", 2, 1)])
def test_both_maps(harness, rows, policy, prefetch, hold_past):
    w = wl.custom(rows=[rows, rows, 700], dim=16, batch=30, pooling=[4, 3, 2],
                  slots=[450, 400, 300], lookahead=3, steps=20, dist=("zipf", 0.8), seed=rows)
    print(f"case rows {rows} {policy} prefetch {prefetch} hold_past {hold_past}", flush=True)
    r = harness.run_parity(w, policy=policy, prefetch=prefetch, hold_past=hold_past,
                           prepare_ahead=2)
    assert r["stats"]["evictions"] > 0


@pytest.mark.parametrize("ids", [100_000, 1_060_000])  # four keys per thread, eight
def test_query_of_many_keys(harness, ids):
    """Two tables, one batch entering per plan, with misses and evictions in every tile."""
    w = wl.custom(rows=[ids, ids // 3], dim=4, batch=100, pooling=[ids * 3 // 400, ids // 400],
                  slots=[ids * 4 // 5, ids // 3], lookahead=1, steps=4, seed=7)
    print(f"case many keys, nnz {w.nnz}", flush=True)
    r = harness.run_parity(w, prepare_ahead=1)
    assert r["stats"]["evictions"] > 0


def test_content_may_change_after_a_rejected_plan(harness):
    """A rejected plan has its window read again at the next call, also batches that an
    earlier plan entered: other content in their place is looked up anew."""
    import torch
    from oracle import oracle
    from paper_2205_04702_amd import scratchpipe as spm
    w = wl.custom(rows=[800, 1200], dim=8, batch=20, pooling=[3, 2], slots=[600, 700],
                  lookahead=2, steps=12, dist=("zipf", 1.0), seed=3)
    print("case changed content", flush=True)
    batches = harness.make_inputs(w)
    host = harness.fresh_host(w)
    ctx = spm.ScratchPipe(w.rows, w.dim, w.slots, w.lookahead, host, w.batch, 4096)
    out = torch.zeros((w.tables * w.batch, w.dim), device="cuda:0")
    ref = [wl.init_table(w, t) for t in range(w.tables)]
    try:
        for u in range(9):
            if u == 4:
                bad = batches[6][0].copy()
                bad[0] = -1
                with pytest.raises(spm.SPError):
                    ctx.plan([batches[4], batches[5], (bad, batches[6][1])])
                batches[4], batches[5] = batches[10], batches[11]  # entered before, now others
            t = ctx.plan(batches[u:u + 3])
            d = ctx.debug_plan(t, int(batches[u][0].size))
            # every position's slot holds its row: distinct rows have distinct slots
            assert np.all(d["slot_u"] >= 0) and np.unique(d["slot_u"]).size == d["slot_u"].size
            ctx.forward(t, out)
            g = wl.grads(w, u)
            ctx.backward_update(t, torch.from_numpy(g).to("cuda:0"), w.lr)
            want = oracle.train_step(ref, *batches[u], w.batch, g, w.lr, want_out=True)
            torch.cuda.synchronize()
            assert harness.row_rel_err(out.cpu().numpy(), want).max() <= harness.REL_TOL
        ctx.flush()
        for t in range(w.tables):
            assert harness.row_rel_err(host[t], ref[t]).max() <= harness.REL_TOL
    finally:
        ctx.close()
        host.close()

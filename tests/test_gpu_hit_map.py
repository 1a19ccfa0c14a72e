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


@pytest.mark.parametrize("kind", ["ids", "capacity"])
@pytest.mark.parametrize("prefetch,hold_past,fill", [(0, 0, "mapped"), (1, 0, "staged"),
                                                     (0, 2, "staged"), (2, 1, "mapped")])
def test_content_may_change_after_a_rejected_plan(harness, kind, prefetch, hold_past, fill):
    """A rejected plan has its window read again at the next call, also batches that an
    earlier plan entered.  Other content in their place has its cached rows held (here the
    least recently used ones, the next victims if they were not) and may ask for rows that
    an earlier plan of the old window evicted; the old content's rows are held no more.
    The slots are few more than a window needs, and all used long before."""
    import torch
    from oracle import oracle
    from paper_2205_04702_amd import scratchpipe as spm
    B, L, steps = 10, 2, 18
    rows = [400, 300]
    slots = [45 * (L + 1 + hold_past), 32 * (L + 1 + hold_past)]  # 40 and 30 rows a batch
    w = wl.custom(rows=rows, dim=8, batch=B, pooling=[4, 3], slots=slots, lookahead=L, steps=steps,
                  seed=3)
    print(f"case changed content {kind} prefetch {prefetch} hold_past {hold_past} {fill}", flush=True)
    rng = np.random.default_rng(4)
    off = wl.fixed_offsets(B, [4, 3])

    def ids_of(*per_table):
        return np.concatenate([np.asarray(x, np.int32) for x in per_table]), off

    batches = [ids_of(*(rng.choice(r, n * B, replace=False) for r, n in zip(rows, (4, 3))))
               for _ in range(steps)]
    bad = batches[0][0].copy()
    bad[-1] = rows[1]
    fat = (np.concatenate([np.arange(slots[0] + 5, dtype=np.int32) % rows[0], np.zeros(3 * B, np.int32)]),
           np.concatenate([[0], np.full(B, slots[0] + 5),
                           slots[0] + 5 + 3 * np.arange(1, B + 1)]).astype(np.int32))
    host = harness.fresh_host(w, fill)
    ref = [wl.init_table(w, t) for t in range(w.tables)]
    planner = oracle.Planner(rows, slots, prefetch=prefetch)
    ctx = spm.ScratchPipe(rows, w.dim, slots, L, host, B, 1024, hold_past=hold_past,
                          prefetch=prefetch, fill=fill)
    out = torch.zeros((w.tables * B, w.dim), device="cuda:0")
    evicted = 0
    try:
        for u in range(steps):
            win = batches[u:u + L + 1]
            if u in (8, 12):
                past = batches[max(0, u - hold_past):u]
                with pytest.raises(spm.SPError) as e:
                    ctx.plan(win[:2] + [(bad, off)])
                assert e.value.status == spm.SP_ERR_INVALID_ARG
                if kind == "capacity":  # batch u is read again, so it may have another shape
                    with pytest.raises(spm.SPError) as e:
                        ctx.plan([fat] + win[1:])
                    assert e.value.status == spm.SP_ERR_CAPACITY
                    with pytest.raises(oracle.PlanError):
                        planner.plan([fat] + win[1:], B, past=past)
                # batches u and u + 1 were entered by plan u - 1; now others: least recently
                # used rows, rows that plan u - 1 evicted, and rows not cached
                new = [[], []]
                for t, n in enumerate((4 * B, 3 * B)):
                    a, z = (0, 4 * B) if t == 0 else (4 * B, 7 * B)
                    kos, lu, sor = planner.state(t)
                    old = np.concatenate([b[0][a:z] for b in batches[u:u + 2]])
                    lru = [r for r in kos[np.lexsort((np.arange(kos.size), lu))] if r not in old]
                    gone = last.v_old_row[(last.m_table == t) & (last.v_old_row >= 0)][:n // 4]
                    out_of = rng.permutation(np.setdiff1d(np.nonzero(sor < 0)[0], gone))
                    for q in range(2):
                        h = lru[q * (n // 4):(q + 1) * (n // 4)]
                        g = gone if q == 0 else gone[:0]
                        rest = out_of[q * n:q * n + n - len(h) - g.size]
                        new[q].append(rng.permutation(np.concatenate([h, g, rest])))
                batches[u], batches[u + 1] = ids_of(*new[0]), ids_of(*new[1])
                win = batches[u:u + L + 1]
            t = ctx.plan(win)
            last = planner.plan(win, B, past=batches[max(0, u - hold_past):u])
            harness.compare_plan(u, ctx.debug_plan(t, batches[u][0].size), last, w.tables, B)
            if u in (8, 12):  # least recently used hits beside as many misses: unheld, they would go
                assert last.hit.sum() >= 15 and last.m_row.size > 15
            evicted += last.n_evict
            ctx.forward(t, out)
            g = wl.grads(w, u)
            ctx.backward_update(t, torch.from_numpy(g).to("cuda:0"), w.lr)
            want = oracle.train_step(ref, *batches[u], B, g, w.lr, want_out=True)
            if u % 4 == 0:
                torch.cuda.synchronize()
                assert harness.row_rel_err(out.cpu().numpy(), want).max() <= harness.REL_TOL
        assert evicted > 20 * 8
        ctx.flush()
        for t in range(w.tables):
            assert harness.row_rel_err(host[t], ref[t]).max() <= harness.REL_TOL
    finally:
        ctx.close()
        host.close()

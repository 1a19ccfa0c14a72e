"""The multi-launch ingest (tables above 8192 IDs, or no bound promised) at the edges of its
tiles, digits and runs, against the oracle: plans bit for bit, outputs and tables per row."""
import pytest

from paper_2205_04702_amd import workload as wl

pytestmark = pytest.mark.gpu

# rows per table, bags per table, IDs per bag of each table
CASES = {
    # one digit, exactly one digit, one more; tables of one entry, a tile, a tile +- 1
    "digits": ([1, 2, 3, 511, 512, 513, 1025], 1, [7, 1, 1023, 1024, 1025, 4096, 4097]),
    # two and three passes beside one; runs that reach over several tiles
    "passes": ([5, 1 << 18, (1 << 18) + 1, 40], 16, [320, 64, 65, 1]),
    # the long tiles (from 2^19 IDs), runs of thousands, 64 bags and more per wave
    "long": ([3, 300_000, 1, 900], 67, [3000, 4100, 61, 700]),
    # few bags of many IDs: several waves share the positions of 64 bags
    "fat": ([300, 5000, 40], 3, [511, 513, 4000]),
    "fattest": ([9000], 1, [20_001]),
    "fat long": ([300_000, 70], 64, [8200, 100]),
    # every table its own
    "many": ([17 + 13 * t for t in range(64)], 33, [1 + t % 40 for t in range(64)]),
}


@pytest.mark.parametrize("device_ids", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_general_ingest_edges(name, device_ids):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    rows, batch, pooling = CASES[name]
    w = wl.custom(rows=rows, dim=16, batch=batch, pooling=pooling, slots=rows, lookahead=1, steps=3,
                  dist=("zipf", 1.05), seed=len(name))
    print(f"case {name} nnz {w.nnz} device_ids {device_ids}", flush=True)
    gpu_harness.run_parity(w, max_table_ids=0, device_ids=device_ids, prepare_ahead=1)


@pytest.mark.parametrize("ids", [300_000, 1_100_000, 2_200_000, 4_400_000])  # 2, 2, 4, 8 tiles
def test_general_ingest_groups_of_tiles(ids):
    """One long table between short ones, its tiles counted in groups, the last one partly filled."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    rows, bags = [300, ids // 3, 5000], 100
    w = wl.custom(rows=rows, dim=4, batch=bags, pooling=[3, ids // bags, 41], slots=rows,
                  lookahead=0, steps=2, dist=("zipf", 0.9), seed=9)
    print(f"case groups of tiles, nnz {w.nnz}", flush=True)
    gpu_harness.run_parity(w, max_table_ids=0)


@pytest.mark.parametrize("longest", [1, 9, 200])
def test_general_ingest_ragged(longest):
    """Bags of 0..longest IDs: empty ones at either end of a wave's 64, long ones across its steps."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    w = wl.custom(rows=[700, 90, 3000], dim=8, batch=130, pooling=4, slots=[700, 90, 3000],
                  lookahead=1, steps=4, dist=("zipf", 1.1), seed=longest)
    print(f"case ragged {longest}", flush=True)
    gpu_harness.run_parity(w, gpu_harness.make_inputs(w, ragged=longest), max_table_ids=0)


def test_general_ingest_few_ragged_bags():
    """Bags of 0..3000 IDs, few enough that several waves share them."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    w = wl.custom(rows=[700, 90, 3000], dim=8, batch=11, pooling=4, slots=[700, 90, 3000],
                  lookahead=1, steps=4, dist=("zipf", 1.1), seed=6)
    print("case few ragged bags", flush=True)
    gpu_harness.run_parity(w, gpu_harness.make_inputs(w, ragged=3000), max_table_ids=0)


def test_general_ingest_time_does_not_follow_the_bag_length():
    """128k IDs as 64 bags of 2000 or as 2000 bags of 64: the same sort and as many positions
    to mark, so about the same time (0.07 and 0.06 ms); as one wave's walk the first took 0.60 ms."""
    import torch
    from paper_2205_04702_amd import scratchpipe as sp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    took = []
    out = torch.zeros((2000, 4), device="cuda:0")
    for batch, pool in ((16, 2000), (500, 64)):
        w = wl.custom(rows=[20_000] * 4, dim=4, batch=batch, pooling=pool, slots=[20_000] * 4,
                      lookahead=0, steps=12, dist=("zipf", 1.05), seed=8)
        print(f"case ingest time {batch} x {pool}", flush=True)
        host = sp.host_tables(w.rows, w.dim)
        batches = [tuple(torch.from_numpy(x).to("cuda:0") for x in wl.batch(w, u))
                   for u in range(w.steps)]
        torch.cuda.synchronize()
        ctx = sp.ScratchPipe(w.rows, w.dim, w.slots, 0, host, batch, w.nnz)
        for u in range(w.steps):
            if u == 4:  # the first steps load the kernels
                ctx.set_flags(sp.SP_FLAG_TIMING)
            ctx.forward(ctx.plan([batches[u]]), out)
            ctx.backward_update(u, out, 0.0)
        st = ctx.stats()
        ctx.close()
        host.close()
        took.append(st["ms_ingest"] / st["timed_ingest"])
    print("ms per ingest", took)
    assert took[0] < 2.5 * took[1], took

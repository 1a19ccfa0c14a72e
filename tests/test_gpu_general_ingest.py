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

"""The update of rows whose runs span several chunks, against the oracle: a block per run up to
a number of such runs that grows with the row width, a wave per run above it, with a hot
row of thousands of chunks, several in one block, and runs of two chunks beside them."""
import numpy as np
import pytest

from paper_2205_04702_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,runs", [(4, 4096), (4, 4097), (16, 1), (16, 4097), (64, 4096),
                                      (64, 4097), (128, 8192), (128, 8193), (256, 16384),
                                      (256, 16385)])
def test_runs_of_several_chunks(dim, runs):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    rng = np.random.default_rng(runs)
    count = np.full(runs, 17)            # two chunks
    count[0] = 20_000                    # the whole block's, in the form of a wave per run
    count[1:6] = 64 * 16 + np.arange(5)[:runs - 1]  # 64 chunks, and 65, one block's
    count[7:40] = rng.integers(18, 3000, 33)[:max(0, runs - 7)]
    bags = 400
    w = wl.custom(rows=[runs + 300], dim=dim, batch=bags, pooling=1, slots=[runs + 300], lookahead=0,
                  steps=2, dist=("uniform",), seed=runs)
    batches = []
    for _ in range(w.steps):
        ids = np.concatenate([np.repeat(np.arange(runs), count), runs + np.arange(300)])
        ids = rng.permutation(ids).astype(np.int32)
        off = np.linspace(0, ids.size, bags + 1).astype(np.int32)
        batches.append((ids, off))
    print(f"case dim {dim}, {runs} runs above a chunk", flush=True)
    gpu_harness.run_parity(w, batches, max_table_ids=0)

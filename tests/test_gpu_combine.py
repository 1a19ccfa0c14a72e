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


@pytest.mark.parametrize("tables,rows,dim,batch,pool,fwd,upd", [
    (4, 3000, 16, 3000, 90, 7.6e-8, 2.8e-8), (4, 3000, 32, 3000, 90, 8.9e-8, 2.8e-8),
    (64, 300, 256, 4000, 60, 7.4e-8, 4.7e-8)])
def test_sums_are_as_close_to_64_bits(tables, rows, dim, batch, pool, fwd, upd):
    """Relative error (2-norm) of one forward and of the updated tables against sums in 64 bits.
    An add's rounding error has a variance in proportion to its result's, so n values in c
    chains, k of them added to one another before each add of a chain, have one in proportion
    to n^2 / (2 c k) + 3 n: 90 rows with c k = 16 and 8 (16 and 32 floats) 7.3e-8 and 8.0e-8,
    with half of that 8.0e-8 and 9.7e-8; runs of 50 chunks of 256 floats in trees of 8 4.1e-8,
    one by one 5.2e-8.  The bounds lie between."""
    import torch
    from paper_2205_04702_amd import scratchpipe as sp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case error {tables} x {rows} x {dim}, {batch} bags of {pool}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    bags, lr = tables * batch, 0.01
    off = (torch.arange(bags + 1, device=dev) * pool).int()
    ids = torch.randint(rows, (bags * pool,), generator=g, device=dev, dtype=torch.int32)
    weights = torch.randn((tables, rows, dim), generator=g, device=dev)
    grad = torch.randn((bags, dim), generator=g, device=dev)
    host = sp.host_tables([rows] * tables, dim)
    for t in range(tables):
        torch.from_numpy(host[t]).copy_(weights[t])
    out = torch.zeros((bags, dim), device=dev)
    torch.cuda.synchronize()
    ctx = sp.ScratchPipe([rows] * tables, dim, [rows] * tables, 0, host, batch, int(ids.numel()))
    try:
        t = ctx.plan([(ids, off)])
        ctx.forward(t, out)
        ctx.backward_update(t, grad, lr)
        ctx.flush()
        bag = torch.arange(bags, device=dev).repeat_interleave(pool)
        key = bag // batch * rows + ids.long()
        weights = weights.view(tables * rows, dim).double()
        want_out = torch.zeros((bags, dim), dtype=torch.float64, device=dev)
        want = weights.clone()
        for a in range(0, key.numel(), 1 << 20):
            k, b = key[a:a + (1 << 20)], bag[a:a + (1 << 20)]
            want_out.index_add_(0, b, weights[k])
            want.index_add_(0, k, grad[b].double(), alpha=-lr)
        got = torch.cat([torch.from_numpy(host[t]).to(dev) for t in range(tables)]).double()
    finally:
        ctx.close()
        host.close()
    errs = [float((x.double() - y).norm() / y.norm()) for x, y in ((out, want_out), (got, want))]
    print("relative errors", errs)
    assert errs[0] < fwd and errs[1] < upd, errs

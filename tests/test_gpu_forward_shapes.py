"""The forward's three forms against the oracle: a group of lanes per bag, a whole wave per bag
(few bags, or long ones), and groups whose block's waves take the long bags among short
ones; at the lengths where one passes into another, for every row width."""
import numpy as np
import pytest

from paper_2205_04702_amd import scratchpipe as sp
from paper_2205_04702_amd import workload as wl

pytestmark = pytest.mark.gpu
DIMS = [4, 8, 16, 32, 64, 128, 256]


@pytest.fixture(scope="module")
def harness():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_harness
    return gpu_harness


def batch_of(rng, rows, lens):
    """One table of len(lens) bags."""
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return rng.integers(0, rows, int(off[-1])).astype(np.int32), off


def skewed(rng, bags):
    """Short bags; single long ones, two in one block, a block of nothing but long ones, and
    the lengths around FWD_LONG = 128."""
    lens = rng.integers(0, 5, bags)
    lens[[0, 7, 700, 1500, 1501, bags - 1]] = [128, 129, 2500, 300, 900, 1000]
    lens[2048:2048 + 32] = 130 + np.arange(32)
    lens[3072:3072 + 5] = 640
    return lens


SHAPES = {  # bag lengths, for a seed
    "few long": lambda r: [1, 0, 2000, 513, 64, 65, 63],
    "few short": lambda r: r.integers(0, 8, 40),                 # mean below 16: groups
    "mean 16": lambda r: np.full(4096, 16),                      # the last whole-wave shape
    "mean 16, more": lambda r: np.full(4097, 16),                # groups
    "mean 100": lambda r: np.full(4099, 100),                    # whole waves
    "mean below 100": lambda r: np.append(np.full(4098, 100), 0),
    "skewed": lambda r: skewed(r, 4999),
}


@pytest.mark.parametrize("dim", DIMS)
@pytest.mark.parametrize("shape", list(SHAPES))
def test_forms(harness, shape, dim):
    rng = np.random.default_rng(len(shape))
    rows = 900
    batches = [batch_of(rng, rows, SHAPES[shape](rng)) for _ in range(2)]
    bags = batches[0][1].size - 1
    w = wl.custom(rows=[rows], dim=dim, batch=bags, pooling=[1], slots=[rows], lookahead=0, steps=2,
                  seed=1)
    print(f"case forward {shape} dim {dim} bags {bags}", flush=True)
    for bound in (0, "auto") if shape != "skewed" else (0,):
        harness.run_parity(w, batches, max_table_ids=bound)


def test_long_bags_are_seen_by_the_one_launch_ingest(harness):
    """Short bags with long ones among them in tables of up to 8192 IDs."""
    rng = np.random.default_rng(5)
    lens = rng.integers(0, 3, (2, 4500))
    lens[0, 17] = lens[1, 4499] = 1500
    lens[1, 100] = 129
    batches = []
    for _ in range(3):
        off = np.concatenate([[0], np.cumsum(lens.ravel())]).astype(np.int32)
        batches.append((rng.integers(0, 700, int(off[-1])).astype(np.int32), off))
    w = wl.custom(rows=[700, 800], dim=16, batch=4500, pooling=[1, 1], slots=[700, 800], lookahead=1,
                  steps=3, seed=2)
    print("case long bags, one-launch ingest", flush=True)
    assert harness.table_bound(w, batches) <= 8192
    harness.run_parity(w, batches)


def forward_us(dim, batches, bags, rows):
    import torch
    dev = [tuple(torch.from_numpy(x).to("cuda:0") for x in b) for b in batches]
    host = sp.host_tables([rows], dim)
    torch.cuda.synchronize()
    ctx = sp.ScratchPipe([rows], dim, [rows], 0, host, bags, max(b[0].size for b in batches))
    out = torch.zeros((bags, dim), device="cuda:0")
    for u in range(16):
        if u == 4:  # the first steps load the kernels
            ctx.set_flags(sp.SP_FLAG_TIMING)
        ctx.forward(ctx.plan([dev[u % len(dev)]]), out)
        ctx.backward_update(u, out, 0.0)
    st = ctx.stats()
    ctx.close()
    host.close()
    return 1e3 * st["ms_forward"] / st["timed_forward"]


@pytest.mark.parametrize("shape", ["few", "skewed"])
def test_narrow_rows_are_no_slower_than_wide_ones(harness, shape):
    """The same bags of 32 floats a row and of 128: with few lanes on a long bag the narrow
    rows took longer (64 bags of 2000: 307 and 242 us; one bag in 200 of 1000: 146 and 129)."""
    rng = np.random.default_rng(9)
    lens = np.full(64, 2000)
    if shape == "skewed":
        lens = rng.integers(1, 5, 53_248)
        lens[rng.random(lens.size) < 0.005] = 1000
    rows = 100_000
    batches = [batch_of(rng, rows, lens) for _ in range(2)]
    print(f"case forward time {shape}", flush=True)
    narrow, wide = (forward_us(d, batches, lens.size, rows) for d in (32, 128))
    print("forward us", narrow, wide)
    assert narrow < 0.85 * wide, (narrow, wide)

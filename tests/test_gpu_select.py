"""Victim choice at the edges of its kernels: one block per table (tables of up to 16384 slots
with up to 8192 victims), the levels and the compaction over all tables with the sort in one
block, and the global sort; one to three digits of priority.  Plans bit for bit."""
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


# slots per table, rows, IDs per bag of each table (one bag row of 64)
CASES = {
    "waves": ([63, 64, 65, 1023, 1024, 1025], [200, 210, 220, 3000, 3000, 3000], [0, 0, 0, 5, 5, 5]),
    "few": ([130, 200], [300, 450], [1, 1]),
    "most": ([16_384, 9000], [60_000, 9100], [130, 60]),      # up to 8192 victims in one block
    "slots": ([16_385, 500], [60_000, 900], [130, 2]),        # one slot more than it takes
    "above": ([30_000, 400], [90_000, 900], [200, 2]),        # more than 8192: the global sort
    "large": ([140_000, 500], [180_000, 900], [600, 2]),
}


@pytest.mark.parametrize("policy", ["lru", "lfu", "random"])
@pytest.mark.parametrize("name", list(CASES))
def test_victims(harness, name, policy):
    slots, rows, pooling = CASES[name]
    batch = 64
    pooling = [p if p else 1 for p in pooling]
    w = wl.custom(rows=rows, dim=4, batch=batch if name != "waves" else 32, pooling=pooling,
                  slots=slots, lookahead=0, steps=14 if name == "large" else 12, seed=len(name))
    print(f"case {name} {policy}", flush=True)
    r = harness.run_parity(w, policy=policy, seed=5)
    assert r["stats"]["evictions"] > 0


def test_two_digits_of_priority(harness):
    """Past plan 2048 LRU priorities take two levels."""
    w = wl.custom(rows=[90], dim=4, batch=3, pooling=[2], slots=[21], lookahead=1, steps=2080)
    print("case two digits", flush=True)
    r = harness.run_parity(w, check_fwd_steps=range(0, 2080, 40), sync_each_step=False)
    assert r["stats"]["evictions"] > 0

"""Performance cases: stretches of embedding training through the public entry points.

One pass trains the next few mini-batches of a stream the way a training loop does: for each
batch ScratchPipe.plan over its look-forward window (two batches more are handed over early
for sorting), forward, backward_update.  The context, its host tables, the batches and the
upstream gradients are what the program holds before the pass; the context has trained one
round of the stream with a zero learning rate, so its scratchpad is in steady state and the
tables still hold their initial values.  The stream repeats after `batches` batches, as
epochs do.  A pass returns the pooled outputs of its steps (later steps gather rows that
earlier ones updated) and, where it ends with a checkpoint, the host tables.

Every value is drawn on the GPU from the seed: IDs uniform or Zipf over a permutation of the
rows, weights U[-0.05, 0.05), gradients N(0, 1).
"""
import functools
import math

import numpy as np
import torch

from paper_2205_04702_amd import scratchpipe as sp

LR = 0.01


def _case(name=None, **kw):
    c = dict(tables=8, rows=100_000, rows_to=0, dim=64, batch=1024, pool=8, pool_to=0, alpha=1.05,
             slots=0, lookahead=3, batches=16, steps=8, policy="lru", prefetch=0, hold_past=0,
             fill="mapped", ids="device", ragged=False, bound=True, static=False, flush=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one small table wholly in the scratchpad, a handful of IDs
        _case("one-table-resident-d16", tables=1, rows=1000, dim=16, batch=16, pool=2, alpha=0.0,
              lookahead=2, batches=12, static=True),
        # the repository's tiny configuration: uniform IDs, most rows miss
        _case("tiny-4x20k-d32", tables=4, rows=20_000, dim=32, batch=128, pool=4, alpha=0.0,
              slots=2048, lookahead=2, batches=24),
        # the benchmark's 8x1M configuration at its full size: a third of the rows miss
        _case("zipf-8x1M-d64", tables=8, rows=1_000_000, dim=64, batch=1024, pool=8,
              slots=100_000, lookahead=3, batches=64),
        # recommendation tables with one ID per sample, LFU, the IDs in host memory
        _case("onehot-26x60k-d16-lfu", tables=26, rows=60_000, dim=16, batch=2048, pool=1,
              alpha=0.8, slots=9000, lookahead=4, batches=24, policy="lfu", ids="host"),
        # odd sizes: ragged and empty bags, wide rows, prefetch and a past window
        _case("ragged-5x50k-d256-prefetch", tables=5, rows=50_000, dim=256, batch=777, pool=13,
              slots=17_001, lookahead=3, batches=16, steps=4, prefetch=1, hold_past=1,
              ragged=True, bound=False),
        # narrow rows, random eviction, more IDs per table than the one-launch sort takes
        _case("random-16x200k-d8", tables=16, rows=200_000, dim=8, batch=1500, pool=10, alpha=0.0,
              slots=80_000, lookahead=2, batches=12, steps=4, policy="random"),
        # batches of the benchmark's 26x4M configuration (rows scaled), staged fill, a quarter
        # of the rows miss
        _case("zipf-26x150k-d128-staged", tables=26, rows=150_000, dim=128, batch=2048, pool=20,
              alpha=1.1, slots=50_000, lookahead=4, batches=16, steps=4, fill="staged"),
        # batches of the benchmark's 26x10M configuration, eight of its tables (rows scaled)
        _case("zipf-8x400k-d128-staged", tables=8, rows=400_000, dim=128, batch=4096, pool=40,
              alpha=0.9, slots=160_000, lookahead=4, batches=12, steps=2, fill="staged"),
        # tables that fit the scratchpad: nothing misses, the IDs in host memory
        _case("resident-26x20k-d64-hostids", tables=26, rows=20_000, dim=64, batch=2048, pool=4,
              batches=8, ids="host"),
        # batches of the benchmark's mixed configuration (rows scaled): 64 tables of very
        # different sizes and poolings, uniform and Zipf, all of them in the scratchpad
        _case("mixed-64t-d64-resident", tables=64, rows=1000, rows_to=400_000, dim=64, batch=8192,
              pool=1, pool_to=80, alpha=1.2, lookahead=6, batches=6, steps=2),
        # batches of the benchmark's 26x10M configuration, every row in the scratchpad
        _case("zipf-26x80k-d128-resident", tables=26, rows=80_000, dim=128, batch=4096, pool=40,
              alpha=0.9, lookahead=4, batches=8, steps=3),
        # a few steps, then a checkpoint: every cached row back to its host table
        _case("checkpoint-4x50k-d64", tables=4, rows=50_000, dim=64, batch=512, pool=8,
              slots=8000, lookahead=2, batches=32, steps=4, fill="staged", flush=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        size = rng.choice(["small", "medium", "large"])
        if size == "small":
            c = _case(tables=rng.randint(1, 16), rows=_log_int(rng, 500, 100_000),
                      dim=rng.choice([4, 8, 16, 32, 64, 128, 256]), batch=_log_int(rng, 1, 700),
                      pool=rng.randint(1, 12), steps=8)
        elif size == "medium":
            c = _case(tables=rng.randint(4, 32), rows=_log_int(rng, 10_000, 200_000),
                      dim=rng.choice([16, 32, 64, 128]), batch=_log_int(rng, 500, 4000),
                      pool=rng.randint(1, 24), steps=4)
        else:
            c = _case(tables=rng.randint(8, 40), rows=_log_int(rng, 10_000, 150_000),
                      dim=rng.choice([32, 64, 128]), batch=rng.randint(2000, 4200),
                      pool=rng.randint(16, 48), steps=2)
        c["alpha"] = rng.choice([0.0, 1.0, 1.0]) * round(rng.uniform(0.8, 1.2), 3)
        c["lookahead"] = rng.randint(0, 5)
        c["policy"] = rng.choice(["lru", "lru", "lru", "lfu", "random"])
        c["prefetch"] = rng.choice([0, 0, 0, 1, 2])
        c["hold_past"] = rng.choice([0, 0, 0, 1, 3])
        c["fill"] = rng.choice(["mapped", "staged"])
        c["ids"] = rng.choice(["device", "device", "host"])
        c["ragged"] = rng.random() < 0.3
        c["bound"] = rng.random() < 0.8
        if size != "small" and rng.random() < 0.2:
            c["rows_to"], c["pool_to"] = c["rows"] * 4, c["pool"] * 2
        c["batches"] = 8
        if rng.random() < 0.6:  # evicting: room for the window's rows, not for the stream's
            ids = _bag_max(c) * c["batch"]
            window = c["lookahead"] + 1 + c["hold_past"]
            least = 1.2 * _table_traffic(c["rows"], window * ids, c["alpha"], c["rows"], 1)[0] + 64
            most_used = 0.9 * _table_traffic(c["rows"], 24 * ids, c["alpha"], c["rows"], 1)[0]
            if least < most_used:
                c["slots"], c["batches"] = int(rng.uniform(least, most_used)), 24
                c["rows_to"] = c["pool_to"] = 0
        if _table_bytes(c) <= 1.8e9 and _cost(c) <= 0.8 * most:
            return c


# ------------------------------------------------------------------ shapes

def _rows(c):
    if not c["rows_to"]:
        return [c["rows"]] * c["tables"]
    f = (c["rows_to"] / c["rows"]) ** (1.0 / max(1, c["tables"] - 1))
    return [int(c["rows"] * f ** ((t * 7) % c["tables"])) for t in range(c["tables"])]


def _pools(c):
    if not c["pool_to"]:
        return [c["pool"]] * c["tables"]
    n = c["pool_to"] - c["pool"] + 1
    return [c["pool"] + (t * 29) % n for t in range(c["tables"])]


def _alphas(c):  # of tables of many sizes, every other one draws uniformly
    return [0.0 if c["rows_to"] and t % 2 else c["alpha"] for t in range(c["tables"])]


def _slots(c):
    return [min(r, c["slots"]) if c["slots"] else r for r in _rows(c)]


def _bag_max(c):
    return 2 * c["pool"] if c["ragged"] else c["pool"]


def _table_bytes(c):
    return sum(_rows(c)) * c["dim"] * 4


def _probs(rows, alpha):
    w = np.arange(1, rows + 1, dtype=np.float64) ** -alpha
    return w / w.sum()


@functools.lru_cache(maxsize=4096)
def _table_traffic(rows, ids, alpha, slots, batches):
    if not alpha:  # one probability for every row
        q, many = np.array([-math.expm1(ids * math.log1p(-min(1 / rows, 1 - 1e-12)))]), rows
    else:
        q, many = -np.expm1(ids * np.log1p(-np.minimum(_probs(rows, alpha), 1 - 1e-12))), 1
    uniq = many * q.sum()
    if slots >= rows or many * (1 - (1 - q) ** batches).sum() <= slots:
        return uniq, 0.0
    lo, hi = 0.0, float(batches)  # steps whose distinct rows fill the slots
    for _ in range(16):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if many * (1 - (1 - q) ** mid).sum() < slots else (lo, mid)
    return uniq, many * (q * (1 - q) ** lo).sum()


def _traffic(c):
    """Expected unique rows and misses of one step (all tables)."""
    uniq = miss = 0.0
    for r, p, a, s in zip(_rows(c), _pools(c), _alphas(c), _slots(c)):
        x = _table_traffic(r, c["batch"] * p, a, s, c["batches"])
        uniq, miss = uniq + x[0], miss + x[1]
    return float(uniq), float(miss)


def _step_bytes(c):
    """HBM and host-link bytes of one step: IDs and offsets once, each unique row read by the
    forward and read and written by the update, outputs and gradients once; a missing row
    from the host into HBM and the row it evicts back."""
    uniq, miss = _traffic(c)
    row = 4 * c["dim"]
    nnz = c["batch"] * sum(_pools(c))
    bags = c["tables"] * c["batch"]
    hbm = nnz * 4 + bags * 4 + uniq * row * 3 + bags * row * 2 + miss * row * 2
    return hbm, miss * row * 2


def _cost(c):
    hbm, link = _step_bytes(c)
    return c["steps"] * (hbm / 3e12 + link / 80e9 + c["batch"] * sum(_pools(c)) * 1e-10)


def work(case):
    hbm, link = _step_bytes(case)
    uniq, _ = _traffic(case)
    nnz = case["batch"] * sum(_pools(case))
    total = case["steps"] * (hbm + link)
    if case["flush"]:
        total += 2 * sum(_slots(case)) * case["dim"] * 4
    return {"bytes": total, "flops": case["steps"] * (2 * nnz + 2 * uniq) * case["dim"]}


# ------------------------------------------------------------------ inputs

def _inputs(case, seed):
    """Initial tables, batches (ids, bag offsets) and gradients, all on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + 17)
    rows, pools, alphas = _rows(case), _pools(case), _alphas(case)
    T, B, D, N = case["tables"], case["batch"], case["dim"], case["batches"]
    tables = [torch.rand((r, D), generator=g, device="cuda").mul_(0.1).sub_(0.05) for r in rows]
    lens = torch.tensor(pools, device="cuda").repeat_interleave(B)
    all_off, counts = [], []
    for _ in range(N):
        n = lens
        if case["ragged"]:
            n = (torch.rand(T * B, generator=g, device="cuda") * 2 * lens).floor().long() + 1
            n = n * (torch.rand(T * B, generator=g, device="cuda") > 0.1)
        all_off.append(torch.nn.functional.pad(n.cumsum(0), (1, 0)).int())
        counts.append(n.view(T, B).sum(1))
    counts = torch.stack(counts).cpu().tolist()
    parts = [[] for _ in range(N)]
    for t in range(T):
        perm = torch.randperm(rows[t], generator=g, device="cuda").int()
        if alphas[t]:
            w = torch.arange(1, rows[t] + 1, device="cuda", dtype=torch.float64) ** -alphas[t]
            cdf = w.cumsum(0)
            cdf /= cdf[-1].clone()
        total = sum(counts[s][t] for s in range(N))
        u = torch.rand(total, generator=g, device="cuda", dtype=torch.float64)
        k = torch.searchsorted(cdf, u) if alphas[t] else (u * rows[t]).long()
        ids = perm[k.clamp_(max=rows[t] - 1)]
        for s, x in enumerate(ids.split([counts[s][t] for s in range(N)])):
            parts[s].append(x)
    batches = [(torch.cat(p), off) for p, off in zip(parts, all_off)]
    grads = [torch.randn((T * B, D), generator=g, device="cuda") for _ in range(case["steps"])]
    most = max(max(c) for c in counts)  # IDs one table has in one batch
    return tables, batches, grads, most


class Session:
    """What a training program keeps: its host tables, the context and its inputs."""

    def __init__(self, case, seed):
        tables, batches, grads, most = _inputs(case, seed)
        self.case, self.grads = case, grads
        self.host = sp.host_tables(_rows(case), case["dim"], case["fill"])
        for t, w in enumerate(tables):
            torch.from_numpy(self.host[t]).copy_(w)
        if case["ids"] == "host":
            batches = [(i.cpu().numpy(), o.cpu().numpy()) for i, o in batches]
        self.batches = batches
        bags = case["tables"] * case["batch"]
        self.out = torch.zeros((case["steps"], bags, case["dim"]), device="cuda")
        self.ctx = sp.ScratchPipe(
            _rows(case), case["dim"], _slots(case), case["lookahead"], self.host,
            max_batch=case["batch"], max_ids=max(int(b[0].shape[0]) for b in batches),
            policy=case["policy"], hold_past=case["hold_past"], seed=seed,
            max_table_ids=most if case["bound"] else 0, prefetch=case["prefetch"],
            fill=case["fill"])
        self.step = 0
        torch.cuda.synchronize()  # the batches are read on the library's streams
        for _ in range(case["batches"]):
            self.train(self.out[0], 0, 0.0)
        self.ctx.sync()

    def train(self, out, i, lr):
        n, ctx = self.case["batches"], self.ctx
        ahead = self.case["lookahead"] + 1 + sp.SP_MAX_AHEAD
        ticket = ctx.plan([self.batches[(self.step + w) % n] for w in range(ahead)])
        ctx.forward(ticket, out)
        (ctx.backward_update_static if self.case["static"] else ctx.backward_update)(
            ticket, self.grads[i], lr)
        self.step += 1

    def close(self):
        ctx, self.ctx = getattr(self, "ctx", None), None
        if ctx is not None:
            ctx.close()
            self.host.close()

    def __del__(self):
        self.close()


def prepare(case, seed):
    return Session(case, seed)


def run(state):
    for i in range(state.case["steps"]):
        state.train(state.out[i], i, LR)
    if not state.case["flush"]:
        return {"pooled": state.out}
    state.ctx.flush()
    return {"pooled": state.out, "tables": [state.host[t] for t in range(len(state.host))]}


def exact(case, seed):
    tables, batches, grads, _ = _inputs(case, seed)
    T, B, N = case["tables"], case["batch"], case["batches"]
    tables = [t.double() for t in tables]
    outs = []
    for i in range(case["steps"]):
        ids, off = batches[i % N]  # the pass starts at a whole round of the stream
        off = off.long()
        bag = torch.repeat_interleave(torch.arange(T * B, device="cuda"), off.diff())
        g = grads[i].double()
        out = torch.zeros((T * B, case["dim"]), dtype=torch.float64, device="cuda")
        edges = off[::B].cpu().tolist()
        for t in range(T):
            rows, b = ids[edges[t]:edges[t + 1]].long(), bag[edges[t]:edges[t + 1]]
            out.index_add_(0, b, tables[t][rows])
            tables[t].index_add_(0, rows, g[b], alpha=-LR)
        outs.append(out)
    res = {"pooled": torch.stack(outs)}
    if case["flush"]:
        res["tables"] = tables
    return res


def tolerance(case):
    # fp32 sums in another order: up to 2.7e-7 from 64 bits was seen
    return {"rel": 1e-6, "max": 4e-5}

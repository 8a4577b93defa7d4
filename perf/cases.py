"""Workloads of the tiered pooled-embedding lookup for timing its public calls.

A case is what a serving or inference program does per batch: apply the
decisions for the next batch to the HBM cache (TieredEmbeddingCache.placement)
and look the batch up (TieredEmbeddingCache.forward), or the lookup alone where
the decisions come late.  Accesses follow a bounded Zipf law, prefetch lists
name the next batch's rows (all of them, or a share beside random ones), and
caching bits say which rows the next two batches use again, 17% of them wrong.

The inputs come from the seed alone.  Every pass takes the next batch of a ring,
on a cache that warm-up placements have filled with its tables' popular rows and
that has already served two batches.
"""
import functools
import math

import numpy as np
import torch

from paper_2511_08568_amd import TieredEmbeddingCache

WARM_BATCHES = 2  # batches a prepared cache has served
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, **kw):
    c = dict(name=name, tables=1, rows_lo=100_000, rows_hi=100_000, dims="64", dtypes="f32", cache=0.1, alpha=1.05,
             bags=256, pooling="fixed 20", onehot=0, policy="lru", ways=0, prefetch="none", miss="zero_copy",
             calls="step", pipelined=False, ring=8)
    assert set(kw) <= set(c)
    c.update(kw)
    return c


def listed():
    return [
        # one online request on a handful of small tables that fit the cache:
        # the smallest lookup, whose latency a caller waits for
        _case("request forward", tables=4, rows_lo=10_000, rows_hi=10_000, dims="32", cache=1.0, bags=16,
              pooling="poisson 8", calls="forward", ring=32),
        # the small configuration of this repository (100,000 x 64 rows, 10,000
        # cached, 256 bags of 20, 20% of the prefetch list random), as a program
        # that runs both calls on one stream has it
        _case("small step", prefetch="replace 0.2", ring=32),
        # the same on the 32-way buffer of production systems, counters read
        # after every batch by a program that watches its hit rate
        _case("small step 32-way watched", prefetch="replace 0.2", ways=32, calls="step+stats", ring=32),
        # a ragged mix: dims that are no power of two, all three storage types,
        # one-hot features beside multi-hot ones
        _case("ragged step", tables=13, rows_lo=1_003, rows_hi=300_007, dims="17,50,100,200,36", dtypes="f32,f16,bf16",
              cache=0.2, alpha=1.0, bags=1000, pooling="poisson 7", onehot=4, policy="priority", prefetch="mix 0.7"),
        # a batch looked up while the next decisions are late: what the cache
        # does not hold is fetched on demand and stays out
        _case("late decisions forward", tables=8, rows_lo=1_000_000, rows_hi=1_000_000, dims="128", cache=0.2,
              alpha=1.1, bags=2048, pooling="poisson 40", calls="forward"),
        # 16-bit tables held whole in HBM: every lookup a hit
        _case("resident f16 forward", tables=26, rows_lo=100_000, rows_hi=100_000, dims="128", dtypes="f16", cache=1.0,
              alpha=1.0, bags=4096, pooling="poisson 30", calls="forward"),
        # the tables of the eight-table fp32 configuration at full size, exact
        # prefetch, placements on a stream of their own
        _case("fp32 step pipelined", tables=8, rows_lo=1_000_000, rows_hi=1_000_000, dims="128", cache=0.05, alpha=1.1,
              bags=2048, pooling="poisson 40", prefetch="exact", pipelined=True),
        # many tables of mixed sizes in fp16, caching bits and a 70% precise
        # prefetch list, fully associative priority ranking
        _case("mixed f16 priority step", tables=26, rows_lo=1_000, rows_hi=2_000_000, dims="128", dtypes="f16",
              cache=0.1, alpha=1.1, bags=4096, pooling="poisson 30", policy="priority", prefetch="mix 0.7"),
        # the LFU baseline, 32-way sets, no prefetch
        _case("lfu 32-way step", tables=8, rows_lo=200_000, rows_hi=200_000, dims="64", cache=0.2, alpha=1.0, bags=1024,
              pooling="poisson 25", policy="lfu", ways=32),
        # tables that stay in pageable host memory, rows gathered on the host
        _case("staged bf16 step", tables=2, rows_lo=1_000_000, rows_hi=1_000_000, dims="128", dtypes="bf16", cache=0.2,
              alpha=1.05, bags=2048, pooling="fixed 40", miss="staged", prefetch="exact"),
        # large bf16 tables behind large caches, long fixed bags, exact prefetch
        _case("large bf16 step", tables=4, rows_lo=4_000_000, rows_hi=4_000_000, dims="128", dtypes="bf16", cache=0.2,
              alpha=1.05, bags=16384, pooling="fixed 80", prefetch="exact"),
        # the most lookups: 32 fp32 tables of mixed widths, geometric pooling,
        # one-hot tail, 32-way priority sets
        _case("wide fp32 32-way step", tables=32, rows_lo=200_000, rows_hi=200_000, dims="32,64,128,256", cache=0.2,
              alpha=1.0, bags=8192, pooling="geometric 25", onehot=8, policy="priority", ways=32, prefetch="mix 0.7"),
    ]


# what a drawn case may take at most: the largest listed case's own sizes
MOST_LOOKUPS, MOST_TABLE_BYTES = 4_000_000, 3_000_000_000


def draw(rng):
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    calls = rng.choice(["step", "step", "step", "forward", "step+stats"])
    policy = rng.choice(["lru", "lru", "priority", "priority", "lfu"])
    c = dict(tables=logu(1, 32), rows_lo=0, rows_hi=0, dims=rng.choice(["64", "128", "32,64,128,256", "16,48", "%d" % logu(8, 256)]),
             dtypes=rng.choice(["f32", "f16", "bf16", "f32,bf16"]), cache=rng.choice([0.02, 0.05, 0.1, 0.2, 0.2, 1.0]),
             alpha=round(rng.uniform(0.85, 1.2), 3), bags=logu(16, 8192),
             pooling=rng.choice(["fixed %d", "poisson %d", "geometric %d"]) % logu(2, 80), onehot=0, policy=policy,
             ways=rng.choice([0, 0, 0, 32, 8]), prefetch=rng.choice(["none", "exact", "replace 0.2", "mix 0.7"]),
             miss=rng.choice(["zero_copy"] * 5 + ["staged"]), calls=calls, pipelined=rng.random() < 0.3, ring=8)
    c["onehot"] = rng.choice([0, c["tables"] // 4])
    c["rows_hi"] = logu(2_000, 2_000_000)
    c["rows_lo"] = max(1_000, int(c["rows_hi"] * rng.choice([1.0, 1.0, 0.1, 0.01])))
    # trimmed to what the listed cases take
    while c["bags"] > 16 and c["tables"] * c["bags"] * _mean(c) > MOST_LOOKUPS:
        c["bags"] = max(16, c["bags"] // 2 + rng.randrange(8))
    while sum(r * d * e for r, d, e, *_ in _tables(c)) > MOST_TABLE_BYTES:
        c["rows_hi"] = c["rows_hi"] // 2 + rng.randrange(100)
        c["rows_lo"] = min(c["rows_lo"], c["rows_hi"])
    return c


# ------------------------------------------------------------------ the shapes of a case

def _mean(c):
    return float(c["pooling"].split()[1])


def _tables(c):
    """(rows, dim, bytes per element, dtype, cached rows, zipf exponent, mean pooling) per table; rows spread evenly
    over their logarithm, the cycles of dims and dtypes of different lengths."""
    T, out = c["tables"], []
    dims, dts = [int(x) for x in c["dims"].split(",")], c["dtypes"].split(",")
    for t in range(T):
        f = t / (T - 1) if T > 1 else 1.0
        rows = int(round(c["rows_lo"] * (c["rows_hi"] / c["rows_lo"]) ** f))
        dt = dts[(t // len(dims)) % len(dts)] if len(dims) > 1 else dts[t % len(dts)]
        alpha = c["alpha"] + (0.0, 0.1, -0.1)[t % 3] * (T > 1)
        mean = 1.0 if t >= T - c["onehot"] else _mean(c)
        out.append((rows, dims[t % len(dims)], DTYPES[dt].itemsize, dt, max(1, int(c["cache"] * rows)), alpha, mean))
    return out


@functools.lru_cache(maxsize=64)
def _cdf(rows, alpha):
    k = np.arange(1, rows + 1, dtype=np.float64)
    return np.cumsum(k ** -alpha)


def _unique(rows, alpha, n):
    """Expected distinct rows of n Zipf draws."""
    p = np.diff(_cdf(rows, alpha), prepend=0.0) / _cdf(rows, alpha)[-1]
    return float(-np.expm1(n * np.log1p(-np.minimum(p, 1 - 1e-15))).sum())


# ------------------------------------------------------------------ inputs

def _inputs(c, seed):
    """Host tables, batches, prefetch lists and caching bits of a case, from the seed alone."""
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1_000_003 + 12345)
    tabs, B, N = _tables(c), c["bags"], c["ring"]
    # the tables side by side in one allocation
    at, starts = 0, []
    for rows, dim, esz, *_ in tabs:
        starts.append(at)
        at += -(-rows * dim * esz // 256) * 256
    arena = torch.empty(at, dtype=torch.uint8, pin_memory=c["miss"] == "zero_copy")
    host, perms, cdfs = [], [], []
    for (rows, dim, esz, dt, _, alpha, _), s in zip(tabs, starts):
        h = arena[s:s + rows * dim * esz].view(DTYPES[dt]).view(rows, dim)
        h.copy_(torch.rand((rows, dim), generator=g, device=dev).mul_(2).sub_(1).to(DTYPES[dt]))
        host.append(h)
        perms.append(torch.randperm(rows, generator=g, device=dev, dtype=torch.int32))
        cdfs.append(torch.from_numpy(_cdf(rows, alpha)).to(dev))
    base = [0]
    for rows, *_ in tabs:
        base.append(base[-1] + rows)

    def pooling(mean):
        kind = "fixed" if mean == 1.0 else c["pooling"].split()[0]
        if kind == "poisson":
            return torch.poisson(torch.full((B,), mean, device=dev), generator=g).long()
        if kind == "geometric":
            u = torch.rand(B, generator=g, device=dev, dtype=torch.float64)
            return torch.ceil(torch.log1p(-u) / math.log1p(-1.0 / mean)).long().clamp_(1, 40 * int(mean))
        return torch.full((B,), int(mean), dtype=torch.long, device=dev)

    batches, keys = [], []  # keys: ids numbered through all tables
    for _ in range(N):
        lens = [pooling(t[6]) for t in tabs]
        idx = []
        for t, n in enumerate(lens):
            u = torch.rand(int(n.sum()), generator=g, device=dev, dtype=torch.float64) * cdfs[t][-1]
            idx.append(perms[t][torch.searchsorted(cdfs[t], u).clamp_(max=tabs[t][0] - 1)])
        off = torch.zeros(len(tabs) * B + 1, dtype=torch.long, device=dev)
        off[1:] = torch.cumsum(torch.cat(lens), 0)
        batches.append((torch.cat(idx), off))
        keys.append(torch.cat([i.long() + b for i, b in zip(idx, base)]))
    starts_t = torch.tensor(base, device=dev)

    def split(k):
        """Numbered ids, ascending by table -> (rows int32, offsets per table)."""
        off = torch.searchsorted(starts_t, k, right=True) - 1
        po = torch.zeros(len(tabs) + 1, dtype=torch.long, device=dev)
        po[1:] = torch.cumsum(torch.bincount(off, minlength=len(tabs)), 0)
        return (k - starts_t[off]).int(), po

    kind = c["prefetch"].split()[0]
    lists, bits = [], []
    uniq = [torch.unique(k) for k in keys]
    for b in range(N):
        if kind == "none":
            k = uniq[b][:0]
        elif kind == "exact":
            k = uniq[b]
        else:  # a share of the batch's rows beside random ones, table by table
            frac = float(c["prefetch"].split()[1])
            t = torch.searchsorted(starts_t, uniq[b], right=True) - 1
            rand = (torch.rand(t.numel(), generator=g, device=dev, dtype=torch.float64) * (starts_t[t + 1] - starts_t[t])).long()
            keep = torch.rand(t.numel(), generator=g, device=dev) < (1 - frac if kind == "replace" else frac)
            k = torch.where(keep, uniq[b], starts_t[t] + rand)
        lists.append(split(k))
    if c["policy"] == "priority":
        for b in range(N):
            again = torch.isin(uniq[b], uniq[(b + 1) % N]) | torch.isin(uniq[b], uniq[(b + 2) % N])
            wrong = torch.rand(uniq[b].numel(), generator=g, device=dev) < 0.17
            bits.append((again ^ wrong)[torch.searchsorted(uniq[b], keys[b])].to(torch.uint8))
    else:
        bits = [None] * N
    return dict(host=host, perms=perms, batches=batches, lists=lists, bits=bits)


def prepare(case, seed):
    c, x = case, _inputs(case, seed)
    tabs = _tables(c)
    caps = [t[4] for t in tabs]
    max_idx = max(i.numel() for i, _ in x["batches"])
    max_pf = max(max(k.numel() for k, _ in x["lists"]), min(sum(caps), 1 << 20))
    cache = TieredEmbeddingCache(x["host"], [t[3] for t in tabs], caps, policy=c["policy"], miss_mode=c["miss"],
                                 max_bags_per_table=c["bags"], max_indices=max_idx, max_prefetch=max_pf, ways=c["ways"])
    s = dict(cache=cache, bags=c["bags"], calls=c["calls"], batches=x["batches"], lists=x["lists"], bits=x["bits"], at=0,
             out=torch.empty(c["bags"] * sum(t[1] for t in tabs), dtype=torch.float32, device="cuda:0"),
             stream=torch.cuda.Stream() if c["pipelined"] and c["calls"] != "forward" else None)
    # the caches start full: each table's most popular rows, the most popular last
    n = -(-sum(caps) // max_pf)
    for k in reversed(range(n)):
        parts = [p[cap * k // n:cap * (k + 1) // n] for p, cap in zip(x["perms"], caps)]
        po = torch.tensor([0] + [p.numel() for p in parts], device="cuda:0").cumsum(0)
        cache.placement(torch.cat(parts).contiguous(), po)
    torch.cuda.synchronize()
    for _ in range(WARM_BATCHES):
        _step(s)
    torch.cuda.synchronize()
    return s


def _step(s):
    b = s["at"] % len(s["batches"])
    if s["calls"] != "forward" or s["at"] == 0:
        rows, po = s["lists"][b]
        s["cache"].placement(rows if rows.numel() else None, po, s["bits"][b - 1] if s["at"] else None, stream=s["stream"])
    idx, off = s["batches"][b]
    s["at"] += 1
    return s["cache"].forward(idx, off, s["bags"], out=s["out"])


def run(state):
    out = _step(state)
    if state["calls"] != "step+stats":
        return out
    last, _ = state["cache"].stats()
    counts = np.array([[v[k] for k in sorted(v) if k != "digest"] for v in last], dtype=np.int64)
    digest = np.array([v["digest"] for v in last], dtype=np.uint64).view(np.int64)
    return {"out": out, "counters": counts, "digest": digest}


# ------------------------------------------------------------------ what a pass needs

def work(case):
    """Each distinct row of the batch read once, indices, offsets, prefetch ids and caching bits read once, the pooled
    sums written once; one addition per element looked up.  (The rows a placement brings in depend on the cache.)"""
    B, nbytes, flops = case["bags"], 0.0, 0.0
    step = case["calls"] != "forward"
    for rows, dim, esz, _, _, alpha, mean in _tables(case):
        n = B * mean
        u = _unique(rows, alpha, n)
        nbytes += u * dim * esz + 4 * n + B * (8 + 4 * dim)
        flops += n * dim
        if step:
            nbytes += (4 * u if case["prefetch"] != "none" else 0) + (n if case["policy"] == "priority" else 0)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # sums of up to some hundred values in [-1, 1] accumulated in fp32 (16-bit rows widen exactly): the distance of
    # this library's sums from 64-bit ones is 0.1e-8 .. 7e-8 over the cases, and another order gives as much
    return {"rel": 3e-7, "max": 6e-6}


def exact(case, seed):
    x = _inputs(case, seed)
    idx, off = x["batches"][WARM_BATCHES % len(x["batches"])]
    B, out = case["bags"], []
    for t, h in enumerate(x["host"]):
        o = off[t * B:(t + 1) * B + 1]
        ids, o = idx[o[0]:o[-1]].long(), (o - o[0])
        bag = torch.repeat_interleave(torch.arange(B, device=o.device), o[1:] - o[:-1])
        table = h.to(o.device)
        acc = torch.zeros((B, h.shape[1]), dtype=torch.float64, device=o.device)
        for k in range(0, ids.numel(), 1 << 20):
            acc.index_add_(0, bag[k:k + (1 << 20)], table[ids[k:k + (1 << 20)]].double())
        out.append(acc.reshape(-1))
    out = torch.cat(out)
    return {"out": out, "counters": None, "digest": None} if case["calls"] == "step+stats" else out

"""The general sequence of calls (tables past the one-block-per-table kernels'
bitmaps) where its loops run several times: blocks that free more slots than
their list holds, rings that compact, thresholds among a placement's own keys.
Counters, digests and resident sets equal the oracle's exactly, pooled sums lie
within the fp32 bound of the summation order."""
import numpy as np
import pytest

import tracegen as tg
from _helpers import FWD_KEYS, PLACE_KEYS, GpuRunner, check_pooled

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BAGS = 24
BIG = (1 << 20) + 77  # rows of a table that neither one-block kernel takes


def _workload(rows, caps, policy, **kw):
    tabs = [tg.Table(n, (4, 9, 16)[t % 3], ("f32", "bf16", "f16")[t % 3], c, 1.0, ("fixed", 1))
            for t, (n, c) in enumerate(zip(rows, caps))]
    return tg.Workload(83, "general", tabs, batches=1, bags=BAGS, policy=policy, eviction_speed=3, **kw)


def _ids(rng, rows, n, hot):
    """n ids: a share from `hot` rows at a moving place, the rest from everywhere."""
    at = int(rng.integers(0, rows))
    return np.where(rng.random(n) < 0.5, (at + rng.integers(0, hot, n)) % rows, rng.integers(0, rows, n)).astype(np.int32)


def _batch(rng, w, counts, hot):
    parts, offs, at = [], [0], 0
    for tb, n in zip(w.tables, counts):
        parts.append(_ids(rng, tb.rows, n, min(hot, tb.rows)))
        cuts = np.sort(rng.integers(0, n + 1, BAGS - 1))
        offs += list(at + cuts) + [at + n]
        at += n
    return np.concatenate(parts), np.array(offs, np.int64)


def _list(rng, w, counts, hot):
    parts = [_ids(rng, tb.rows, n, min(hot, tb.rows)) for tb, n in zip(w.tables, counts)]
    return np.concatenate(parts), np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)


class Against:
    """A cache and the oracle taking the same calls, compared after each."""

    def __init__(self, w, max_indices, max_prefetch, **kw):
        import oracle
        self.w = w
        self.tabs = [w.table_values(t) for t in range(w.num_tables)]
        self.f64 = [tg.storage_to_f64(a, tb.dtype) for a, tb in zip(self.tabs, w.tables)]
        self.g = GpuRunner(w, self.tabs, max_indices=max_indices, max_prefetch=max_prefetch, **kw)
        self.o = oracle.for_workload(w, self.tabs)
        self.k = 0

    def _counters(self, keys, res=None):
        got, _, *_ = self.g.cache.stats() if res is None else res
        for t in range(self.w.num_tables):
            ref = self.o.stats(t)
            for key in keys:
                assert got[t][key] == ref[key], f"call {self.k} table {t} {key}: {got[t][key]} {ref[key]}"
            if res is not None:
                assert np.array_equal(res[2][t], self.o.resident(t)), f"call {self.k} table {t}: resident set"
        self.k += 1
        return got

    def placement(self, P, poff, bits=None):
        self.g.placement(P, poff, bits)
        assert self.o.placement(P, poff, bits) == 0
        return self._counters(PLACE_KEYS, self.g.cache.stats(dump=True))

    def forward(self, idx, off):
        out = self.g.forward(idx, off)
        st, _, r64 = self.o.forward(idx, off, self.w.bags, want64=True)
        assert st == 0
        got = self._counters(FWD_KEYS)
        check_pooled(self.w, self.f64, idx, off, out, r64, f"call {self.k - 1}")
        return got

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.g.close()
        self.o.close()


@pytest.mark.parametrize("policy", ["lru", "priority", "lfu"])
def test_many_evictions_per_block(policy):
    """One of eight tables takes nearly all ids, so few blocks (their number
    goes by the mean) free tens of thousands of its slots: every block empties
    its list several times.  LRU: the ring compacts about every third
    placement, and lists longer than the cache put the threshold among the
    placement's own keys (and free the batch's and the last list's rows)."""
    rows, caps = [BIG] + [500] * 7, [90_000 if policy != "lru" else 30_000] + [20] * 7
    w = _workload(rows, caps, policy)
    rng = np.random.default_rng(31)
    counts = lambda n: [n] + [9] * 7
    lists = [counts(n) for n in (50_000, 20_000, 64_000, 0, 64_000, 1_000, 40_000, 64_000, 64_000, 30_000, 64_000, 20)]
    most = past = 0
    with Against(w, 64_100, 64_100) as a:
        last = None
        for k, pc in enumerate(lists):
            P, poff = _list(rng, w, pc, 20_000)
            bits = (rng.random(last) < 0.4).astype(np.uint8) if policy == "priority" and last else None
            got = a.placement(P, poff, bits)
            most = max(most, got[0]["evicted"])
            past += got[0]["prefetch_dropped"] > 0
            idx, off = _batch(rng, w, counts((60_000, 8_000, 33_000)[k % 3]), 15_000)
            a.forward(idx, off)
            last = idx.size
    # a list of 2,048 slots is emptied past 1,024.  PRIORITY and LFU: 4,096 slots per block (LFU frees fewer of
    # them); LRU: a ring's chunk per iteration, in at most 130,000 / 8 / 1,024 + 1 blocks
    assert most > (24 * 1024 if policy != "lfu" else 10_000) and (policy != "lru" or past > 2)


@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("lfu", 0), ("lru", 8)])
def test_both_sides_of_the_ids_per_table(policy, ways):
    """Placements whose lists mean 5,500 and 5,501 ids (the line of fully
    associative LRU and PRIORITY tables), and far apart, in turn on one cache."""
    w = _workload([60_000], [9_000], policy, ways=ways)
    rng = np.random.default_rng(9)
    with Against(w, 9_000, 9_000) as a:
        last = None
        for pc, n in ((5_500, 5_500), (5_500, 5_501), (5_501, 5_500), (2_000, 9_000), (2_001, 9_000), (9_000, 40), (9_000, 9_000),
                      (1, 2_000), (9_000, 5_500)):
            P, poff = _list(rng, w, [pc], 9_000)
            a.placement(P, poff, (rng.random(last) < 0.4).astype(np.uint8) if policy == "priority" and last else None)
            idx, off = _batch(rng, w, [n], 9_000)
            a.forward(idx, off)
            last = n


@pytest.mark.parametrize("policy", ["priority", "lru"])
def test_static_workspace_without_the_optional_memory(policy):
    """A configuration that the library's 32 MiB array holds only without the
    memory that makes calls faster: PRIORITY ranks 100,000 slots in one block
    where several blocks would have their histograms, LRU marks 60,000 ids of
    a table in one part.  The same counters and sums."""
    from paper_2511_08568_amd import binding as bd
    lru = policy == "lru"
    rows, caps = ([300_000], [100_000]) if not lru else ([1_000_000], [10_000])
    w = _workload(rows, caps, policy)
    w.tables[0].dim = 32 if not lru else 8
    full = 32 << 20
    mi, step = (20_000, 50) if not lru else (60_000, 1_000)
    query = lambda n: bd.recmg_query_workspace(_cfg_of(w, n))[0]
    while query(mi) <= full:
        mi += step
    rng = np.random.default_rng(8)
    with Against(w, mi, mi, static_workspace=True) as a:
        last = None
        for k in range(6):
            P, poff = _list(rng, w, [(mi, mi // 2, 100)[k % 3]], 20_000)
            a.placement(P, poff, (rng.random(last) < 0.4).astype(np.uint8) if last and not lru else None)
            idx, off = _batch(rng, w, [(mi, 500)[k % 2]], 9_000)
            a.forward(idx, off)
            last = idx.size


def _cfg_of(w, n):
    """The configuration that `Against` makes for a one-table workload, to ask for its workspace."""
    import ctypes
    from paper_2511_08568_amd import binding as bd
    tb = w.tables[0]
    cfg = bd.recmg_config_t()
    cfg._keep = [(ctypes.c_int64 * 1)(tb.rows), (ctypes.c_int32 * 1)(tb.dim), (ctypes.c_int32 * 1)(bd.RECMG_F32),
                 (ctypes.c_void_p * 1)(4096), (ctypes.c_int64 * 1)(tb.cap)]
    cfg.num_tables = 1
    cfg.rows, cfg.dims, cfg.dtypes, cfg.host_tables, cfg.cache_rows = cfg._keep
    cfg.policy, cfg.eviction_speed = bd.POLICY_CODES[w.policy], w.eviction_speed
    cfg.max_bags_per_table, cfg.max_indices, cfg.max_prefetch = w.bags, n, n
    return cfg

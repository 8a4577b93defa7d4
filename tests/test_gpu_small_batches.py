"""Calls on both sides of the line between the one-block-per-table kernels and
the general sequence, in turn on one cache (each must read what the other
left), at sizes where their tiles end: tables of one bitmap block of rows and
one row more, of the most rows a block's LDS bitmap holds, one table with
nearly all ids, tables with none.  Counters, digests and resident sets equal
the oracle's exactly, pooled sums lie within the fp32 bound of the summation
order."""
import numpy as np
import pytest

import tracegen as tg
from _helpers import FWD_KEYS, PLACE_KEYS, GpuRunner, check_pooled

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BAGS = 24


def _ids(rng, rows, n):
    """n ids of a table: mostly a hot tenth, first and last row among them."""
    ids = np.where(rng.random(n) < 0.7, rng.integers(0, max(rows // 10, 1), n), rng.integers(0, rows, n))
    ids[:2] = (0, rows - 1)[:max(0, min(2, n))]
    return ids.astype(np.int32)


def _batch(rng, tables, counts):
    parts, offs, at = [], [0], 0
    for tb, n in zip(tables, counts):
        parts.append(_ids(rng, tb.rows, n))
        cuts = np.sort(rng.integers(0, n + 1, BAGS - 1))
        offs += list(at + cuts) + [at + n]
        at += n
    return np.concatenate(parts), np.array(offs, np.int64)


# (rows per table, cap as a share of them); 32,768 rows are one bitmap block, 2^20 fill a block's LDS
SHAPES = {
    "one block and one row": ([32768, 32769, 5], 0.1),
    "eight blocks and one row": ([262144, 262145, 1000, 31], 0.02),
    "the largest bitmap": ([1 << 20, 70], 0.004),
    "past the largest bitmap": ([(1 << 20) + 1, 40000], 0.004),
    "all resident": ([5000, 300, 1], 1.0),
}


@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("lfu", 0), ("lru", 32), ("priority", 5)])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_small_and_general_calls_in_turn(shape, policy, ways):
    import oracle
    rows, share = SHAPES[shape]
    T = len(rows)
    w = tg.Workload(77, shape, [tg.Table(n, (9, 64, 4, 32)[t % 4], ("f32", "f16", "bf16")[t % 3], max(1, int(share * n)),
                                         1.0, ("fixed", 1)) for t, n in enumerate(rows)],
                    batches=1, bags=BAGS, policy=policy, ways=ways, eviction_speed=2)
    tabs = [w.table_values(t) for t in range(T)]
    f64 = [tg.storage_to_f64(a, tb.dtype) for a, tb in zip(tabs, w.tables)]
    rng = np.random.default_rng(11)
    even = lambda n: [n // T + (t < n % T) for t in range(T)]
    skew = lambda n: [n - (T - 1) * 3] + [3] * (T - 1)
    none = lambda n: [n] + [0] * (T - 1)
    # ids per call: far below the line, at the total's line and one past it, far past it, enough per table (in two
    # tables) to be marked in parts
    plan = [even(200), even(32768), even(32769), skew(9000), even(60), none(5000), skew(32768), even(130001), even(700),
            even(0), skew(120000), even(1500)]
    g = GpuRunner(w, tabs, max_indices=130001, max_prefetch=130001)
    o = oracle.for_workload(w, tabs)
    try:
        last = None
        for k, counts in enumerate(plan):
            if k % 4 != 3:  # now and then a batch without a placement before it
                # prefetch lists from the next-but-one call's sizes: small lists after large batches and the reverse
                pc = plan[(k * 5 + 2) % len(plan)]
                P = np.concatenate([_ids(rng, n, c) for n, c in zip(rows, pc)]) if sum(pc) else np.zeros(0, np.int32)
                poff = np.concatenate([[0], np.cumsum(pc)]).astype(np.int64)
                bits = None if last is None or policy != "priority" else (rng.random(last) < 0.4).astype(np.uint8)
                g.placement(P, poff, bits)
                assert o.placement(P, poff, bits) == 0
                got, _, res = g.cache.stats(dump=True)
                for t in range(T):
                    ref = o.stats(t)
                    for key in PLACE_KEYS:
                        assert got[t][key] == ref[key], f"call {k} table {t} placement {key}: {got[t][key]} {ref[key]}"
                    assert np.array_equal(res[t], o.resident(t)), f"call {k} table {t}"
            idx, off = _batch(rng, w.tables, counts)
            out = g.cache.forward(g.to_dev(idx) if idx.size else g.to_dev(np.zeros(1, np.int32))[:0], g.to_dev(off),
                                  BAGS).cpu().numpy()
            st, _, r64 = o.forward(idx, off, BAGS, want64=True)
            assert st == 0
            last = idx.size
            got, _ = g.cache.stats()
            for t in range(T):
                ref = o.stats(t)
                for key in FWD_KEYS:
                    assert got[t][key] == ref[key], f"call {k} table {t} forward {key}: {got[t][key]} {ref[key]}"
            check_pooled(w, f64, idx, off, out, r64, f"call {k}")
    finally:
        g.close()
        o.close()


@pytest.mark.parametrize("what", ["row past the end", "negative row", "offsets decrease", "offsets end short"])
def test_small_forward_raises_the_error_word(what):
    """One malformed table among good ones: the error is reported, nothing of
    the call is published, and later calls stay no-ops."""
    from paper_2511_08568_amd import binding as bd
    w = tg.Workload(78, "bad", [tg.Table(1000, 8, "f32", 100, 1.0, ("fixed", 1)) for _ in range(3)], batches=1, bags=BAGS)
    tabs = [w.table_values(t) for t in range(3)]
    rng = np.random.default_rng(5)
    g = GpuRunner(w, tabs, max_indices=4000, max_prefetch=64)
    try:
        idx, off = _batch(rng, w.tables, [500, 600, 700])
        g.forward(idx, off)
        _, before = g.cache.stats()
        bad, boff = idx.copy(), off.copy()
        if what == "row past the end":
            bad[700] = 1000
        elif what == "negative row":
            bad[700] = -1
        elif what == "offsets decrease":
            boff[BAGS + 3] = boff[BAGS + 2] - 1
            assert boff[BAGS + 3] >= 0
        else:
            boff[-1] -= 1
            boff[-2] = min(boff[-2], boff[-1])
        for _ in range(2):
            g.forward(bad, boff)
            _, total, code = g.cache.stats(strict=False)
            assert code == bd.RECMG_E_RANGE and total == before
    finally:
        g.close()

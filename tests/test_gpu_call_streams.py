"""Calls on both sides of the lines between the small and the general kernels,
on several streams, with and without a copy stream: fills inside a placement's
last kernel, fills apart, on the copy stream or the placement's own; locations
written beside the fetch or before it.  The library orders the calls by events;
nothing here synchronises between them.  Counters, digests and resident sets
equal the oracle's exactly, pooled sums lie within the fp32 bound of the
summation order."""
import numpy as np
import pytest

import tracegen as tg
from _helpers import FWD_KEYS, PLACE_KEYS, GpuRunner, check_pooled

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

BAGS = 24


class Sequence:
    """A cache and the oracle taking the same calls, compared by the stats log
    and the pooled sums at the end."""

    def __init__(self, w, n, calls, **kw):
        import oracle
        self.w, self.tabs = w, [w.table_values(t) for t in range(w.num_tables)]
        self.g = GpuRunner(w, self.tabs, max_indices=n, max_prefetch=n, stats_log_calls=calls, **kw)
        self.o = oracle.for_workload(w, self.tabs)
        self.log, self.outs = [], []

    def _record(self, keys):
        self.log.append([{k: st[k] for k in keys} for st in (self.o.stats(t) for t in range(self.w.num_tables))])

    def inputs(self, *arrays):
        """Device copies, ready before the calls that take them (a call orders what the library does, not copies)."""
        d = [None if a is None or not a.size else self.g.to_dev(a) for a in arrays]
        torch.cuda.synchronize()
        return d

    def placement(self, P, poff, bits, stream, dev):
        self.g.cache.placement(dev[0], dev[1], dev[2], stream=stream)
        assert self.o.placement(P, poff, bits) == 0
        self._record(PLACE_KEYS)

    def forward(self, idx, off, stream, dev):
        empty = torch.zeros(1, dtype=torch.int32, device="cuda")[:0]
        out = torch.empty(self.w.bags * sum(tb.dim for tb in self.w.tables), device="cuda")
        self.g.cache.forward(dev[0] if idx.size else empty, dev[1], self.w.bags, out=out, stream=stream)
        st, _, r64 = self.o.forward(idx, off, self.w.bags, want64=True)
        assert st == 0
        self._record(FWD_KEYS)
        self.outs.append((out, r64.copy(), idx, off))

    def check(self):
        f64 = [tg.storage_to_f64(a, tb.dtype) for a, tb in zip(self.tabs, self.w.tables)]
        _, _, res = self.g.cache.stats(dump=True)
        got = self.g.cache.stats_log()
        assert len(got) == len(self.log)
        for k, (a, b) in enumerate(zip(got, self.log)):
            for t in range(self.w.num_tables):
                for key, v in b[t].items():
                    assert a[t][key] == v, f"call {k} table {t} {key}: {a[t][key]} {v}"
        for t in range(self.w.num_tables):
            assert np.array_equal(res[t], self.o.resident(t)), f"table {t}: resident set"
        for k, (out, r64, idx, off) in enumerate(self.outs):
            check_pooled(self.w, f64, idx, off, out.cpu().numpy(), r64, f"forward {k}")

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.g.close()
        self.o.close()


def _ids(rng, rows, n):
    return np.where(rng.random(n) < 0.6, rng.integers(0, max(rows // 8, 1), n), rng.integers(0, rows, n)).astype(np.int32)


def _batch(rng, w, counts):
    parts, offs, at = [], [0], 0
    for tb, n in zip(w.tables, counts):
        parts.append(_ids(rng, tb.rows, n))
        offs += list(at + np.sort(rng.integers(0, n + 1, BAGS - 1))) + [at + n]
        at += n
    return np.concatenate(parts), np.array(offs, np.int64)


def _list(rng, w, counts):
    return (np.concatenate([_ids(rng, tb.rows, n) for tb, n in zip(w.tables, counts)]),
            np.concatenate([[0], np.cumsum(counts)]).astype(np.int64))


@pytest.mark.parametrize("overlap", [True, False])
@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("lru", 8)])
def test_wide_rows_in_small_placements(policy, ways, overlap):
    """Rows of 8 KiB: lists of 2,048 ids (16 MiB, the most that a placement's last
    kernel fills beside a copy stream) and 2,049, and far apart, in turn,
    placements on a stream of their own; two in a row now and then.  Without a
    copy stream such a placement's fill is always apart."""
    w = tg.Workload(95, "wide", [tg.Table(6000, 2048, "f32", 3000, 1.0, ("fixed", 1))], batches=1, bags=BAGS,
                    policy=policy, ways=ways, eviction_speed=2)
    rng = np.random.default_rng(14)
    lists = (2048, 2049, 2048, 4000, 300, 2049, 0, 4000, 100, 2048)
    with Sequence(w, 4000, 40, overlap=overlap) as q:
        own, last = torch.cuda.Stream(), None
        calls = []
        for k, n in enumerate(lists):
            for _ in range(2 if k % 4 == 3 else 1):
                P, poff = _list(rng, w, [n])
                bits = (rng.random(last) < 0.4).astype(np.uint8) if policy == "priority" and last else None
                calls.append(("p", (P, poff, bits), q.inputs(P, poff, bits)))
                last = None  # the next placement comes after no forward
            idx, off = _batch(rng, w, [(1500, 300)[k % 2]])
            calls.append(("f", (idx, off), q.inputs(idx, off)))
            last = idx.size
        for kind, args, dev in calls:
            if kind == "p":
                q.placement(*args, own, dev)
            else:
                q.forward(*args, None, dev)
        q.check()


def _counts(kind, n, T):
    """n ids over T tables: evenly, or nearly all in the first."""
    return [n // T + (t < n % T) for t in range(T)] if kind == "even" else [n - 3 * (T - 1)] + [3] * (T - 1)


@pytest.mark.parametrize("overlap", [True, False])
@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("lfu", 0), ("lru", 4), ("lfu", 32)])
@pytest.mark.parametrize("big", [False, True])
def test_random_sequences_across_the_line(big, policy, ways, overlap):
    """Random placements and forwards, two of a kind in a row among them, small
    and general ones in turn.  The first calls share one stream, the later ones
    come on three, placements and forwards apart: the first placement on another
    stream follows a general forward, whose locations are written beside its
    fetch.  big: a table past the small kernels' bitmaps, so every call takes the
    general sequence, whatever its size."""
    rows = [(1 << 20) + 77, 5000, 300] if big else [60_000, 5000, 300]
    tabs = [tg.Table(n, (16, 64, 9)[t], ("f32", "f16", "bf16")[t], max(ways, n // 25 if t else 4000), 1.0, ("fixed", 1))
            for t, n in enumerate(rows)]
    w = tg.Workload(96, "across", tabs, batches=1, bags=BAGS, policy=policy, ways=ways, eviction_speed=2)
    rng = np.random.default_rng(60 + 7 * big + 3 * ways + overlap)
    sizes = (40, 900, 12_000, 34_000)
    calls, last = [], None
    for k in range(36):
        # one stream; from call 12 on placements on two others, forwards on two
        kind = "f" if k in (5, 11) else "p" if k == 12 else ("p", "f")[int(rng.integers(2))]
        n = 34_000 if k in (11, 12) else int(rng.choice(sizes))
        c = _counts("even" if rng.random() < 0.6 else "skew", n, 3)
        s = 0 if k < 12 else 1 + int(rng.integers(2)) if kind == "p" else 2 * int(rng.integers(2))
        if kind == "p":
            P, poff = _list(rng, w, c) if rng.random() < 0.85 or k == 12 else (np.zeros(0, np.int32), np.zeros(4, np.int64))
            bits = (rng.random(last) < 0.4).astype(np.uint8) if policy == "priority" and last else None
            calls.append(("p", (P, poff, bits), s))
            last = None
        else:
            calls.append(("f", _batch(rng, w, c), s))
            last = calls[-1][1][0].size
    with Sequence(w, 34_000, len(calls), overlap=overlap) as q:
        streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
        dev = [q.inputs(*args) for _, args, _ in calls]
        for (kind, args, s), d in zip(calls, dev):
            (q.placement if kind == "p" else q.forward)(*args, streams[s], d)
        q.check()


@pytest.mark.parametrize("overlap", [True, False])
@pytest.mark.parametrize("policy", ["lru", "priority"])
def test_general_placements_in_a_row_on_streams(policy, overlap):
    """Two general placements in a row, each on a stream other than the last
    call's, then a forward on a third: the second frees slots that the first
    one's fill may still be writing.  A small one follows now and then, whose
    fill runs in its last kernel."""
    w = tg.Workload(97, "row", [tg.Table(600_000, 32, "f32", 12_000, 1.0, ("fixed", 1)),
                                tg.Table(4000, 32, "f16", 600, 1.0, ("fixed", 1))], batches=1, bags=BAGS,
                    policy=policy, eviction_speed=2)
    v = tg.Workload(98, "row", [tg.Table(200_000, 32, "f32", 12_000, 1.0, ("fixed", 1)),
                                tg.Table(4000, 32, "f16", 600, 1.0, ("fixed", 1))], batches=1, bags=BAGS,
                    policy=policy, eviction_speed=2)
    rng = np.random.default_rng(19)
    for x, lists in ((w, (9_000, 12_500, 300)), (v, (20_000, 24_000, 300))):
        with Sequence(x, 26_000, 64, overlap=overlap) as q:
            streams = [torch.cuda.Stream() for _ in range(3)]
            calls = []
            for b in range(6):
                for rep in range(3 if b % 2 else 2):
                    calls.append(("p", (*_list(rng, x, [lists[rep], 200]), None), rep % 2))
                calls.append(("f", _batch(rng, x, [(6_000, 300)[b % 2], 200]), 2))
            dev = [q.inputs(*args) for _, args, _ in calls]
            for (kind, args, s), d in zip(calls, dev):
                (q.placement if kind == "p" else q.forward)(*args, streams[s], d)
            q.check()

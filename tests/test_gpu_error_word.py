"""The device's error word under calls that overlap: a malformed call raises it
while another call's kernels run on their own stream.  Every kernel's block then
either does its whole work or none (no wave leaves the others with half-set
tables), the error is reported, and every later call is a no-op."""
import numpy as np
import pytest

import tracegen as tg
from _helpers import GpuRunner

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_2511_08568_amd import binding as bd  # noqa: E402

DIMS = (4, 64, 9, 32)


def _case(rows, bags, seed, per_bag, **kw):
    """Tables of several pooled-kernel kinds, none of their rows cached to begin with, and two batches."""
    w = tg.Workload(91, "overlap", [tg.Table(n, DIMS[t % 4], ("f32", "f16")[t % 2], max(1, n // 10), 1.0, ("fixed", 1))
                                    for t, n in enumerate(rows)], batches=1, bags=bags, **kw)
    rng = np.random.default_rng(seed)
    batches = []
    for _ in range(2):
        idx = np.concatenate([rng.integers(0, n, bags * per_bag) for n in rows]).astype(np.int32)
        batches.append((idx, np.arange(len(rows) * bags + 1, dtype=np.int64) * per_bag))
    return w, [w.table_values(t) for t in range(len(rows))], batches


@pytest.mark.parametrize("what", ["prefetch row past the end", "prefetch offsets decrease"])
@pytest.mark.parametrize("rows,bags", [([3000] * 6, 60), ([(1 << 20) + 5, 40000, 3000, 3000], 2000)])
@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("priority", 8)])
def test_malformed_placement_beside_a_forward(rows, bags, policy, ways, what):
    """Few bags: the small kernels and the shared pooled launch; many, over a
    table past the small kernels' bitmap: the general sequence and a launch per
    kind."""
    w, tabs, batches = _case(rows, bags, 3, 20, policy=policy, ways=ways)
    T = len(rows)
    P = np.concatenate([np.arange(0, n, 7) for n in rows]).astype(np.int32)
    poff = np.concatenate([[0], np.cumsum([len(range(0, n, 7)) for n in rows])]).astype(np.int64)
    bad, boff = P.copy(), poff.copy()
    if what == "prefetch row past the end":
        bad[poff[1]:poff[2]][-1] = rows[1]
    else:
        boff[2] = boff[1] - 1
    for delay in range(3):  # the bad list behind nothing, behind one copy, behind some
        g = GpuRunner(w, tabs, max_indices=batches[0][0].size, max_prefetch=P.size)
        own = torch.cuda.Stream()
        try:
            d = [(g.to_dev(i), g.to_dev(o)) for i, o in batches]
            dP, dpo, dbad, dboff = (g.to_dev(x) for x in (P, poff, bad, boff))
            out = torch.empty(bags * sum(tb.dim for tb in w.tables), device="cuda")
            junk = torch.empty(1 << 22, device="cuda")
            torch.cuda.synchronize()
            g.cache.placement(dP, dpo, None, stream=own)
            g.cache.forward(*d[0], bags, out=out)
            g.cache.forward(*d[1], bags, out=out)
            with torch.cuda.stream(own):
                for _ in range(delay * delay):
                    junk.fill_(1.0)
            g.cache.placement(dbad, dboff, None, stream=own)  # may overlap the forward's fetch and pooled sums
            _, total, code = g.cache.stats(strict=False)
            assert code == bd.RECMG_E_RANGE
            out.fill_(7.0)
            g.cache.placement(dP, dpo, None, stream=own)
            g.cache.forward(*d[0], bags, out=out)
            _, after, code = g.cache.stats(strict=False)
            assert code == bd.RECMG_E_RANGE and after == total
            assert bool((out == 7.0).all()), "a call after the error wrote its output"
        finally:
            g.close()


@pytest.mark.parametrize("what", ["row past the end", "negative row", "offsets decrease", "offsets end short",
                                  "empty list, offsets malformed"])
@pytest.mark.parametrize("policy,ways", [("lru", 0), ("priority", 0), ("lfu", 0), ("priority", 5), ("lfu", 5)])
def test_malformed_small_placement_changes_nothing(policy, ways, what):
    """One malformed table between good ones, in the kernel that runs a whole
    placement per table: no block may change its table's cache for a call that
    another table makes void.  The caller's workspace shows it: after the call
    only the error word differs."""
    w, tabs, batches = _case([3000, 700, 2000], 60, 5, 20, policy=policy, ways=ways)
    P = np.concatenate([np.arange(0, tb.rows, 3) for tb in w.tables]).astype(np.int32)
    poff = np.concatenate([[0], np.cumsum([len(range(0, tb.rows, 3)) for tb in w.tables])]).astype(np.int64)
    idx, off = batches[0]
    bits = (np.arange(idx.size) % 3 == 0).astype(np.uint8) if policy == "priority" else None
    g = GpuRunner(w, tabs, max_indices=idx.size, max_prefetch=P.size)
    try:
        g.placement(P, poff)
        g.forward(idx, off)
        _, total, code = g.cache.stats(strict=False)
        assert code == bd.RECMG_OK
        bad, boff = (P + 1) % 700, poff.copy()
        if what == "row past the end":
            bad[poff[2] - 1] = 700
        elif what == "negative row":
            bad[poff[1]] = -1
        elif what == "offsets decrease":
            boff[2] = boff[1] - 1
        elif what == "offsets end short":
            boff[3] -= 1
        else:
            bad, boff = bad[:0], np.array([0, 0, 1, 0], np.int64)
        d = g.to_dev(bad) if bad.size else None, g.to_dev(boff), None if bits is None else g.to_dev(bits)
        torch.cuda.synchronize()
        before = g.cache.workspace.clone()
        g.cache.placement(*d)
        _, after, code = g.cache.stats(strict=False)
        assert code == bd.RECMG_E_RANGE and after == total
        at = torch.nonzero(before != g.cache.workspace).flatten()
        assert 1 <= at.numel() <= 4 and int(at[-1]) - int(at[0]) < 4, f"{at.numel()} bytes of the workspace changed"
    finally:
        g.close()


@pytest.mark.parametrize("n", ["none", "few", "many"])
@pytest.mark.parametrize("bags", [16384, 16385, 40000])
def test_offsets_of_many_bags(bags, n):
    """Bag counts on both sides of the line past which a kernel of its own
    checks the offsets: a good call is served, one that decreases in the last
    table's last bags is found, whatever the number of indices."""
    w = tg.Workload(92, "bags", [tg.Table(500, 4, "f32", 50, 1.0, ("fixed", 1)) for _ in range(3)], batches=1, bags=bags)
    tabs = [w.table_values(t) for t in range(3)]
    rng = np.random.default_rng(6)
    total = {"none": 0, "few": 900, "many": 60000}[n]
    idx = rng.integers(0, 500, total).astype(np.int32)
    off = np.concatenate([[0], np.sort(rng.integers(0, total + 1, 3 * bags - 1)), [total]]).astype(np.int64)
    off[:3 * bags - 1] = np.minimum(off[:3 * bags - 1], max(total - 2, 0))
    off[3 * bags - 1] = total  # the last bag but one ends the batch
    g = GpuRunner(w, tabs, max_indices=max(total, 1), max_prefetch=1)
    try:
        call = lambda o: g.cache.forward(g.to_dev(idx) if total else g.to_dev(np.zeros(1, np.int32))[:0], g.to_dev(o), bags)
        out = call(off).cpu().numpy().reshape(3, bags, 4)
        g.cache.stats()
        ref = np.stack([np.concatenate([np.zeros((1, 4)), np.cumsum(tabs[t][idx].astype(np.float64), 0)]) for t in range(3)])
        for t in range(3):
            o = off[t * bags:(t + 1) * bags + 1]
            assert np.abs(out[t] - (ref[t][o[1:]] - ref[t][o[:-1]])).max() <= 1e-3
        bad = off.copy()
        bad[3 * bags - 1] = bad[3 * bags] + 1  # past the end, then back
        out = call(bad)
        _, _, code = g.cache.stats(strict=False)
        assert code == bd.RECMG_E_RANGE
    finally:
        g.close()

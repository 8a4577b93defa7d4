// Resident rings: the LRU_BATCH placement of fully associative tables (Alg. 1
// and Alg. 2 applied between batches, Sec. VI-B) without ranking every slot.
//
// Under LRU_BATCH a score is the number b of the placement that last touched
// the row (the last batch's rows take lru_touch = b) or named it in a
// prefetch list (pscore = b + 1).  Scores only grow, and a placement changes
// the scores of the rows it touches or names and of no other.  So each table
// keeps its residents sorted by key (score, row), the smallest first:
//
//   ring      one run per earlier placement, in placement order: the rows
//             that took that placement's touch score, ascending (scores < b)
//   pending   the rows the previous placement named (score b), ascending;
//             kept apart because placement b adds rows of the same score
//
// Placement b then, per table:
//   touch   the last batch's hits and the prefetch list's residents take
//           their new scores; their ring entries go stale (slot_pos = -1)
//   zones   Z1, the keys of score b in row order: the pending rows neither
//           touched nor named again, merged with the last batch's rows that
//           are not named (hits; misses as candidates).  Z2, the keys of score
//           b + 1, is the prefetch list itself (PU, ascending)
//   cut     with D = |K| - min(Cap, |K|) keys to drop: if the ring holds at
//           least D live entries, its first D go (the D smallest keys) and
//           every candidate stays; otherwise the whole ring goes and the
//           threshold key falls at rank D - |ring| of Z1, else of Z2
//   evict   the ring entries before the cut (and Z1/Z2 residents below the
//           threshold)
//   admit   every candidate at or above the threshold (placement.hip)
//   append  Z1's kept keys go to the back of the ring as one run (holes
//           where a key was dropped); Z2's kept rows become the pending list
//
// The cost is O(touched + named + evicted) per placement, not O(Cap): live
// entries per chunk of kRingChunk entries are counted, so the cut is found by
// reading chunk counts.  Stale entries stay until the front passes them;
// when an append would run past the end of the buffer, the live entries are
// first compacted, in order, into the other buffer.  The kept set is the one
// the radix-select placement keeps: the same keys, ties in score broken by row.
#include <algorithm>

#include "launch.h"
#include "placement_device.h"

namespace recmg {

constexpr int kRingEvictBuf = 2048;

// Merging two ascending lists A and B (an element of A goes before an equal one
// of B): how many of the first d merged elements are A's.  By one wave: 64
// probes per step, so three or four dependent loads where a binary search makes
// eighteen.  Every lane calls and gets the result.
__device__ __forceinline__ int32_t merge_split(const int32_t *A, int32_t na, const int32_t *B, int32_t nb, int32_t d) {
    int32_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    const int lane = threadIdx.x & 63;
    while (lo < hi) {  // the answer is in [lo, hi]: the first a with A[a] > B[d - 1 - a], or hi
        const int32_t a = lo + (int32_t)(((int64_t)(hi - lo) * lane) >> 6);
        const bool more = (int32_t)gload4(A + a) <= (int32_t)gload4(B + (d - 1 - a));  // true up to the answer
        const int c = __popcll(__ballot(more));
        const int32_t last = __shfl(a, c > 0 ? c - 1 : 0), next = __shfl(a, c < 64 ? c : 63);
        if (c < 64) hi = next;
        if (c > 0) lo = last + 1;
    }
    return lo;
}

// First index of the LDS list a[0, n) (ascending) holding a value >= v, or > v if upper.
__device__ __forceinline__ int lds_bound(const int32_t *a, int n, int32_t v, bool upper) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int32_t x = a[mid];
        if (x < v || (upper && x == v)) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One pass over the pending rows, the last batch's distinct rows and the
// prefetch list:
//  * Z1 by merging two ascending lists: pending entry i lands at i + (U rows
//    below it), U entry u at u + (pending rows at or below it), so a row in
//    both (a pending row the batch touched) takes two places, the pending one
//    a hole.  A key is a pending row neither touched nor named again, a hit or
//    miss the list does not name (F_INP, set by classification).  A block takes
//    tiles of kTile merged entries: the tile's ends in both lists by
//    merge_split, its rows into LDS, where each finds its place.  (A binary
//    search in the other list for every row was bound by the number of loads
//    in flight: 102 us on 290,000 + 170,000 rows in each of 4 tables.)
//  * new scores: hits take the touch score, or pscore if the list names them
//    (and lose F_PF); the list's untouched residents take pscore.  So their ring
//    entries go stale (slot_pos = -1).  F_INP stays until the append.
//  * the misses' scores, which admission reads.
// A thread reads a pending row's flags only if the batch did not touch it,
// and only hit threads write flags (of touched slots), so the reads see
// settled values.
constexpr int kTileQ = 4, kTile = kTileQ * kBlock;
__global__ void __launch_bounds__(kBlock) k_ring_touch(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int32_t s_row[kTile];  // the tile's pending rows, then its U rows
    __shared__ int32_t s_split[2];
    __shared__ int tmp[16];
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    if (!tb.ring_cap) return;
    TState &st = g.st[t];
    const int64_t ts = g.tstart[t], ps = g.pstart[t];
    const int32_t nu = p.have_fwd ? st.ucount : 0, pn = st.pend_n;
    const int32_t *prow = g.pend_row[st.pend_buf] + st.pend_off;
    const int32_t *pslot = g.pend_slot[st.pend_buf] + st.pend_off;
    const int32_t *urow = g.U + ts, *uslot = g.slotU + ts;
    int32_t *rcnt = tb.rcnt[st.r_buf];
    int2 *z = ring_zone(g, st, t);
    const int32_t n1 = pn + nu, np = st.pcount;
    if (blockIdx.x == 0 && threadIdx.x == 0) st.z1_len = n1;
    const int32_t *touch = tb.slot_touch, *pos = tb.slot_pos;
    const int32_t cap = tb.cap;
    const int tid = threadIdx.x, wave = tid >> 6;
    int keys = 0, stale = 0;
    // the ring entries e of slots sl (-1: none) go stale; every lane of the wave calls
    auto unring = [&](const int32_t (&sl)[kTileQ], const int32_t (&e)[kTileQ]) {
#pragma unroll
        for (int q = 0; q < kTileQ; ++q) {
            if (e[q] >= 0) {  // pending rows have no ring entry
                tb.slot_pos[sl[q]] = -1;
                ++stale;
            }
            chunk_sub(e[q] >= 0, e[q] / kRingChunk, rcnt);
        }
    };
    const int32_t tiles1 = (n1 + kTile - 1) / kTile, tiles = tiles1 + (np + kTile - 1) / kTile;
    for (int32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {  // block-uniform
        int32_t sl[kTileQ], e[kTileQ];  // residents whose score changes, their ring entries
        if (tile >= tiles1) {           // the prefetch list's residents
            const int32_t i0 = (tile - tiles1) * kTile;
            int32_t tch[kTileQ];
#pragma unroll
            for (int q = 0; q < kTileQ; ++q) {
                const int32_t i = i0 + q * kBlock + tid;
                sl[q] = i < np ? (int32_t)gload4(g.puref + ps + i) : -1;
            }
#pragma unroll
            for (int q = 0; q < kTileQ; ++q) {
                tch[q] = sl[q] >= 0 ? (int32_t)gload4(touch + sl[q]) : 0;
                e[q] = sl[q] >= 0 ? (int32_t)gload4(pos + sl[q]) : -1;
            }
#pragma unroll
            for (int q = 0; q < kTileQ; ++q)
                if (tch[q] == p.last_stamp) e[q] = -1;  // touched: its hit entry takes care of it
            unring(sl, e);
            continue;
        }
        const int32_t d0 = tile * kTile, d1 = d0 + kTile < n1 ? d0 + kTile : n1;
        if (wave < 2) {
            const int32_t a = merge_split(prow, pn, urow, nu, wave == 0 ? d0 : d1);
            if ((tid & 63) == 0) s_split[wave] = a;
        }
        __syncthreads();
        const int32_t a0 = s_split[0], na = s_split[1] - a0, b0 = d0 - a0, nt = d1 - d0;  // na pending, nt - na of U
        int32_t row[kTileQ], ref[kTileQ];
        uint32_t f[kTileQ], mf[kTileQ];
        int32_t tch[kTileQ];
#pragma unroll
        for (int q = 0; q < kTileQ; ++q) {
            const int32_t k = q * kBlock + tid;
            row[q] = 0, ref[q] = -1;
            if (k < na) {
                row[q] = (int32_t)gload4(prow + a0 + k);
                ref[q] = (int32_t)gload4(pslot + a0 + k);
                if (ref[q] >= cap) ref[q] = -1;
            } else if (k < nt) {
                row[q] = (int32_t)gload4(urow + b0 + (k - na));
                ref[q] = (int32_t)gload4(uslot + b0 + (k - na));
            }
            if (k < nt) s_row[k] = row[q];
        }
#pragma unroll
        for (int q = 0; q < kTileQ; ++q) {
            const int32_t k = q * kBlock + tid;
            const bool slot = k < nt && ref[q] >= 0, hit = slot && k >= na, miss = k >= na && k < nt && !slot;
            f[q] = slot ? gload4(tb.slot_flags + ref[q]) : 0u;
            tch[q] = slot && k < na ? (int32_t)gload4(touch + ref[q]) : 0;
            mf[q] = miss ? gload4(g.mflags + ts + (-ref[q] - 1)) : 0u;
            sl[q] = hit ? ref[q] : -1;
            e[q] = hit ? (int32_t)gload4(pos + ref[q]) : -1;
        }
        __syncthreads();  // the tile's rows are in LDS
#pragma unroll
        for (int q = 0; q < kTileQ; ++q) {
            const int32_t k = q * kBlock + tid;
            if (k >= nt) continue;
            int32_t at, zr = kRingHole;
            if (k < na) {
                at = d0 + k + lds_bound(s_row + na, nt - na, row[q], false);
                if (ref[q] >= 0 && tch[q] != p.last_stamp && !(f[q] & F_INP)) zr = ref[q];
            } else {
                at = d0 + (k - na) + lds_bound(s_row, na, row[q], true);
                if (ref[q] >= 0) {
                    if (!(f[q] & F_INP)) zr = ref[q];
                    if (f[q] & F_PF) tb.slot_flags[ref[q]] = f[q] & ~F_PF;
                } else {
                    const int32_t m = -ref[q] - 1;
                    const bool inp = (mf[q] & F_INP) != 0;
                    g.mscore[ts + m] = inp ? p.pscore : p.lru_touch;
                    if (!inp) zr = ring_ref_miss(m);
                }
            }
            z[at] = make_int2(zr, row[q]);
            keys += zr != kRingHole ? 1 : 0;
        }
        unring(sl, e);
        __syncthreads();  // before the next tile's rows take the LDS
    }
    const int k = block_sum(keys, tmp), ns = block_sum(stale, tmp);
    if (threadIdx.x == 0 && (k | ns)) atomicAdd(&st.touched, ((unsigned long long)k << 32) | (uint32_t)ns);
}

// One block per table: ring_cut, kept in the table's state for the kernels
// that apply it.
__global__ void __launch_bounds__(kRingThreads) k_ring_cut(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    const int t = blockIdx.x;
    const DTable &tb = g.tabs[t];
    if (!tb.ring_cap) return;
    TState &st = g.st[t];
    const Counts c = table_counts(tb, st, p);
    const int32_t nold = st.r_valid - (int32_t)(uint32_t)st.touched, z1 = (int32_t)(st.touched >> 32);
    const RingCut o = ring_cut(g, p, t, tb, st, c, nold, z1, st.z1_len, st.pcount, tmp);
    if (threadIdx.x == 0) {
        if (o.bad) atomicOr(g.err, ERR_INTERNAL);
        st.sel_mode = o.mode;
        st.prefix = o.thr;
        st.plc_nm = c.nm;
        st.r_cut = o.cut;
        st.r_zevict = o.zev;
        st.r_compact = o.compact ? 1 : 0;
        st.r_moved = o.moved;
    }
}

// Evict the live ring entries in [r_tail, r_cut) and, when the cut passed
// the whole ring, the Z1 and Z2 residents below the threshold.  When
// compacting, the live entries after the cut go, in order, to the front of
// the other buffer (whose chunk counts are set here; their slots learn their
// new index in the append, after every move has read the old ones).  A
// chunk per block iteration, one count update per chunk; freed slots gather
// in LDS and reach the free stack with one atomic per flush.
__global__ void __launch_bounds__(kBlock) k_ring_evict(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    __shared__ int s_base, s_n;
    __shared__ int32_t s_free[kRingEvictBuf];
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    if (!tb.ring_cap) return;
    TState &st = g.st[t];
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    auto flush = [&]() {  // every thread calls
        const int n = s_n;
        if (n == 0) return;
        if (threadIdx.x == 0) s_base = atomicAdd(&st.free_top, n);
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const int64_t at = (int64_t)s_base + i;
            if (at < tb.cap) tb.free_stack[at] = s_free[i];
            else atomicOr(g.err, ERR_INTERNAL);
        }
        __syncthreads();
        if (threadIdx.x == 0) s_n = 0;
        __syncthreads();
    };
    const bool reb = st.rebuild != 0;
    if (reb) map_clear_share(tb, blockIdx.x, gridDim.x);
    int nev = 0, nring = 0;
    unsigned long long dig = 0;
    // frees Q slots sl of rows r (where ev) and lists them; every lane of the wave
    // calls.  A slot's row and flags: k_ring_append, unless an admitted row takes it.
    constexpr int Q = 4;
    auto evict = [&](const bool (&ev)[Q], const int32_t (&sl)[Q], const int32_t (&r)[Q]) {
        if (!reb) map_delete_n<Q>(tb, r, ev);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint64_t m = __ballot(ev[q]);
            int wb = 0;
            if (lane == 0 && m) wb = atomicAdd(&s_n, __popcll(m));
            wb = __shfl(wb, 0);
            if (!ev[q]) continue;
            tb.slot_pos[sl[q]] = -1;
            dig += mix64(((unsigned long long)t << 40) | (unsigned long long)(uint32_t)r[q]);
            ++nev;
            s_free[wb + __popcll(m & ((1ull << lane) - 1ull))] = sl[q];
        }
    };
    const int32_t tail = st.r_tail, cut = st.r_cut, head = st.r_head, moved = st.r_moved;
    const bool compact = st.r_compact != 0;
    const int cur = st.r_buf;
    const int32_t *ring = tb.ring[cur];
    int32_t *dst = tb.ring[cur ^ 1];
    // chunks [tail's, hi): up to the cut's, or to the last live one when moving
    const int32_t hi = compact && moved > 0 ? (int32_t)(((int64_t)head + kRingChunk - 1) / kRingChunk)
                       : cut > tail          ? (cut - 1) / kRingChunk + 1
                                             : 0;
    for (int32_t ch = tail / kRingChunk + (int32_t)blockIdx.x; ch < hi; ch += (int32_t)gridDim.x) {
        const int32_t e0 = ch * kRingChunk + 4 * (int32_t)threadIdx.x;
        const uint4 v = gload16(ring + e0);
        const int32_t sl[Q] = {(int32_t)v.x, (int32_t)v.y, (int32_t)v.z, (int32_t)v.w};
        bool mv[Q], ev[Q];
        int32_t r[Q], ps[Q];
        int here = 0, nmv = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {  // eight loads in flight
            const bool ok = sl[i] >= 0 && sl[i] < tb.cap;
            ps[i] = ok ? (int32_t)gload4(tb.slot_pos + sl[i]) : -1;
            r[i] = ok ? (int32_t)gload4(tb.slot_row + sl[i]) : 0;
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int32_t e = e0 + i;
            const bool live = e >= tail && e < head && ps[i] == e;
            ev[i] = live && e < cut;
            mv[i] = live && !ev[i] && compact;
            here += ev[i] ? 1 : 0;
            nmv += mv[i] ? 1 : 0;
        }
        evict(ev, sl, r);
        int tot;
        const int ex = block_excl_scan(nmv, tmp, &tot);
        if (tot) {  // block-uniform; chunks with movers lie at or after the cut's
            int32_t at = tb.roff[ch] + ex;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!mv[i]) continue;
                if (at < moved) dst[at++] = sl[i];
                else atomicOr(g.err, ERR_INTERNAL);  // counts and entries disagree (never expected)
            }
        }
        const int hn = block_sum(here, tmp);
        if (threadIdx.x == 0 && hn) atomicSub(&tb.rcnt[cur][ch], hn);
        nring += here;
        if (list_past(&s_n, kRingEvictBuf - 4 * (int)blockDim.x)) flush();
    }
    if (compact) {  // the other buffer's chunk counts: [0, moved) live
        const int32_t nchunks = tb.ring_cap / kRingChunk;
        for (int32_t ch = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); ch < nchunks; ch += (int32_t)(gridDim.x * blockDim.x)) {
            const int64_t left = (int64_t)moved - (int64_t)ch * kRingChunk;
            tb.rcnt[cur ^ 1][ch] = left <= 0 ? 0 : left >= kRingChunk ? kRingChunk : (int32_t)left;
        }
    }
    if (st.r_zevict) {
        const int mode = st.sel_mode;
        const uint64_t thr = st.prefix;
        const int2 *z = ring_zone(g, st, t);
        const int64_t ps = g.pstart[t];
        const int32_t n1 = st.z1_len, n = n1 + st.pcount;
        for (int32_t base = (int32_t)(blockIdx.x * blockDim.x) * Q; base < n; base += (int32_t)(gridDim.x * blockDim.x) * Q) {
            int32_t sl[Q], r[Q];
            bool ev[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int32_t k = base + q * kBlock + (int32_t)threadIdx.x;
                sl[q] = -1, r[q] = 0;
                if (k < n1) {
                    const int2 zr = z[k];
                    r[q] = zr.y;
                    if (zr.x >= 0 && !kept(mode, make_key(p.lru_touch, zr.y, p.rowbits), thr)) sl[q] = zr.x;
                } else if (k < n) {
                    const int32_t v = g.puref[ps + (k - n1)];
                    r[q] = g.PU[ps + (k - n1)];
                    if (v >= 0 && !kept(mode, make_key(p.pscore, r[q], p.rowbits), thr)) sl[q] = v;
                }
                ev[q] = sl[q] >= 0;
            }
            evict(ev, sl, r);
            if (list_past(&s_n, kRingEvictBuf - Q * (int)blockDim.x)) flush();
        }
    }
    __syncthreads();
    flush();
    const int e = block_sum(nev, tmp), er = block_sum(nring, tmp);
    __shared__ unsigned long long s_dig[kBlock / 64];
    const unsigned long long d = block_sum64(dig, s_dig);
    if (threadIdx.x == 0) {
        if (d) atomicAdd(&st.digest_acc, 0ull - d);
        if (e != er) atomicAdd(&st.z_evicted, e - er);
    }
}

// After admission: when compacting, the moved slots' new indices (every move
// has read the old ones); Z1's kept keys to ring entries [head, + z1_len) of
// the buffer that stays current (a chunk per block iteration); Z2's rows and
// their slots (-1 where not kept) to the pending list of buffer wr, the kept
// residents losing F_INP.  Admitted candidates' slots come from admission.
__global__ void __launch_bounds__(kBlock) k_ring_append(DGlobal g, PlcParams p, int wr) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    if (!tb.ring_cap) return;
    TState &st = g.st[t];
    const int mode = st.sel_mode;
    const uint64_t thr = st.prefix;
    const int64_t ts = g.tstart[t], ps = g.pstart[t];
    const bool compact = st.r_compact != 0;
    const int buf = compact ? st.r_buf ^ 1 : st.r_buf;
    const int32_t n1 = st.z1_len, head = compact ? st.r_moved : st.r_head;
    if ((int64_t)head + n1 > tb.ring_cap) {  // compaction made room; never expected
        if (threadIdx.x == 0) atomicOr(g.err, ERR_INTERNAL);
        return;
    }
    int32_t *ring = tb.ring[buf];
    if (compact) {
        for (int32_t k = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); k < head; k += (int32_t)(gridDim.x * blockDim.x)) {
            const int32_t sl = ring[k];
            if (sl >= 0 && sl < tb.cap) tb.slot_pos[sl] = k;
            else atomicOr(g.err, ERR_INTERNAL);
        }
    }
    const int2 *z = ring_zone(g, st, t);
    int added = 0;
    if (n1 > 0) {
        const int32_t c1 = (head + n1 - 1) / kRingChunk;
        for (int32_t ch = head / kRingChunk + (int32_t)blockIdx.x; ch <= c1; ch += (int32_t)gridDim.x) {
            int add = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t e = ch * kRingChunk + 4 * (int32_t)threadIdx.x + i;
                if (e < head || e >= head + n1) continue;
                const int2 zr = z[e - head];
                int32_t sl = kRingHole;
                if (zr.x != kRingHole && kept(mode, make_key(p.lru_touch, zr.y, p.rowbits), thr))
                    sl = zr.x >= 0 ? zr.x : g.mslot[ts + (-1 - zr.x)];
                if (sl != kRingHole && (sl < 0 || sl >= tb.cap)) {
                    atomicOr(g.err, ERR_INTERNAL);
                    sl = kRingHole;
                }
                ring[e] = sl;
                if (sl != kRingHole) {
                    tb.slot_pos[sl] = e;
                    ++add;
                }
            }
            const int an = block_sum(add, tmp);
            if (threadIdx.x == 0 && an) atomicAdd(&tb.rcnt[buf][ch], an);
            added += an;
        }
    }
    // slots freed and not taken again (the free stack's new entries below its
    // new top); in a full cache in steady state there are none
    const int32_t left = st.free_top - st.popped;
    for (int32_t k = st.free0 + (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); k < left; k += (int32_t)(gridDim.x * blockDim.x)) {
        const int32_t sl = tb.free_stack[k];
        tb.slot_row[sl] = -1;
        tb.slot_flags[sl] = 0;
    }
    int keepn = 0;
    int32_t *prow = g.pend_row[wr] + ps, *pslot = g.pend_slot[wr] + ps;
    for (int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < st.pcount; i += (int32_t)(gridDim.x * blockDim.x)) {
        const int32_t row = g.PU[ps + i], v = g.puref[ps + i];
        int32_t sl = -1;
        if (kept(mode, make_key(p.pscore, row, p.rowbits), thr)) {
            if (v >= 0) {
                sl = v;
                tb.slot_flags[v] &= ~F_INP;
            } else {
                sl = v > kRingNewBase ? g.mslot[ts + (-1 - v)] : g.npslot[ps + (kRingNewBase - v)];
            }
        }
        prow[i] = row;
        pslot[i] = sl;
        keepn += sl >= 0 ? 1 : 0;
    }
    const int kn = block_sum(keepn, tmp);
    if (threadIdx.x == 0 && (kn | added)) atomicAdd(&st.appended, ((unsigned long long)added << 32) | (uint32_t)kn);
    if (blockIdx.x == 0 && threadIdx.x == 0) st.pend_buf = wr;
}

// ----------------------------------------------------------------- launchers

static inline unsigned ring_grid(int64_t n, int per_block, unsigned cap) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (int64_t)cap) b = cap;
    return (unsigned)b;
}

void launch_ring_rank(const DGlobal &g, const PlcParams &p, int64_t item_bound, hipStream_t s) {
    k_ring_touch<<<dim3(ring_grid(item_bound, kTile, 1024), g.T), kBlock, 0, s>>>(g, p);
    k_ring_cut<<<g.T, kRingThreads, 0, s>>>(g, p);
}

void launch_ring_evict(const DGlobal &g, const PlcParams &p, int64_t item_bound, int32_t ring_chunks, hipStream_t s) {
    // the cut is typically a few chunks past the front; a compaction walks
    // every chunk, so blocks loop
    const unsigned gx = std::max(ring_grid(item_bound, kBlock * 4, 512), ring_grid(ring_chunks, 64, 256));
    k_ring_evict<<<dim3(gx, g.T), kBlock, 0, s>>>(g, p);
}

void launch_ring_store(const DGlobal &g, const PlcParams &p, int64_t item_bound, int32_t max_cap, int wr,
                       hipStream_t s) {
    const unsigned gx = std::max(ring_grid(item_bound, kBlock * 4, 1024), ring_grid(max_cap, kBlock * 16, 1024));
    k_ring_append<<<dim3(gx, g.T), kBlock, 0, s>>>(g, p, wr);
}

}  // namespace recmg

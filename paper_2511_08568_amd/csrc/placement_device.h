// Device code of the placement shared by the kernels that run one step of it
// over many blocks (placement.hip, ring.hip, setassoc.hip) and the kernel that
// runs all of it for a table in one block (small.hip).
#pragma once

#include "launch.h"

namespace recmg {

// ----------------------------------------------------------------- ranking

__device__ __forceinline__ int pass_shift(const PlcParams &p, int pass) { return kRadixBits * (p.passes - 1 - pass); }
__device__ __forceinline__ int pass_width(const PlcParams &p, int pass) {
    return pass == 0 ? p.total_bits - kRadixBits * (p.passes - 1) : kRadixBits;
}

// Histogram increment, aggregated over the wave for the first active lane's
// bin: the keys of one table bunch up in few digits (LRU scores are batch
// numbers), and 64 lanes adding 1 to one LDS word would serialise.
__device__ __forceinline__ void hist_add(int *h, bool active, uint32_t bin) {
    const uint64_t act = __ballot(active);
    if (act == 0) return;
    const int lead = __ffsll((unsigned long long)act) - 1;
    const uint32_t b0 = (uint32_t)__shfl((int)bin, lead);
    const uint64_t same = __ballot(active && bin == b0);
    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&h[b0], __popcll(same));
    if (active && bin != b0) atomicAdd(&h[bin], 1);
}

// The digit of one pass from a table's histogram in LDS: bins are taken from
// the top until `need` keys are covered; the bin reached (*digit) extends the
// threshold prefix and the keys still needed inside it (*rest) carry over to
// the next pass.  Every thread of the block calls; blockDim.x divides kRadix;
// the results are valid in every thread.
__device__ __forceinline__ void pick_digit(const int *s_hist, int need, int *tmp, int *digit, int *rest) {
    __shared__ int s_digit, s_rest;
    // thread k owns bin group (groups - 1 - k), so an exclusive scan gives the
    // keys in the groups above
    if (threadIdx.x == 0) {  // a histogram short of `need` (never, when the counts hold) keeps digit 0
        s_digit = 0;
        s_rest = need;
    }
    const int per = kRadix / (int)blockDim.x;
    const int grp = (int)blockDim.x - 1 - (int)threadIdx.x;
    int cs = 0;
    for (int b = 0; b < per; ++b) cs += s_hist[grp * per + b];
    int tot;
    const int above = block_excl_scan(cs, tmp, &tot);
    if (above < need && above + cs >= need) {
        int cum = above;
        for (int b = grp * per + per - 1; b >= grp * per; --b) {
            if (cum + s_hist[b] >= need) {
                s_digit = b;
                s_rest = need - cum;
                break;
            }
            cum += s_hist[b];
        }
    }
    __syncthreads();
    *digit = s_digit;
    *rest = s_rest;
    __syncthreads();
}

// The scans over every slot (score update, select passes, evict) take four
// consecutive slots per thread with 16-byte loads issued together: with one
// slot per thread and a score load that waited for the row load, they were
// bound by load latency (configuration 4's 78 million slots: about 1 TB/s).
// Slots [k0, k0 + 4) of a table, absent ones (k >= cap) reading row -1.
__device__ __forceinline__ void slot_quad(const int32_t *a, int64_t k0, int64_t cap, int32_t fill, int32_t (&v)[4]) {
    if (k0 + 3 < cap) {
        const uint4 w = gload16(a + k0);
        v[0] = (int32_t)w.x, v[1] = (int32_t)w.y, v[2] = (int32_t)w.z, v[3] = (int32_t)w.w;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = k0 + i < cap ? (int32_t)gload4(a + k0 + i) : fill;
    }
}

// Scores of every candidate of table t (written back) and, when `sel`, the
// histogram of the first select pass, over items tid, tid + stride, ...
// (stride a multiple of 64: hist_add is wave-wide).  inp_of(row, flags): whether
// the prefetch list names the row (of a slot or a miss with these flags).
template <class Inp>
__device__ __forceinline__ void update_items(const DGlobal &g, const PlcParams &p, const DTable &tb, const Counts &c,
                                             int t, int *s_hist, bool sel, int64_t tid, int64_t stride, Inp inp_of) {
    const int64_t ts = g.tstart[t], ps = g.pstart[t];
    const int shift = pass_shift(p, 0);
    const uint32_t dmask = (1u << pass_width(p, 0)) - 1u;
    const int64_t cap = c.cap;
    // resident slots, four per thread; every lane runs the same number of
    // iterations (hist_add is wave-wide)
    const int64_t ngrp = (cap + 3) / 4, ngrp_r = (ngrp + 63) & ~(int64_t)63;
    for (int64_t q = tid; q < ngrp_r; q += stride) {
        const int64_t k0 = 4 * q;
        const int64_t lim = q < ngrp ? cap : 0;  // lanes past the last group see no slot
        int32_t row[4], sc[4], fl[4], tch[4];
        slot_quad(tb.slot_row, k0, lim, -1, row);
        slot_quad(tb.slot_score, k0, lim, 0, sc);
        slot_quad(reinterpret_cast<const int32_t *>(tb.slot_flags), k0, lim, 0, fl);
        slot_quad(tb.slot_touch, k0, lim, -1, tch);
        uint32_t cbw = 0;
        if (k0 + 3 < lim) cbw = gload4(tb.slot_cbit + k0);
        else
            for (int i = 0; i < 4; ++i)
                if (k0 + i < lim) cbw |= (uint32_t)tb.slot_cbit[k0 + i] << (8 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t k = k0 + i;
            const int32_t r = row[i];
            int32_t s = sc[i];
            uint32_t f = (uint32_t)fl[i];
            const int cb = (int)((cbw >> (8 * i)) & 0xffu);
            if (k < lim) {
                if (p.prio) s = s > 0 ? s - 1 : 0;
                if (r >= 0 && tch[i] == p.last_stamp) {
                    f &= ~F_PF;
                    s = touch_score(p, tb, r, cb);
                }
                if (r >= 0 && s < p.pscore && inp_of(r, f)) s = p.pscore;
                // written back only where they change (most slots keep both)
                if (r >= 0 && s != sc[i]) tb.slot_score[k] = s;
                if (r >= 0 && (f & ~F_INP) != (uint32_t)fl[i]) tb.slot_flags[k] = f & ~F_INP;
            }
            if (sel) hist_add(s_hist, k < lim && r >= 0, (uint32_t)(make_key(s, r < 0 ? 0 : r, p.rowbits) >> shift) & dmask);
        }
        if (cbw) {  // caching bits are zero between placements
            if (k0 + 3 < lim) *reinterpret_cast<uint32_t *>(tb.slot_cbit + k0) = 0u;
            else
                for (int i = 0; i < 4; ++i)
                    if (k0 + i < lim && ((cbw >> (8 * i)) & 0xffu)) tb.slot_cbit[k0 + i] = 0;
        }
    }
    // candidates: the last batch's misses, then new prefetch rows
    const int64_t nc = (int64_t)c.nm + c.nnp, nc_r = (nc + 63) & ~(int64_t)63;
    for (int64_t k = tid; k < nc_r; k += stride) {
        int32_t row = -1, s = 0;
        if (k >= nc) {
        } else if (k < c.nm) {
            const int64_t m = ts + k;
            row = g.M[m];
            const uint32_t f = g.mflags[m];
            s = touch_score(p, tb, row, g.mcbit[m]);
            if (s < p.pscore && inp_of(row, f)) s = p.pscore;
            g.mscore[m] = s;
        } else {
            row = g.NP[ps + (k - c.nm)];
            s = new_prefetch_score(p, tb, row);
        }
        if (sel) hist_add(s_hist, row >= 0, (uint32_t)(make_key(s, row < 0 ? 0 : row, p.rowbits) >> shift) & dmask);
    }
}

// Key of candidate k (k < nm: a miss of the last batch; else a new prefetch row).
__device__ __forceinline__ uint64_t cand_key(const DGlobal &g, const DTable &tb, const Counts &c, const PlcParams &p,
                                             int64_t ts, int64_t ps, int64_t k) {
    int32_t row, s;
    if (k < c.nm) {
        const int64_t m = ts + k;
        row = g.M[m];
        s = g.mscore[m];
    } else {
        row = g.NP[ps + (k - c.nm)];
        s = new_prefetch_score(p, tb, row);
    }
    return make_key(s, row, p.rowbits);
}

// Histogram of pass `pass` over the keys of table t whose higher digits equal
// `prefix`, over items tid, tid + stride, ... (stride a multiple of 64).
__device__ __forceinline__ void select_items(const DGlobal &g, const PlcParams &p, const DTable &tb, const Counts &c,
                                             int t, int *s_hist, int pass, uint64_t prefix, int64_t tid,
                                             int64_t stride) {
    const int64_t ts = g.tstart[t], ps = g.pstart[t];
    const int shift = pass_shift(p, pass);
    const int64_t cap = c.cap;
    const int64_t ngrp = (cap + 3) / 4, ngrp_r = (ngrp + 63) & ~(int64_t)63;
    for (int64_t q = tid; q < ngrp_r; q += stride) {
        const int64_t k0 = 4 * q;
        const int64_t lim = q < ngrp ? cap : 0;
        int32_t row[4], sc[4];
        slot_quad(tb.slot_row, k0, lim, -1, row);
        slot_quad(tb.slot_score, k0, lim, 0, sc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t key = make_key(sc[i], row[i] < 0 ? 0 : row[i], p.rowbits);
            const bool in = row[i] >= 0 && (key >> (shift + kRadixBits)) == prefix;
            hist_add(s_hist, in, (uint32_t)(key >> shift) & (kRadix - 1));
        }
    }
    const int64_t nc = (int64_t)c.nm + c.nnp, nc_r = (nc + 63) & ~(int64_t)63;
    for (int64_t k = tid; k < nc_r; k += stride) {
        const uint64_t key = k < nc ? cand_key(g, tb, c, p, ts, ps, k) : 0;
        const bool in = k < nc && (key >> (shift + kRadixBits)) == prefix;
        hist_add(s_hist, in, (uint32_t)(key >> shift) & (kRadix - 1));
    }
}

struct FlagInp {  // the general sequence: classification has flagged the named rows
    __device__ bool operator()(int32_t, uint32_t f) const { return (f & F_INP) != 0; }
};

// The whole ranking of a table by one block: the scores of every candidate and,
// when some must go (SEL_SELECT), the threshold key from every pass's histogram
// in LDS.  blockDim.x divides kRadix; every thread calls; ends with a barrier.
template <class Inp>
__device__ __forceinline__ uint64_t rank_block(const DGlobal &g, const PlcParams &p, const DTable &tb, const Counts &c,
                                               int t, int *s_hist, int *tmp, Inp inp_of) {
    const bool sel = c.mode == SEL_SELECT;
    for (int b = threadIdx.x; b < kRadix; b += blockDim.x) s_hist[b] = 0;
    __syncthreads();
    update_items(g, p, tb, c, t, s_hist, sel, threadIdx.x, blockDim.x, inp_of);
    __syncthreads();  // also makes the scores written above visible to the block
    uint64_t prefix = 0;
    int need = c.keep;
    for (int pass = 0; sel && pass < p.passes; ++pass) {
        if (pass > 0) {
            for (int b = threadIdx.x; b < kRadix; b += blockDim.x) s_hist[b] = 0;
            __syncthreads();
            select_items(g, p, tb, c, t, s_hist, pass, prefix, threadIdx.x, blockDim.x);
            __syncthreads();
        }
        int digit, rest;
        pick_digit(s_hist, need, tmp, &digit, &rest);
        prefix = pass == 0 ? (uint64_t)digit : ((prefix << kRadixBits) | (uint64_t)digit);
        need = rest;
    }
    return prefix;
}

// ----------------------------------------------------------------- the last batch

// What a placement takes from the last batch besides its misses: PRIORITY the
// caching bits, OR-ed per row into a byte of the slot (hit) or of the miss entry
// (every writer stores the same value 1, so plain byte stores suffice, no
// read-modify-write atomics on popular rows); LFU_BATCH one more batch for every
// distinct row (rows of U are distinct, so plain increments suffice).  This block's
// share of n indices; bits: NULL under LFU_BATCH.  It depends on nothing the
// placement computes and is wanted by its scores only, so it rides with a kernel
// that comes before them (a kernel of its own took 7 us on a batch of 13,000 ids
// and 15 us on 1.7 million; a step of 26 32-way LFU tables 182 -> 172 us, of 13
// ragged PRIORITY tables 257 -> 247).
__device__ __forceinline__ void last_batch_share(const DGlobal &g, const uint8_t *__restrict__ bits, int64_t n) {
    __shared__ int64_t s_ts[RECMG_MAX_TABLES + 1];
    __shared__ int32_t s_uc[RECMG_MAX_TABLES];
    for (int t = threadIdx.x; t <= g.T; t += blockDim.x) {
        s_ts[t] = g.tstart[t];
        if (t < g.T) s_uc[t] = g.st[t].ucount;
    }
    __syncthreads();
    int64_t lo, hi;
    block_share(n, &lo, &hi);
    if (lo >= hi) return;
    int t = find_seg(s_ts, g.T, lo);
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        if (bits && !bits[i]) continue;
        while (i >= s_ts[t + 1]) ++t;
        if (bits) {
            const int32_t s = g.src[i];
            uint8_t *f = s >= 0 ? &g.tabs[t].slot_cbit[s] : &g.mcbit[s_ts[t] + (-(int64_t)s - 1)];
            if (!*f) *f = 1;
        } else if (i - s_ts[t] < s_uc[t]) {
            g.tabs[t].freq[g.U[i]] += 1;
        }
    }
}

// ----------------------------------------------------------------- freed slots

// Whether a block's LDS list has grown past `limit`, the same answer in every
// thread: the count is read between two barriers, so no wave appends to it again
// before the slowest has read it.  (With the first barrier alone a fast wave's
// next append can fall between two waves' reads; they would then part ways in
// front of the flush, which has barriers of its own.)  Every thread calls.
__device__ __forceinline__ bool list_past(const int *s_n, int limit) {
    __syncthreads();
    const bool past = *s_n > limit;
    __syncthreads();
    return past;
}

// ----------------------------------------------------------------- map upkeep

// A map of many deleted entries is rebuilt in the placement after the one that
// passed a quarter of it (TState::rebuild): its lookups go first, then eviction
// clears the map instead of deleting from it, admission inserts nothing, and
// the placement's last kernel inserts every resident (map_refill_share).  So no
// kernel is launched for a rebuild that most placements do not need.
__device__ __forceinline__ void map_clear_share(const DTable &tb, int block, int nblocks) {
    const int64_t n2 = ((int64_t)tb.map_mask + 1) / 2;  // 16 bytes are two entries; at least 64 entries
    int4 *m = reinterpret_cast<int4 *>(tb.map);
    for (int64_t i = (int64_t)block * blockDim.x + threadIdx.x; i < n2; i += (int64_t)nblocks * blockDim.x)
        m[i] = make_int4(kEmpty, -1, kEmpty, -1);
}
__device__ __forceinline__ void map_refill_share(const DTable &tb, int block, int nblocks) {
    if (tb.ways) return;
    for (int64_t k = (int64_t)block * blockDim.x + threadIdx.x; k < tb.cap; k += (int64_t)nblocks * blockDim.x) {
        const int32_t row = (int32_t)gload4(tb.slot_row + k);
        if (row >= 0) map_insert(tb, row, (int32_t)k);
    }
}

// ----------------------------------------------------------------- resident rings (ring.hip)

constexpr int kRingThreads = 1024;  // one-block-per-table kernels: one entry of a chunk per thread
static_assert(kRingThreads == kRingChunk, "the cut takes a chunk's entries one per thread");

__device__ __forceinline__ bool ring_live(const DTable &tb, int32_t slot, int32_t e) {
    return slot >= 0 && slot < tb.cap && tb.slot_pos[slot] == e;
}

// One live entry less in the chunk of every lane with `want`.  Rows come in
// order and so did the run that holds their entries, so a wave's entries lie in
// few chunks: one atomic each for the first four, as 42,000 atomics on some 20
// words took 70 us where all residents of a small cache are touched.  Every lane
// of the wave calls.
__device__ __forceinline__ void chunk_sub(bool want, int32_t chunk, int32_t *rcnt) {
    const int lane = threadIdx.x & 63;
    uint64_t pending = __ballot(want);
    for (int k = 0; k < 4 && pending; ++k) {
        const int leader = __ffsll((unsigned long long)pending) - 1;
        const int32_t c = __shfl(chunk, leader);
        const uint64_t grp = __ballot(want && chunk == c);
        if (lane == leader) atomicSub(&rcnt[c], (int)__popcll(grp));
        if (chunk == c) want = false;
        pending &= ~grp;
    }
    if (want) atomicSub(&rcnt[chunk], 1);
}

// Table t's zone Z1: entries [pend_off + tstart[t], + z1_len) of g.zone.
// Tables' regions are disjoint: pend_off and tstart partition the prefetch
// and index spaces, and z1_len = pend_n + (last forward's distinct rows).
__device__ __forceinline__ int2 *ring_zone(const DGlobal &g, const TState &st, int t) {
    return g.zone + st.pend_off + g.tstart[t];
}

// Where the D keys to drop end: the mode and threshold key that admission
// applies to the candidates, the ring's cut, whether Z1/Z2 residents go, and
// whether the live entries after the cut move to the front of the other buffer
// (when this placement's run would not fit behind them), with each chunk's
// first new index in roff.  By one block of kRingThreads threads; every thread
// calls and gets the result.  nold: live ring entries; z1: keys of Z1 in
// z1_len zone entries; z2: distinct prefetch rows.
struct RingCut {
    int32_t mode, cut, zev, moved;
    bool compact, bad;
    uint64_t thr;
};

__device__ __forceinline__ RingCut ring_cut(const DGlobal &g, const PlcParams &p, int t, const DTable &tb,
                                            const TState &st, const Counts &c, int32_t nold, int32_t z1,
                                            int32_t z1_len, int32_t z2, int *tmp) {
    __shared__ int32_t s_at, s_rest;
    const int64_t nk = (int64_t)st.n_res + c.nm + c.nnp;
    const int64_t drop = nk - c.keep;
    const int32_t head = st.r_head, tail = st.r_tail;
    // selects: an index would put a local copy of the descriptor in scratch memory
    const int32_t *ring = st.r_buf ? tb.ring[1] : tb.ring[0];
    const int32_t *rcnt = st.r_buf ? tb.rcnt[1] : tb.rcnt[0];
    const int32_t nch = (int32_t)(((int64_t)head + kRingChunk - 1) / kRingChunk);
    bool bad = nold < 0 || (int64_t)nold + z1 + z2 != nk;  // every key sits in the ring, Z1 or Z2
    int32_t mode = c.mode, cut = tail, zev = 0, cut_live = 0;  // cut_live: live entries of cut's chunk before it
    uint64_t thr = make_key(p.lru_touch, 0, p.rowbits);  // below every key of Z1 and Z2
    if (!bad && drop > 0 && drop <= nold) {
        // the drop-th live entry from the front: whole chunks by their counts,
        // then the entries of the chunk that reaches it
        mode = SEL_SELECT;
        int32_t need = (int32_t)drop, cc = -1;
        for (int32_t base = tail / kRingChunk; base < nch; base += kRingThreads) {
            const int32_t ch = base + (int32_t)threadIdx.x;
            const int v = ch < nch ? rcnt[ch] : 0;
            int tot;
            const int ex = block_excl_scan(v, tmp, &tot);
            if (need <= tot) {  // block-uniform
                if (ex < need && ex + v >= need) {
                    s_at = ch;
                    s_rest = need - ex;
                }
                __syncthreads();
                cc = s_at;
                need = s_rest;
                __syncthreads();  // read before s_at is reused below
                break;
            }
            need -= tot;
        }
        if (cc < 0) {
            bad = true;
        } else {
            const int32_t e = cc * kRingChunk + (int32_t)threadIdx.x;
            const bool live = e >= tail && e < head && ring_live(tb, ring[e], e);
            if (threadIdx.x == 0) s_at = -1;
            int tot;
            const int ex = block_excl_scan(live ? 1 : 0, tmp, &tot);  // its barriers order s_at's reset
            if (live && ex + 1 == need) s_at = e + 1;
            __syncthreads();
            cut = s_at;
            if (cut < 0) bad = true;
            else if (cut / kRingChunk == cc) cut_live = need;
        }
    } else if (!bad && drop > nold) {
        // the whole ring goes; the threshold is the key of rank r of Z1, or of
        // rank r - |Z1| of Z2 (every prefetch row is a key)
        cut = head;
        zev = 1;
        const int32_t r = (int32_t)(drop - nold);
        if (r < z1) {
            const int2 *z = ring_zone(g, st, t);
            const int32_t n = z1_len;
            int32_t want = r;
            if (threadIdx.x == 0) s_at = -1;
            __syncthreads();
            for (int32_t base = 0; base < n; base += kRingThreads) {
                const int32_t j = base + (int32_t)threadIdx.x;
                const int2 zr = j < n ? z[j] : make_int2(kRingHole, 0);
                const bool key = zr.x != kRingHole;
                int tot;
                const int ex = block_excl_scan(key ? 1 : 0, tmp, &tot);
                if (want < tot) {  // block-uniform
                    if (key && ex == want) s_at = zr.y;
                    __syncthreads();
                    break;
                }
                want -= tot;
            }
            if (s_at < 0) bad = true;
            thr = make_key(p.lru_touch, s_at < 0 ? 0 : s_at, p.rowbits);
            mode = SEL_SELECT;
        } else if (r - z1 < z2) {
            thr = make_key(p.pscore, g.PU[g.pstart[t] + (r - z1)], p.rowbits);
            mode = SEL_SELECT;
        } else {
            mode = SEL_NONE;
        }
    } else if (!bad) {
        mode = SEL_ALL;  // nothing to drop
    }
    const int32_t moved = bad ? 0 : (int32_t)(drop <= 0 ? nold : drop <= nold ? nold - drop : 0);
    const bool compact = (int64_t)head + z1_len > tb.ring_cap;
    if (compact && moved > 0) {
        // first new index of each chunk from cut's on: its live entries at or after the cut
        int32_t run = 0;
        const int32_t c0 = cut / kRingChunk;
        for (int32_t base = c0; base < nch; base += kRingThreads) {
            const int32_t ch = base + (int32_t)threadIdx.x;
            const int v = ch < nch ? rcnt[ch] - (ch == c0 ? cut_live : 0) : 0;
            int tot;
            const int ex = block_excl_scan(v, tmp, &tot);
            if (ch < nch) tb.roff[ch] = run + ex;
            run += tot;
        }
        if (run != moved) bad = true;
    }
    RingCut o;
    o.mode = mode, o.cut = cut, o.zev = zev, o.moved = moved, o.compact = compact, o.bad = bad, o.thr = thr;
    return o;
}

// ----------------------------------------------------------------- set-associative counts

// Set-associative placement blocks' records [8] of table kt (in sa_btab order),
// slice `part` of `parts` of its blocks, added to the table's counters: one
// atomic per counter.  Every thread of the block calls.
__device__ __forceinline__ void sa_sum_records(const DGlobal &g, int kt, int part, int parts, long long *tmp) {
    TState &st = g.st[g.sa_btab[kt]];
    const int32_t b0 = g.sa_bstart[kt], b1 = g.sa_bstart[kt + 1];
    long long v[7] = {0, 0, 0, 0, 0, 0, 0};
    long long dg = 0;  // digests add modulo 2^64
    for (int32_t b = b0 + part * (int32_t)blockDim.x + (int32_t)threadIdx.x; b < b1; b += parts * (int32_t)blockDim.x) {
#pragma unroll
        for (int k = 0; k < 7; ++k) v[k] += g.sa_part[(int64_t)b * 8 + k];
        dg = (long long)((unsigned long long)dg + (unsigned long long)g.sa_part[(int64_t)b * 8 + 7]);
    }
    long long tot[7], d;
#pragma unroll
    for (int k = 0; k < 7; ++k) (void)block_excl_scan64(v[k], tmp, &tot[k]);
    (void)block_excl_scan64(dg, tmp, &d);
    if (threadIdx.x != 0) return;
    if (parts == 1) {  // the only adder: plain updates, which this thread may read back
        st.evicted += (int32_t)tot[0];
        st.adm_miss += (int32_t)tot[1];
        st.p_fill += (int32_t)tot[2];
        st.p_drop += (int32_t)tot[3];
        st.m_drop += (int32_t)tot[4];
        st.n_res += (int32_t)tot[5];
        st.p_res += (int32_t)tot[6];
        st.digest_acc += (unsigned long long)d;
    } else {
        if (tot[0]) atomicAdd(&st.evicted, (int32_t)tot[0]);
        if (tot[1]) atomicAdd(&st.adm_miss, (int32_t)tot[1]);
        if (tot[2]) atomicAdd(&st.p_fill, (int32_t)tot[2]);
        if (tot[3]) atomicAdd(&st.p_drop, (int32_t)tot[3]);
        if (tot[4]) atomicAdd(&st.m_drop, (int32_t)tot[4]);
        if (tot[5]) atomicAdd(&st.n_res, (int32_t)tot[5]);
        if (tot[6]) atomicAdd(&st.p_res, (int32_t)tot[6]);
        if (d) atomicAdd(&st.digest_acc, (unsigned long long)d);
    }
}

// The same for table t by the block that goes on to publish the table.
__device__ __forceinline__ void sa_sum_table(const DGlobal &g, int t, int nsa, long long *tmp) {
    for (int kt = 0; kt < nsa; ++kt)  // t's place in sa_btab
        if (g.sa_btab[kt] == t) {
            sa_sum_records(g, kt, 0, 1, tmp);
            break;
        }
}

}  // namespace recmg

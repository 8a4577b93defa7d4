// Batches of few ids per table: one block of 1,024 threads per table does the
// work of several kernels, with barriers of the block between its steps.
//
// What bounds them: a batch of some thousand ids gives every kernel of the
// general sequence a few microseconds of dependent loads and a launch, and
// those add up to the whole call.  The ids of a table meet in one block here,
// so the presence bitmap, its prefix sums and every counter stay in LDS, and
// what passes from step to step costs a barrier instead of a launch.
#include "launch.h"
#include "placement_device.h"

namespace recmg {

constexpr int kSmallThreads = 1024;
// bitmap words per group whose first rank is kept (a rank is that plus the
// popcounts of at most eight words)
constexpr int kRankGroup = 8;

// Presence bitmap of one table in LDS: NB bitmap blocks (32,768 rows each) at
// most, with the rank of the first set bit of every kRankGroup words.
template <int NB>
struct LdsBitmap {
    uint4 w4[NB * kWordsPerBlock / 4];
    int pre[NB * kWordsPerBlock / kRankGroup];

    __device__ uint32_t *words() { return reinterpret_cast<uint32_t *>(w4); }
    __device__ void clear(int nw) {  // nw: words in use, a multiple of kWordsPerBlock
        for (int k = threadIdx.x; k < nw / 4; k += kSmallThreads) w4[k] = make_uint4(0u, 0u, 0u, 0u);
    }
    __device__ bool test(uint32_t pos) { return words()[pos >> 5] >> (pos & 31) & 1u; }
    __device__ void set(uint32_t pos) {
        uint32_t *w = words() + (pos >> 5);
        const uint32_t bit = 1u << (pos & 31);
        if (!(*w & bit)) atomicOr(w, bit);  // popular rows: no atomic for a bit seen set
    }
    // Fills pre; returns the number of set bits.  Every thread calls, after a
    // barrier that follows the last set(); ends with a barrier.
    __device__ int scan(int nw, int *tmp) {
        // a group is two 16-byte words, counted by neighbouring lanes
        for (int k = threadIdx.x; k < nw / 4; k += kSmallThreads) {
            const uint4 v = w4[k];
            int c = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
            c += __shfl_xor(c, 1);
            if (!(k & 1)) pre[k >> 1] = c;
        }
        __syncthreads();
        constexpr int per = (NB * kWordsPerBlock / kRankGroup + kSmallThreads - 1) / kSmallThreads;
        const int ng = nw / kRankGroup, g0 = (int)threadIdx.x * per;
        int v[per], s = 0;
#pragma unroll
        for (int i = 0; i < per; ++i) {
            v[i] = g0 + i < ng ? pre[g0 + i] : 0;
            s += v[i];
        }
        int tot;
        int at = block_excl_scan(s, tmp, &tot);
#pragma unroll
        for (int i = 0; i < per; ++i) {
            if (g0 + i < ng) pre[g0 + i] = at;
            at += v[i];
        }
        __syncthreads();
        return tot;
    }
    // Set bits below pos (pos itself set or not).
    __device__ int rank(uint32_t pos) {
        const uint32_t w = pos >> 5, g = w / kRankGroup, in = w % kRankGroup;
        const uint4 a = w4[2 * g], b = w4[2 * g + 1];
        const uint32_t v[kRankGroup] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        int r = pre[g];
#pragma unroll
        for (int k = 0; k < kRankGroup; ++k)
            r += k < (int)in ? __popc(v[k]) : k == (int)in ? __popc(v[k] & ((1u << (pos & 31)) - 1u)) : 0;
        return r;
    }
    // f(word index, its bits, rank of its first set bit) for every non-zero
    // word.  nw is a multiple of kSmallThreads, so every lane runs the same
    // iterations and the eight words of a group meet in eight neighbouring lanes.
    template <class F>
    __device__ void each_word(int nw, F f) {
        for (int w = threadIdx.x; w < nw; w += kSmallThreads) {
            const uint32_t bits = words()[w];
            const int c = __popc(bits);
            int x = c;
#pragma unroll
            for (int d = 1; d < kRankGroup; d <<= 1) {
                const int y = __shfl_up(x, d, kRankGroup);
                if ((int)(threadIdx.x & (kRankGroup - 1)) >= d) x += y;
            }
            if (bits) f(w, bits, pre[w / kRankGroup] + x - c);
        }
    }
};
static_assert(kWordsPerBlock % kSmallThreads == 0, "each_word: whole passes of the block");

// slots (or misses) of a table's first distinct rows kept in LDS for the
// per-index pass, which looks each up several times; the others come from L2
constexpr int kLdsSlots = 3072;

// Positions handed out to the lanes with `want` from an LDS counter, one LDS
// atomic per wave.  Every lane of the wave calls.
__device__ __forceinline__ int lds_append(bool want, int *counter) {
    const int lane = threadIdx.x & 63;
    const uint64_t m = __ballot(want);
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(counter, __popcll(m));
    base = __shfl(base, 0);
    return base + __popcll(m & ((1ull << lane) - 1ull));
}
__device__ __forceinline__ void lds_count(bool want, int *counter) {
    const uint64_t m = __ballot(want);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(counter, __popcll(m));
}

// Marks ids [lo, hi) of `keys` (rows of tb) in the bitmap; false in a thread
// that met a row out of range (which is not marked).
template <int NB>
__device__ __forceinline__ bool mark_ids(LdsBitmap<NB> &bm, const DTable &tb, const int32_t *__restrict__ keys,
                                         int64_t lo, int64_t hi) {
    constexpr int Q = 4;
    const int64_t rows = tb.rows;
    const int32_t ns = tb.nsets, qb = tb.qbits;
    bool ok = true;
    for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += Q * kSmallThreads) {
        int32_t r[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) r[q] = i0 + q * kSmallThreads < hi ? keys[i0 + q * kSmallThreads] : 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (i0 + q * kSmallThreads >= hi) continue;
            if (r[q] < 0 || (int64_t)r[q] >= rows) ok = false;
            else bm.set(bm_pos(ns, qb, r[q]));
        }
    }
    return ok;
}

// Everything of a forward before its miss fetch, for one table per block:
// bag offsets checked, distinct rows (U, rank words), cache probe, per-index
// location, prefetch coverage.  Same results as k_fwd_prep,
// k_mark_own, k_bm_*, k_fwd_probe and k_fwd_src.  A table whose
// offsets or ids are malformed raises the error word and stops; nothing is
// published for any table then (the later kernels read the word).
template <int NB>
__global__ void __launch_bounds__(kSmallThreads) k_fwd_small(DGlobal g, const int32_t *__restrict__ indices,
                                                             const int64_t *__restrict__ offsets, int32_t B, int64_t n,
                                                             int32_t stamp, int cover) {
    __shared__ LdsBitmap<NB> bm;
    __shared__ int tmp[16];
    __shared__ int s_err, s_bad_off, s_bad_id, s_hits, s_pf, s_miss, s_cov;
    __shared__ int32_t s_slot[kLdsSlots];
    const int t = blockIdx.x;
    const DTable tb = g.tabs[t];  // a copy: read through a reference its fields would be reloaded after every store
    TState &st = g.st[t];
    if (threadIdx.x == 0) {
        s_err = *g.err;  // read once: another block may set it meanwhile
        s_bad_off = s_bad_id = s_hits = s_pf = s_miss = s_cov = 0;
    }
    const int nw = tb.bm_words;
    bm.clear(nw);
    __syncthreads();
    if (s_err) return;  // block-uniform
    const int64_t *ob = offsets + (int64_t)t * B;
    const int64_t lo = ob[0], hi = ob[B];
    bool bad = lo < 0 || hi < lo || hi > n || (t == 0 && lo != 0) || (t == g.T - 1 && hi != n);
    const int nb = B <= kPrepBags ? B : 0;  // more: k_bag_offsets
    for (int j = threadIdx.x; j < nb; j += kSmallThreads) bad |= ob[j] > ob[j + 1];
    if (bad) s_bad_off = 1;
    __syncthreads();
    if (s_bad_off) {  // block-uniform
        if (threadIdx.x == 0) atomicOr(g.err, ERR_OFFSETS);
        return;
    }
    if (threadIdx.x == 0) {
        g.tstart[t] = lo;
        if (t == g.T - 1) g.tstart[g.T] = hi;
    }
    if (!mark_ids(bm, tb, indices, lo, hi)) s_bad_id = 1;
    __syncthreads();
    if (s_bad_id) {
        if (threadIdx.x == 0) atomicOr(g.err, ERR_RANGE);
        return;
    }
    const int nu = bm.scan(nw, tmp);
    int32_t *U = g.U + lo;
    bm.each_word(nw, [&](int w, uint32_t bits, int u) {
        tb.rank[w] = make_uint4((uint32_t)u, bits, (uint32_t)stamp, 0u);
        while (bits) {
            const int b = __ffs(bits) - 1;
            bits &= bits - 1;
            U[u++] = bm_row(tb, (uint32_t)(w * 32 + b));
        }
    });
    __syncthreads();
    // cache probe of the distinct rows, kProbe per thread in flight
    constexpr int kProbe = 4;
    for (int u0 = 0; u0 < nu; u0 += kProbe * kSmallThreads) {  // block-uniform
        int32_t row[kProbe], slot[kProbe];
        bool in[kProbe];
#pragma unroll
        for (int q = 0; q < kProbe; ++q) {
            const int u = u0 + q * kSmallThreads + (int)threadIdx.x;
            in[q] = u < nu;
            row[q] = in[q] ? U[u] : 0;
        }
        if (tb.ways) {
#pragma unroll
            for (int q = 0; q < kProbe; ++q) slot[q] = in[q] ? set_find_wide(tb, row[q]) : -1;
        } else {
            map_find_n<kProbe>(tb, row, in, slot);
        }
        uint32_t fl[kProbe];
#pragma unroll
        for (int q = 0; q < kProbe; ++q) fl[q] = in[q] && slot[q] >= 0 ? gload4(tb.slot_flags + slot[q]) : 0u;
#pragma unroll
        for (int q = 0; q < kProbe; ++q) {
            const int u = u0 + q * kSmallThreads + (int)threadIdx.x;
            const bool hit = in[q] && slot[q] >= 0, miss = in[q] && slot[q] < 0;
            if (u0 + q * kSmallThreads >= nu) break;  // block-uniform
            if (hit) tb.slot_touch[slot[q]] = stamp;
            lds_count(hit, &s_hits);
            lds_count(hit && (fl[q] & F_PF), &s_pf);
            const int m = lds_append(miss, &s_miss);
            const int32_t sl = hit ? slot[q] : -(m + 1);
            if (in[q]) {
                g.slotU[lo + u] = sl;
                if (u < kLdsSlots) s_slot[u] = sl;
            }
            if (miss) {
                g.M[lo + m] = row[q];
                g.mflags[lo + m] = 0;
                g.mcbit[lo + m] = 0;
            }
        }
    }
    __syncthreads();
    // location of every index
    const int32_t ns = tb.nsets, qb = tb.qbits;
    constexpr int kSrc = 4;
    for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kSrc * kSmallThreads) {
        int32_t r[kSrc], sl[kSrc];
#pragma unroll
        for (int q = 0; q < kSrc; ++q) r[q] = i0 + q * kSmallThreads < hi ? indices[i0 + q * kSmallThreads] : -1;
#pragma unroll
        for (int q = 0; q < kSrc; ++q) {
            const int u = r[q] >= 0 ? bm.rank(bm_pos(ns, qb, r[q])) : 0;
            sl[q] = u < kLdsSlots ? s_slot[u] : g.slotU[lo + u];
        }
#pragma unroll
        for (int q = 0; q < kSrc; ++q) {
            if (r[q] < 0) continue;  // past the table's end (every id was checked above)
            const int64_t i = i0 + q * kSmallThreads;
            g.src[i] = sl[q];
        }
    }
    if (cover) {  // distinct rows of the last placement's list that the batch touches
        const int64_t ps = g.pstart[t];
        const int pc = st.pcount;
        for (int i = threadIdx.x; i - (int)threadIdx.x < pc; i += kSmallThreads)
            lds_count(i < pc && bm.test(bm_pos(ns, qb, i < pc ? g.PU[ps + i] : 0)), &s_cov);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st.ucount = nu;
        st.mcount = s_miss;
        st.hits = s_hits;
        st.hits_pf = s_pf;
        st.covered = s_cov;
    }
}

// ----------------------------------------------------------------- placement

// Block totals of a count held per thread, one LDS atomic per wave.
__device__ __forceinline__ void lds_sum(int v, int *counter) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(counter, v);
}

// Whether every id of a list lies in its table, whose first ids s_po gives: a
// wave takes a contiguous share, its lanes neighbouring ids.  The loads of the
// first kCheck of a thread's ids may be issued well before they are looked at.
constexpr int kCheck = 8;
struct IdCheck {
    int64_t lo, hi;
    uint32_t r[kCheck];
    __device__ void load(const int32_t *__restrict__ keys, int64_t i0) {
#pragma unroll
        for (int q = 0; q < kCheck; ++q) r[q] = i0 + q * 64 < hi ? (uint32_t)keys[i0 + q * 64] : 0u;
    }
    __device__ void start(const int32_t *__restrict__ keys, int64_t n) {
        const int64_t per = ((n + kSmallThreads - 1) / kSmallThreads) * 64;
        lo = ((int64_t)threadIdx.x >> 6) * per;
        hi = lo + per < n ? lo + per : n;
        lo += threadIdx.x & 63;
        load(keys, lo);
    }
    // true in every thread that met no bad id
    __device__ bool finish(const int32_t *__restrict__ keys, int T, const int64_t *s_po, const uint32_t *s_rows) {
        if (lo >= hi) return true;
        int t = find_seg(s_po, T, lo);
        bool ok = true;
        for (int64_t i0 = lo;;) {
#pragma unroll
            for (int q = 0; q < kCheck; ++q) {
                if (i0 + q * 64 >= hi) continue;
                while (i0 + q * 64 >= s_po[t + 1]) ++t;
                ok &= r[q] < s_rows[t];  // negative ids too
            }
            i0 += kCheck * 64;
            if (i0 >= hi) return ok;
            load(keys, i0);
        }
    }
};

// Everything of a placement but the sets of set-associative tables, the fill
// and the published counters, for one table per block.  Same results as the
// general sequence (placement.hip, ring.hip, k_sa_heads); what k_plc_end reads
// from the table's state is written once, by thread 0, at the end.
// Every block checks the whole list, its other tables' ids too (at most some ten
// thousand, read beside its own), before it changes anything: no launch comes
// between the check and the change, so a block that looked at its own table alone
// would change the cache in a call that another table's ids make void.
//   all tables   list offsets checked, caching bits or batch counts of the last
//                batch, set(P) sorted (PU)
//   set-assoc.   each set's event segments and the prefetch rows' staging rows
//                (then k_sa_place plays the sets)
//   others       classification of PU; ranking: the radix select of rank_block,
//                or the resident ring's cut; eviction; admission; the ring's run
//                and pending list
// The ring's zone Z1 (keys of the touch score in row order) comes from the same
// kind of LDS bitmap as the dedup: its rows are marked, and a row's place is its
// rank.  So Z1 has no holes here, and no row is searched for in the other list.
// P's bitmap answers whether a row is named, so no slot or miss is flagged.
// What bounds it is the one CU's rate of scattered accesses (some 10 ns each),
// so each step makes as few per row as it can.
template <int NB>
__global__ void __launch_bounds__(kSmallThreads) k_plc_small(DGlobal g, PlcParams p, const int32_t *__restrict__ rows,
                                                             const int64_t *__restrict__ poff, int64_t np,
                                                             const uint8_t *__restrict__ bits, int wr) {
    enum { C_PRES, C_NP, C_STALE, C_EV, C_RING_EV, C_POP, C_ADM, C_PDROP, C_REUSE, C_RUN, C_KEEP, C_N };
    __shared__ LdsBitmap<NB> bm, bz;  // the rows of P; the rows of Z1 (or the ranking's histogram)
    __shared__ int tmp[16];
    constexpr int Q = 4;  // items per thread whose loads are in flight together
    __shared__ int s_c[C_N], s_ch[Q];
    __shared__ int s_err, s_bad_id;
    __shared__ unsigned long long s_dig;
    __shared__ int64_t s_po[RECMG_MAX_TABLES + 1];
    __shared__ uint32_t s_rows[RECMG_MAX_TABLES];
    static_assert(sizeof(bz.w4) >= kRadix * sizeof(int), "the ranking's histogram takes a bitmap's place");
    const int t = blockIdx.x, tid = threadIdx.x;
    const DTable tb = g.tabs[t];
    TState &st = g.st[t];
    if (tid == 0) {
        s_err = *g.err;  // read once: another block may set it meanwhile
        s_bad_id = 0;
        s_dig = 0;
        s_po[g.T] = np;
    }
    if (tid < g.T) {
        s_po[tid] = poff[tid];
        s_rows[tid] = (uint32_t)g.tabs[tid].rows;
    }
    if (tid < C_N) s_c[tid] = 0;
    if (tid < Q) s_ch[tid] = 0;
    const int nw = tb.bm_words;
    bm.clear(nw);
    const int64_t lo = poff[t], hi = poff[t + 1];
    const bool bad_off = list_malformed(g, poff, np);
    __syncthreads();
    if (s_err) return;  // block-uniform
    if (bad_off) {      // block-uniform
        if (tid == 0) atomicOr(g.err, ERR_OFFSETS);
        return;
    }
    // what the last batch brings (a thread's first Q of it) is read beside the
    // ids, and applied once they are known to be good
    const int64_t ts = g.tstart[t], te = g.tstart[t + 1], fts = p.have_fwd ? ts : 0;
    const int32_t nu = p.have_fwd ? st.ucount : 0, nm = p.have_fwd ? st.mcount : 0;
    const int32_t n_res = st.n_res;
    const bool reb = st.rebuild_next != 0, or_bits = p.prio && bits && p.have_fwd;
    int32_t lv[Q], lw[Q];  // PRIORITY: caching bit, location; LFU_BATCH: row, its count
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = ts + q * kSmallThreads + tid;
        lv[q] = lw[q] = 0;
        if (or_bits && i < te) lv[q] = bits[i], lw[q] = (int32_t)gload4(g.src + i);
        if (p.lfu && i - ts < nu) lv[q] = (int32_t)gload4(g.U + i);
    }
    IdCheck check;
    if (g.T > 1) check.start(rows, np);
    if (p.lfu)
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q * kSmallThreads + tid < nu) lw[q] = (int32_t)gload4(tb.freq + lv[q]);
    if (!mark_ids(bm, tb, rows, lo, hi)) s_bad_id = 1;
    if (g.T > 1 && !check.finish(rows, g.T, s_po, s_rows)) s_bad_id = 1;
    __syncthreads();
    if (s_bad_id) {  // block-uniform
        if (tid == 0) atomicOr(g.err, ERR_RANGE);
        return;
    }
    if (tid == 0) {
        g.pstart[t] = lo;
        g.ftstart[t] = fts;
        if (t == g.T - 1) {
            g.pstart[g.T] = hi;
            g.ftstart[g.T] = p.have_fwd ? te : 0;
        }
    }
    if (or_bits) {
        // OR of the caching bits per row; every writer stores the same value
        auto set_bit = [&](int32_t s) {
            uint8_t *f = s >= 0 ? tb.slot_cbit + s : g.mcbit + ts + (-(int64_t)s - 1);
            if (!*f) *f = 1;
        };
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lv[q]) set_bit(lw[q]);
        for (int64_t i = ts + Q * kSmallThreads + tid; i < te; i += kSmallThreads)
            if (bits[i]) set_bit(g.src[i]);
    }
    if (p.lfu) {  // distinct rows
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (q * kSmallThreads + tid < nu) tb.freq[lv[q]] = lw[q] + 1;
        for (int32_t u = Q * kSmallThreads + tid; u < nu; u += kSmallThreads) tb.freq[g.U[ts + u]] += 1;
    }
    const int32_t pc = bm.scan(nw, tmp);
    int32_t *PU = g.PU + lo;
    bm.each_word(nw, [&](int w, uint32_t b, int u) {
        while (b) {
            const int k = __ffs(b) - 1;
            b &= b - 1;
            PU[u++] = bm_row(tb, (uint32_t)(w * 32 + k));
        }
    });
    __syncthreads();
    // place of a row among the last batch's distinct rows, or -1 (its rank word
    // carries the batch's stamp and the row's bit)
    auto in_batch = [&](uint4 rk, uint32_t pos) -> int32_t {
        const uint32_t bit = 1u << (pos & 31);
        return (int32_t)rk.z == p.last_stamp && (rk.y & bit) ? (int32_t)rk.x + __popc(rk.y & (bit - 1u)) : -1;
    };
    if (tb.ways) {  // block-uniform
        const uint32_t ns = (uint32_t)tb.nsets;
        int *seg = reinterpret_cast<int *>(tb.seg);
        auto bounds = [&](const int32_t *list, int32_t n, int32_t k, int field) {
            const uint32_t set = (uint32_t)list[k] % ns;
            if (k == 0 || (uint32_t)list[k - 1] % ns != set) seg[4 * (int64_t)set + field] = k;
            if (k + 1 == n || (uint32_t)list[k + 1] % ns != set) seg[4 * (int64_t)set + field + 1] = k + 1;
        };
        for (int32_t u = tid; u < nu; u += kSmallThreads) bounds(g.U + ts, nu, u, 0);
        for (int32_t i = tid; i < pc; i += kSmallThreads) {
            bounds(PU, pc, i, 2);
            int32_t from = -1;  // its staging row if the last batch missed it
            if (p.have_fwd) {
                const uint32_t pos = bm_pos(tb, PU[i]);
                const int32_t u = in_batch(gload16(tb.rank + (pos >> 5)), pos);
                const int32_t su = u >= 0 ? g.slotU[ts + u] : 0;
                if (su < 0) from = -su - 1;
            }
            g.pfrom[lo + i] = from;
        }
        if (tid == 0) {
            st.pcount = pc;
            st.npcount = st.popped = st.p_res = st.evicted = st.adm_miss = st.p_fill = st.p_drop = st.m_drop = 0;
            st.rebuild = 0;
            st.digest_acc = st.digest;
        }
        return;
    }
    // ---- classification of the prefetch rows: resident, missed, or new
    for (int32_t u0 = 0; u0 < pc; u0 += Q * kSmallThreads) {  // block-uniform
        int32_t row[Q], slot[Q];
        uint4 rk[Q];
        bool in[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t u = u0 + q * kSmallThreads + tid;
            in[q] = u < pc;
            row[q] = in[q] ? PU[u] : 0;
        }
        map_find_n<Q>(tb, row, in, slot);
#pragma unroll
        for (int q = 0; q < Q; ++q)
            rk[q] = in[q] && slot[q] < 0 ? gload16(tb.rank + ((uint32_t)row[q] >> 5)) : make_uint4(0u, 0u, ~0u, 0u);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (u0 + q * kSmallThreads >= pc) break;  // block-uniform
            const int32_t u = u0 + q * kSmallThreads + tid;
            const bool res = in[q] && slot[q] >= 0;
            bool fresh = false;
            int32_t ref = slot[q];
            if (!res && in[q]) {
                const int32_t k = p.have_fwd ? in_batch(rk[q], (uint32_t)row[q]) : -1;
                if (k >= 0) {
                    ref = ring_ref_miss(-g.slotU[ts + k] - 1);
                } else {
                    fresh = true;
                }
            }
            lds_count(res, &s_c[C_PRES]);
            const int k = lds_append(fresh, &s_c[C_NP]);
            if (fresh) {
                g.NP[lo + k] = row[q];
                ref = ring_ref_new(k);
            }
            if (in[q]) g.puref[lo + u] = ref;
        }
    }
    __syncthreads();
    Counts c;
    c.cap = tb.cap;
    c.nm = nm;
    c.nnp = s_c[C_NP];
    const int64_t nk = (int64_t)n_res + c.nm + c.nnp;
    c.keep = (int32_t)(nk < c.cap ? nk : c.cap);
    c.mode = nk <= c.cap ? SEL_ALL : (c.keep == 0 ? SEL_NONE : SEL_SELECT);
    const int32_t top0 = st.free_top;
    const bool ring = tb.ring_cap != 0;
    if (reb) map_clear_share(tb, 0, 1);  // no lookup follows; k_plc_end inserts every resident
    unsigned long long dig = 0;  // this thread's share of the digest (ring: of its change)
    // frees Q slots sl of rows r (where ev); every lane of the wave calls.  Their
    // rows and flags are cleared after admission, if no admitted row takes the slot.
    auto evict = [&](const bool (&ev)[Q], const int32_t (&sl)[Q], const int32_t (&r)[Q]) {
        if (!reb) map_delete_n<Q>(tb, r, ev);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int at = top0 + lds_append(ev[q], &s_c[C_EV]);
            if (!ev[q]) continue;
            if (at < tb.cap) tb.free_stack[at] = sl[q];
            else atomicOr(g.err, ERR_INTERNAL);
        }
    };
    auto named = [&](int32_t r, uint32_t) { return bm.test((uint32_t)r); };  // r in P
    int32_t mode = c.mode;
    uint64_t thr = 0;
    RingCut cut{};
    int32_t z1 = 0;
    int2 *z = nullptr;
    if (!ring) {
        // ---- scores of every slot and candidate, the threshold, eviction
        thr = rank_block(g, p, tb, c, t, reinterpret_cast<int *>(bz.w4), tmp, named);
        const int32_t ngrp = (tb.cap + 3) / 4;
        for (int32_t q0 = 0; q0 < ngrp; q0 += kSmallThreads) {  // block-uniform
            const int32_t k0 = 4 * (q0 + tid), lim = q0 + tid < ngrp ? tb.cap : 0;
            int32_t row[4], sc[4];
            slot_quad(tb.slot_row, k0, lim, -1, row);
            slot_quad(tb.slot_score, k0, lim, 0, sc);
            bool ev[Q];
            int32_t sl[Q];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool live = row[i] >= 0;
                const bool keep = live && kept(mode, make_key(sc[i], row[i], p.rowbits), thr);
                if (keep) dig += mix64(((unsigned long long)t << 40) | (unsigned long long)row[i]);
                ev[i] = live && !keep;
                sl[i] = k0 + i;
            }
            evict(ev, sl, row);
        }
        __syncthreads();
    } else {
        // ---- new scores of the touched and named rows, Z1
        const int32_t pn = st.pend_n;
        const bool pb = st.pend_buf != 0, rb = st.r_buf != 0;
        const int32_t *prow = (pb ? g.pend_row[1] : g.pend_row[0]) + st.pend_off;
        const int32_t *pslot = (pb ? g.pend_slot[1] : g.pend_slot[0]) + st.pend_off;
        const int32_t *urow = g.U + ts;
        int32_t *rcnt = rb ? tb.rcnt[1] : tb.rcnt[0], *rcnt2 = rb ? tb.rcnt[0] : tb.rcnt[1];
        z = ring_zone(g, st, t);
        bz.clear(nw);
        __syncthreads();
        int stale = 0;
        // the ring entries e of slots sl, whose scores change, go stale (-1: none);
        // every lane of the wave calls
        auto unring = [&](const int32_t (&sl)[Q], const int32_t (&e)[Q]) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (e[q] >= 0) {
                    tb.slot_pos[sl[q]] = -1;
                    ++stale;
                }
                chunk_sub(e[q] >= 0, e[q] / kRingChunk, rcnt);
            }
        };
        // pending rows neither touched nor named again
        for (int32_t j = tid; j < pn; j += kSmallThreads) {
            const int32_t q = pslot[j], r = prow[j];
            if (q >= 0 && q < tb.cap && !named(r, 0) && tb.slot_touch[q] != p.last_stamp) bz.set((uint32_t)r);
        }
        for (int32_t u0 = 0; u0 < nu; u0 += Q * kSmallThreads) {  // block-uniform
            int32_t h[Q], e[Q];
            uint32_t f[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int32_t u = u0 + q * kSmallThreads + tid;
                h[q] = u < nu ? (int32_t)gload4(g.slotU + ts + u) : -1;
                if (u < nu) {
                    const int32_t r = (int32_t)gload4(urow + u);
                    if (!named(r, 0)) bz.set((uint32_t)r);
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                f[q] = h[q] >= 0 ? gload4(tb.slot_flags + h[q]) : 0u;
                e[q] = h[q] >= 0 ? (int32_t)gload4(tb.slot_pos + h[q]) : -1;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (f[q] & F_PF) tb.slot_flags[h[q]] = f[q] & ~F_PF;
            unring(h, e);
        }
        for (int32_t i0 = 0; i0 < pc; i0 += Q * kSmallThreads) {  // block-uniform
            int32_t v[Q], e[Q], tch[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int32_t i = i0 + q * kSmallThreads + tid;
                v[q] = i < pc ? (int32_t)gload4(g.puref + lo + i) : -1;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                tch[q] = v[q] >= 0 ? (int32_t)gload4(tb.slot_touch + v[q]) : 0;
                e[q] = v[q] >= 0 ? (int32_t)gload4(tb.slot_pos + v[q]) : -1;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (tch[q] == p.last_stamp) e[q] = -1;  // touched: done above
            unring(v, e);
        }
        lds_sum(stale, &s_c[C_STALE]);
        __syncthreads();
        z1 = bz.scan(nw, tmp);
        // a pending row the batch touched has the batch's entry, of the same slot
        for (int32_t j = tid; j < pn; j += kSmallThreads) {
            const int32_t q = pslot[j], r = prow[j];
            if (q >= 0 && q < tb.cap && bz.test((uint32_t)r)) z[bz.rank((uint32_t)r)] = make_int2(q, r);
        }
        for (int32_t u = tid; u < nu; u += kSmallThreads) {
            const int32_t r = urow[u], h = g.slotU[ts + u];
            if (bz.test((uint32_t)r)) z[bz.rank((uint32_t)r)] = make_int2(h >= 0 ? h : ring_ref_miss(-h - 1), r);
        }
        __syncthreads();
        // ---- the cut, eviction from the ring's front, compaction
        cut = ring_cut(g, p, t, tb, st, c, st.r_valid - s_c[C_STALE], z1, z1, pc, tmp);
        if (cut.bad) {  // block-uniform; never expected
            if (tid == 0) atomicOr(g.err, ERR_INTERNAL);
            return;
        }
        mode = cut.mode;
        thr = cut.thr;
        const int32_t tail = st.r_tail, head = st.r_head;
        const int32_t *ringb = rb ? tb.ring[1] : tb.ring[0];
        int32_t *dst = rb ? tb.ring[0] : tb.ring[1];
        const int32_t hi_ch = cut.compact && cut.moved > 0 ? (int32_t)(((int64_t)head + kRingChunk - 1) / kRingChunk)
                              : cut.cut > tail             ? (cut.cut - 1) / kRingChunk + 1
                                                           : 0;
        int32_t run = 0;  // entries moved so far
        // Q chunks at a time, their loads in flight together
        for (int32_t ch = tail / kRingChunk; ch < hi_ch; ch += Q) {
            int32_t sl[Q], r[Q], pos[Q];
            bool ev[Q], mv[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) sl[q] = ch + q < hi_ch ? (int32_t)gload4(ringb + (ch + q) * kRingChunk + tid) : -1;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const bool ok = sl[q] >= 0 && sl[q] < tb.cap;
                pos[q] = ok ? (int32_t)gload4(tb.slot_pos + sl[q]) : -1;
                r[q] = ok ? (int32_t)gload4(tb.slot_row + sl[q]) : 0;
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int32_t e = (ch + q) * kRingChunk + tid;
                const bool live = e >= tail && e < head && pos[q] == e;
                ev[q] = live && e < cut.cut;
                mv[q] = live && !ev[q] && cut.compact;
                if (ev[q]) {
                    tb.slot_pos[sl[q]] = -1;
                    dig -= mix64(((unsigned long long)t << 40) | (unsigned long long)(uint32_t)r[q]);
                }
                lds_count(ev[q], &s_ch[q]);
            }
            evict(ev, sl, r);
            if (cut.compact) {  // block-uniform
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    int tot;
                    const int at = run + block_excl_scan(mv[q] ? 1 : 0, tmp, &tot);
                    if (mv[q]) {
                        if (at < cut.moved) dst[at] = sl[q];
                        else atomicOr(g.err, ERR_INTERNAL);  // counts and entries disagree (never expected)
                    }
                    run += tot;
                }
            }
            __syncthreads();
            if (tid < Q && s_ch[tid]) {
                rcnt[ch + tid] -= s_ch[tid];
                atomicAdd(&s_c[C_RING_EV], s_ch[tid]);
                s_ch[tid] = 0;
            }
            __syncthreads();
        }
        if (cut.zev) {  // Z1 and Z2 residents below the threshold
            const int32_t n = z1 + pc;
            for (int32_t b0 = 0; b0 < n; b0 += Q * kSmallThreads) {  // block-uniform
                int32_t sl[Q], r[Q];
                bool ev[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int32_t k = b0 + q * kSmallThreads + tid;
                    sl[q] = -1, r[q] = 0;
                    if (k < z1) {
                        const int2 zr = z[k];
                        r[q] = zr.y;
                        if (zr.x >= 0 && !kept(mode, make_key(p.lru_touch, zr.y, p.rowbits), thr)) sl[q] = zr.x;
                    } else if (k < n) {
                        const int32_t v = g.puref[lo + (k - z1)];
                        r[q] = PU[k - z1];
                        if (v >= 0 && !kept(mode, make_key(p.pscore, r[q], p.rowbits), thr)) sl[q] = v;
                    }
                    ev[q] = sl[q] >= 0;
                    if (ev[q]) {
                        tb.slot_pos[sl[q]] = -1;
                        dig -= mix64(((unsigned long long)t << 40) | (unsigned long long)(uint32_t)r[q]);
                    }
                }
                evict(ev, sl, r);
            }
        }
        __syncthreads();
        if (cut.compact) {  // moved slots learn their new index once no entry is tested any more
            for (int32_t k = tid; k < cut.moved; k += kSmallThreads) {
                const int32_t sl = dst[k];
                if (sl >= 0 && sl < tb.cap) tb.slot_pos[sl] = k;
                else atomicOr(g.err, ERR_INTERNAL);
            }
            for (int32_t ch = tid; ch < tb.ring_cap / kRingChunk; ch += kSmallThreads) {
                const int64_t left = (int64_t)cut.moved - (int64_t)ch * kRingChunk;
                rcnt2[ch] = left <= 0 ? 0 : left >= kRingChunk ? kRingChunk : (int32_t)left;
            }
            __syncthreads();
        }
    }
    // ---- admission
    const int32_t nev = s_c[C_EV], top = top0 + nev;
    const int32_t items = c.nm + c.nnp;
    int n_adm = 0, n_pdrop = 0, n_reuse = 0;
    for (int32_t b0 = 0; b0 < items; b0 += Q * kSmallThreads) {  // block-uniform
        int32_t row[Q], sc[Q], slot[Q], at[Q];
        bool adm[Q], inp[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t k = b0 + q * kSmallThreads + tid;
            row[q] = sc[q] = 0;
            if (k < c.nm) {
                row[q] = (int32_t)gload4(g.M + ts + k);
                if (!ring) sc[q] = (int32_t)gload4(g.mscore + ts + k);
            } else if (k < items) {
                row[q] = (int32_t)gload4(g.NP + lo + (k - c.nm));
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t k = b0 + q * kSmallThreads + tid;
            inp[q] = k >= c.nm || named(row[q], 0);
            if (k >= c.nm) sc[q] = k < items ? new_prefetch_score(p, tb, row[q]) : 0;
            else if (ring) sc[q] = inp[q] ? p.pscore : p.lru_touch;
            adm[q] = k < items && kept(mode, make_key(sc[q], row[q], p.rowbits), thr);
            at[q] = lds_append(adm[q], &s_c[C_POP]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t fi = top - 1 - at[q];
            const int64_t fj = fts + lo + at[q];  // this row's entry in the fill list
            slot[q] = adm[q] && fi >= 0 && fi < tb.cap && fj >= 0 && fj < g.fill_cap ? (int32_t)gload4(tb.free_stack + fi) : -1;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int32_t k = b0 + q * kSmallThreads + tid;
            const bool is_miss = k < c.nm;
            if (adm[q] && (uint32_t)slot[q] >= (uint32_t)tb.cap) {
                atomicOr(g.err, ERR_INTERNAL);
                adm[q] = false;
            }
            if (!adm[q]) {
                n_pdrop += k < items && inp[q] ? 1 : 0;
                continue;
            }
            // (the slot's touch stamp, of a forward before this placement, is older
            // than any a later placement asks for)
            tb.slot_row[slot[q]] = row[q];
            if (!ring) tb.slot_score[slot[q]] = sc[q];
            tb.slot_flags[slot[q]] = inp[q] ? F_PF : 0u;
            const int64_t fj = fts + lo + at[q];
            g.fill_src[fj] = is_miss ? k : -(row[q] + 1);
            g.fill_slot[fj] = slot[q];
            if (ring) {
                if (is_miss) g.mslot[ts + k] = slot[q];
                else g.npslot[lo + (k - c.nm)] = slot[q];
            }
            dig += mix64(((unsigned long long)t << 40) | (unsigned long long)row[q]);
            n_adm += is_miss ? 1 : 0;
        }
        if (!reb) n_reuse += map_insert_n<Q>(tb, row, slot, adm);
    }
    lds_sum(n_adm, &s_c[C_ADM]);
    lds_sum(n_pdrop, &s_c[C_PDROP]);
    lds_sum(n_reuse, &s_c[C_REUSE]);
    dig = wave_sum64(dig);
    if ((tid & 63) == 0 && dig) atomicAdd(&s_dig, dig);
    __syncthreads();
    for (int32_t j = top0 + tid; j < top - s_c[C_POP]; j += kSmallThreads) {  // freed and not taken again
        const int32_t sl = tb.free_stack[j];
        tb.slot_row[sl] = -1;
        tb.slot_flags[sl] = 0;
    }
    // ---- the ring's new run and pending list
    if (ring) {
        const bool buf1 = (st.r_buf != 0) != cut.compact;
        const int32_t head = cut.compact ? cut.moved : st.r_head;
        int32_t *ringb = buf1 ? tb.ring[1] : tb.ring[0], *rcnt = buf1 ? tb.rcnt[1] : tb.rcnt[0];
        if ((int64_t)head + z1 > tb.ring_cap) {  // block-uniform; compaction made room, never expected
            if (tid == 0) atomicOr(g.err, ERR_INTERNAL);
            return;
        }
        for (int32_t j0 = 0; j0 < z1; j0 += kSmallThreads) {  // block-uniform
            const int32_t j = j0 + tid, e = head + j;
            int32_t sl = kRingHole;
            if (j < z1) {
                const int2 zr = z[j];
                if (kept(mode, make_key(p.lru_touch, zr.y, p.rowbits), thr)) sl = zr.x >= 0 ? zr.x : g.mslot[ts + (-1 - zr.x)];
                if (sl != kRingHole && (sl < 0 || sl >= tb.cap)) {
                    atomicOr(g.err, ERR_INTERNAL);
                    sl = kRingHole;
                }
                ringb[e] = sl;
                if (sl != kRingHole) tb.slot_pos[sl] = e;
            }
            const bool live = sl != kRingHole;
            lds_count(live, &s_c[C_RUN]);
            // live entries of the wave's two chunks at most
            const int32_t c0 = __builtin_amdgcn_readfirstlane(e) / kRingChunk;
            const uint64_t m0 = __ballot(live && e / kRingChunk == c0), m1 = __ballot(live && e / kRingChunk != c0);
            if ((tid & 63) == 0) {
                if (m0) atomicAdd(&rcnt[c0], (int)__popcll(m0));
                if (m1) atomicAdd(&rcnt[c0 + 1], (int)__popcll(m1));
            }
        }
        int32_t *nrow = (wr ? g.pend_row[1] : g.pend_row[0]) + lo, *nslot = (wr ? g.pend_slot[1] : g.pend_slot[0]) + lo;
        int keepn = 0;
        for (int32_t i = tid; i < pc; i += kSmallThreads) {
            const int32_t row = PU[i], v = g.puref[lo + i];
            int32_t sl = -1;
            if (kept(mode, make_key(p.pscore, row, p.rowbits), thr)) {
                if (v >= 0) {
                    sl = v;
                } else {
                    sl = v > kRingNewBase ? g.mslot[ts + (-1 - v)] : g.npslot[lo + (kRingNewBase - v)];
                }
            }
            nrow[i] = row;
            nslot[i] = sl;
            keepn += sl >= 0 ? 1 : 0;
        }
        lds_sum(keepn, &s_c[C_KEEP]);
        __syncthreads();
    }
    if (tid == 0) {
        st.pcount = pc;
        st.npcount = c.nnp;
        st.popped = s_c[C_POP];
        st.p_res = s_c[C_PRES];
        st.adm_miss = s_c[C_ADM];
        st.p_drop = s_c[C_PDROP];
        st.plc_nm = nm;
        st.free0 = top0;
        st.free_top = top;
        st.rebuild = reb ? 1 : 0;
        st.reused = s_c[C_REUSE];
        st.digest_acc = (ring ? st.digest : 0ull) + s_dig;
        if (ring) {
            st.touched = (uint32_t)s_c[C_STALE];
            st.z_evicted = nev - s_c[C_RING_EV];
            st.appended = ((unsigned long long)s_c[C_RUN] << 32) | (uint32_t)s_c[C_KEEP];
            st.r_cut = cut.cut;
            st.r_compact = cut.compact ? 1 : 0;
            st.r_moved = cut.moved;
            st.z1_len = z1;
            st.pend_buf = wr;
        }
    }
}

// ----------------------------------------------------------------- launchers

constexpr int kSmallBlocksLow = 8, kSmallBlocksHigh = kOwnSliceBlocks;  // bitmap blocks: 32 and 128 KiB of LDS
constexpr int kSmallBlocksPlc = 16;  // a placement's two bitmaps

// Where one block per table is the faster form.  It saves the launches of three
// kernels, 6 to 8 us per forward, and pays for doing a table's work on one CU.
// Forwards of Zipf-distributed ids, 64 fp32 values per row, here and in the
// general sequence:
//   100,000 rows, 1 table: 2,000 ids 21 and 27 us, 4,000 28 and 29, 6,000 34 and 32,
//     8,000 40 and 35
//   100,000 rows, 8 tables: 2,000 each 25 and 31, 3,000 37 and 42, 4,000 49 and 51
//   500,000 rows, 1 table: 1,000 24 and 27, 3,000 28 and 28, 6,000 34 and 28
//   20,000 rows, 26 tables: 1,000 each 39 and 46
// So one table crosses at some 4,500 ids (3,000 with 16 bitmap blocks) and the line
// below lies past it, at a cost of up to 6 us: it was drawn when the general
// sequence took longer.  The host knows only the mean of the tables' ids, and one table may hold nearly
// all of them: the bound on the total keeps that case's loss to some 30 us.
#ifndef RECMG_SMALL_MAX
#define RECMG_SMALL_MAX 32768
#endif
bool small_batch(int32_t T, int64_t n, int32_t max_nblk) {
    return max_nblk <= kSmallBlocksHigh && n <= RECMG_SMALL_MAX && 7 * n <= (75000 - 2000 * (int64_t)max_nblk) * T;
}

void launch_fwd_small(const DGlobal &g, const int32_t *indices, const int64_t *offsets, int32_t B, int64_t n,
                      int32_t stamp, bool cover, int32_t max_nblk, hipStream_t s) {
    if (max_nblk <= kSmallBlocksLow)
        k_fwd_small<kSmallBlocksLow><<<g.T, kSmallThreads, 0, s>>>(g, indices, offsets, B, n, stamp, cover ? 1 : 0);
    else
        k_fwd_small<kSmallBlocksHigh><<<g.T, kSmallThreads, 0, s>>>(g, indices, offsets, B, n, stamp, cover ? 1 : 0);
}

// The same for a placement, by the mean of its two lists (the last batch's ids,
// the prefetch ids).  It saves six to nine launches, 40 .. 60 us.  A table's rows
// cost its CU more here than in a forward, so the total that bounds the loss of a
// batch with nearly all ids in one table is half as large; tables with more slots
// than one block ranks take the general sequence too.  What a row costs goes by
// its new slot, map entry and ring entry, so it is dear in fully associative
// tables whose rows change at every batch.  Steps of 1 table (40,000 x 64 fp32, half of each
// list of m distinct rows new, as many ids in the batch), here and in the general
// sequence, placements on the forward's stream and on one of their own:
//           LRU                        PRIORITY                   32-way LRU
//   m 2,000  82, 96    122, 136         75, 89    104, 112         70, 82   85, 98
//     5,000  131, 153  132, 157        117, 138   126, 151         94, 110  102, 127
//     6,000  153, 177  140, 165        134, 157   133, 162         99, 117  105, 130
//    10,000  219, 254  161, 169        189, 221   158, 194        126, 147  118, 155
// Zipf-distributed ids repeat (8,000 ids and a list of 3,067: LRU 127, 143 against
// 155, 144).  So LRU and PRIORITY keep to kSmallFaIds per table where one is fully
// associative; sets and LFU_BATCH (10,000: 170, 187 against 187, 201) need no line
// of their own.
#ifndef RECMG_SMALL_PLC_MAX
#define RECMG_SMALL_PLC_MAX (RECMG_SMALL_MAX / 2)
#endif
constexpr int64_t kSmallFaIds = 5500;
bool small_placement(int32_t T, int64_t last_n, int64_t np, int32_t max_nblk, int32_t max_fa_cap, bool dear) {
    const int64_t n = (last_n + np + 1) / 2;
    return last_n + np > 0 && n <= RECMG_SMALL_PLC_MAX && max_nblk <= kSmallBlocksPlc && max_fa_cap <= kRankSmallItems &&
           (!dear || n <= kSmallFaIds * T) && small_batch(T, n, max_nblk);
}

// Where a small placement's last kernel copies the prefetch rows too.  With a copy
// stream that saves a launch and two streams' waits for one another, some 15 us,
// and the next forward's dedup and a placement on a stream of its own wait for the
// rows: worth it up to some 16 MiB of list (a bound of the rows that it brings;
// 300 us of host link).  Without one there is no stream to wait for: a fill apart
// lets the next forward's dedup start where the placement is on another stream,
// and gains nothing where it is not.  Steps with half of each list new, in that
// kernel | apart; in each: on the forward's stream and on one of its own with a copy
// stream, on one of its own without:
//   1 x   300 rows of   64 B (0.02 MiB)  56  67  67     77  68  64
//   4 x 1,000 rows of  256 B (0.98 MiB)  80  92  91    105 119  90
//   1 x 3,000 rows of 1 KiB  (2.9 MiB)  127 142 142    141 134 129
//   3 x 2,000 rows of 1 KiB  (5.9 MiB)  151 166 166    174 190 158
//   4 x 3,000 rows of 1 KiB  (11.7 MiB) 232 247 248    253 276 236
//   1 x 5,000 rows of 4 KiB  (19.5 MiB) 351 358 357    355 377 330
//   3 x 3,000 rows of 4 KiB  (35.2 MiB) 508 511 512    523 431 497
// (apart, a placement on its own stream now and then settles a whole step ahead,
// as in the 431.)
#ifndef RECMG_SMALL_FILL_BYTES
#define RECMG_SMALL_FILL_BYTES (16 << 20)
#endif
bool fill_in_end(int64_t bytes, bool copy_stream, bool own_stream) {
    return copy_stream ? bytes <= RECMG_SMALL_FILL_BYTES : !own_stream;
}

void launch_plc_small(const DGlobal &g, const PlcParams &p, const int32_t *rows, const int64_t *poff, int64_t np,
                      const uint8_t *bits, int wr, int32_t max_nblk, hipStream_t s) {
    if (max_nblk <= kSmallBlocksLow)
        k_plc_small<kSmallBlocksLow><<<g.T, kSmallThreads, 0, s>>>(g, p, rows, poff, np, bits, wr);
    else
        k_plc_small<kSmallBlocksPlc><<<g.T, kSmallThreads, 0, s>>>(g, p, rows, poff, np, bits, wr);
}

}  // namespace recmg

// Batches of few ids per table: one block of 1,024 threads per table does the
// work of several kernels, with barriers of the block between its steps.
//
// What bounds them: a batch of some thousand ids gives every kernel of the
// general sequence a few microseconds of dependent loads and a launch, and
// those add up to the whole call.  The ids of a table meet in one block here,
// so the presence bitmap, its prefix sums and every counter stay in LDS, and
// what passes from step to step costs a barrier instead of a launch.
#include "launch.h"

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
// location and row address, prefetch coverage.  Same results as k_fwd_prep,
// k_mark_own, k_bm_*, k_fwd_probe, k_fwd_src and k_fwd_cover.  A table whose
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
    for (int j = threadIdx.x; j < B; j += kSmallThreads) bad |= ob[j] > ob[j + 1];
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
    // location and address of every index
    const char *pool = tb.pool, *stg = g.staging + lo * g.stage_stride;
    const int64_t rb = tb.row_bytes, ss = g.stage_stride;
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
            g.raddr[i] = (uint64_t)(sl[q] >= 0 ? pool + sl[q] * rb : stg + (-(int64_t)sl[q] - 1) * ss);
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

// ----------------------------------------------------------------- launchers

constexpr int kSmallBlocksLow = 8, kSmallBlocksHigh = kOwnSliceBlocks;  // bitmap blocks: 32 and 128 KiB of LDS

// Where one block per table is the faster form.  It saves the launches of three
// kernels, about 12 us per forward, and pays for doing a table's work on one
// CU: about 1.4 us per 1,000 ids of a table and 0.4 us per bitmap block more
// than the general sequence (1, 8 and 26 tables of 10,000 .. 1,000,000 rows,
// 2,000 .. 64,000 ids each: 8 tables of 100,000 rows take 26.4 against 39.7 us
// at 2,000 ids each, 42.9 against 45.9 at 8,000, 62 against 50 at 16,000).  The
// host knows only the mean of the tables' ids, and one table may hold nearly
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

}  // namespace recmg

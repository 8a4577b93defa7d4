// Per-batch dedup + sort of row ids (a counting sort over the row-id domain).
//
// Each table owns a presence bitmap of ceil(N_t / 32) words in HBM.  A batch
// of ids is deduplicated by setting one bit per id; the distinct ids then come
// out in ascending order by scanning the bitmap: a block-wide popcount gives
// each 1024-word block its count, a per-table scan turns counts into offsets,
// and the emit pass writes every set bit's row at its rank.  For a forward the
// emit also stores, per non-zero word, (rank of its first set bit, the word,
// the forward's stamp), so the rank of any id of the batch is one load plus a
// popcount, and "was row r in the last batch" is one load.  Cost is
// O(ids + N_t / 32) with no comparison passes, which suits ids drawn from a
// bounded domain; the emit clears the bitmap behind it.
//
// Set-associative tables mark row r at bm_pos(r) = (set << qbits) | (r / nsets)
// instead of r, so U and PU come out grouped by set and ascending within each
// set (the order in which a set takes its events); the resident dump keeps
// plain row positions.
//
// Marking.  A table whose bitmap spans at most kOwnMaxSlices slices of
// kOwnSliceWords words is marked in LDS: one block per slice reads all of the
// table's ids, sets the bits that fall in its slice with LDS atomics, then
// stores the slice's non-zero words and the popcount of each of its bitmap
// blocks (so the count pass is not needed).  Its ids cost one 4-byte read per
// slice and the bitmap one write.  Larger tables are marked in HBM: Zipf-popular
// rows make many threads set the same bit, so each block first deduplicates its
// ids in a small LDS hash set and a popular row costs one device atomic per
// block instead of one per occurrence.  A bitmap word there is shared by blocks
// on every XCD, so that atomic (and the load before it) is served past the
// XCD's L2, a cache line per distinct id and block.
#include <algorithm>

#include "launch.h"

namespace recmg {

constexpr int kLdsSet = 2048;  // entries of the per-block LDS set (power of two)
constexpr int kLdsProbes = 8;

__global__ void __launch_bounds__(kBlock) k_mark(DGlobal g, const int32_t *__restrict__ keys,
                                                 const int64_t *__restrict__ starts, int64_t n) {
    // The error word is read once per block: another block of this kernel may
    // set it meanwhile, and the waves of a block must agree before its barriers.
    __shared__ int s_err;
    if (threadIdx.x == 0) s_err = *g.err;
    __shared__ int64_t s_start[RECMG_MAX_TABLES + 1];
    __shared__ int64_t s_rows[RECMG_MAX_TABLES];
    __shared__ uint32_t *s_bm[RECMG_MAX_TABLES];
    __shared__ int32_t s_ns[RECMG_MAX_TABLES], s_qb[RECMG_MAX_TABLES];
    __shared__ bool s_own[RECMG_MAX_TABLES];
    __shared__ unsigned long long s_set[kLdsSet];
    for (int t = threadIdx.x; t <= g.T; t += blockDim.x) {
        s_start[t] = starts[t];
        if (t < g.T) {
            s_rows[t] = g.tabs[t].rows;
            s_bm[t] = g.tabs[t].bitmap;
            s_ns[t] = g.tabs[t].nsets;
            s_qb[t] = g.tabs[t].qbits;
            s_own[t] = owns_bitmap(g.tabs[t].bm_nblk);
        }
    }
    for (int k = threadIdx.x; k < kLdsSet; k += blockDim.x) s_set[k] = ~0ull;
    __syncthreads();
    if (s_err) return;  // block-uniform
    // each block takes a contiguous chunk, so repeats within the chunk meet in LDS
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
        const int t = find_seg(s_start, g.T, i);
        if (s_own[t]) continue;  // marked by k_mark_own
        const int32_t r = keys[i];
        if (r < 0 || (int64_t)r >= s_rows[t]) {
            atomicOr(g.err, ERR_RANGE);
            continue;
        }
        const unsigned long long key = ((unsigned long long)t << 32) | (uint32_t)r;
        bool mine = true;  // this thread must set the global bit
        uint32_t h = hash_row(r ^ (t * 0x9e3779b9)) & (kLdsSet - 1);
        for (int p = 0; p < kLdsProbes; ++p) {
            unsigned long long cur = s_set[h];
            if (cur == ~0ull) cur = atomicCAS(&s_set[h], ~0ull, key);
            if (cur == ~0ull) break;           // inserted here: mark globally
            if (cur == key) {                  // another thread of the block marks it
                mine = false;
                break;
            }
            h = (h + 1) & (kLdsSet - 1);
        }
        if (mine) {
            const uint32_t pos = bm_pos(s_ns[t], s_qb[t], r);
            uint32_t *w = s_bm[t] + (pos >> 5);
            const uint32_t bit = 1u << (pos & 31);
            if (!(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(w, bit);
        }
    }
}

constexpr int kOwnThreads = 1024;
static_assert(kOwnSliceWords * 32 == 1 << 20, "a slice holds 2^20 bitmap positions");
static_assert(kOwnSliceBlocks <= kOwnThreads && kOwnSliceWords % kWordsPerBlock == 0, "slice = whole bitmap blocks");

// The first kernel of a forward's or a placement's dedup.  Block (slice, table)
// of a grid (slices, T).  Slice 0 of every table checks the call's offsets and
// sets up the table's state (forward_prep / placement_prep); each block of an
// owned table then marks its slice in LDS: the slice's non-zero words go to the
// (all-zero) bitmap and the popcount of each of its bitmap blocks to blocksum.
// Blocks of other tables, and slices past a table's bitmap, end there.
// `offs`: bag offsets with B per table, or the prefetch list's with B = 1.  A
// block whose own range is malformed raises the error and reads no id; range
// errors of ids are raised by slice 0 only.
// A block reads its ids 16 bytes per lane, four loads in flight, with 32-bit
// offsets.  It is bound by the instructions and LDS accesses per id of its CU
// (26 us for 123,000 ids), so many ids are split over parts: a part's block
// writes all of its slice's words to its own copy (part_bm), and k_bm_merge puts
// the copies together and counts them.
template <int MODE>
__global__ void __launch_bounds__(kOwnThreads) k_mark_own(DGlobal g, const int32_t *__restrict__ keys,
                                                          const int64_t *__restrict__ offs, int32_t B, int64_t n,
                                                          int32_t have_fwd) {
    __shared__ uint4 s_bm[kOwnSliceWords / 4];
    __shared__ int s_cnt[kOwnSliceBlocks];
    __shared__ int s_err;
    const int t = blockIdx.y, sl = blockIdx.x, part = blockIdx.z, parts = gridDim.z;
    const DTable &tb = g.tabs[t];
    const int nblk = tb.bm_nblk;
    const bool mark = owns_bitmap(nblk) && sl * kOwnSliceBlocks < nblk;  // block-uniform
    if (!mark && (sl || part)) return;
    // the error word is read once: another block may set it meanwhile, and the
    // waves of the block must agree before its barriers
    if (threadIdx.x == 0) s_err = *g.err;
    const int64_t lo = offs[(int64_t)t * B], hi = offs[(int64_t)(t + 1) * B];
    if (sl == 0 && part == 0) {
        if (MODE == EMIT_FORWARD) forward_prep(g, t, offs, B, n);
        else placement_prep(g, t, offs, n, have_fwd);
    }
    if (!mark) return;  // block-uniform
    const int sblk = nblk - sl * kOwnSliceBlocks < kOwnSliceBlocks ? nblk - sl * kOwnSliceBlocks : kOwnSliceBlocks;
    const int nq = sblk * (kWordsPerBlock / 4);  // uint4 words of the slice
    for (int k = threadIdx.x; k < nq; k += kOwnThreads) s_bm[k] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < kOwnSliceBlocks) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    if (s_err || lo < 0 || hi < lo || hi > n) return;  // block-uniform; forward_prep / placement_prep raise the latter
    uint32_t *bm = reinterpret_cast<uint32_t *>(s_bm);
    const uint32_t rows = (uint32_t)tb.rows;  // < 2^31
    const int32_t ns = tb.nsets, qb = tb.qbits;
    bool bad = false;
    auto mark_id = [&](uint32_t r) {
        if (r >= rows) {  // negative ids too
            bad = true;
            return;
        }
        const uint32_t pos = bm_pos(ns, qb, (int32_t)r);
        if ((int)(pos >> 20) != sl) return;  // the position's slice
        const uint32_t w = (pos >> 5) & (kOwnSliceWords - 1), bit = 1u << (pos & 31);
        if (!(bm[w] & bit)) atomicOr(&bm[w], bit);
    };
    // ids before the first 16-byte boundary, whole 16-byte groups, the rest
    const int64_t plo = lo + (hi - lo) * part / parts, phi = lo + (hi - lo) * (part + 1) / parts;
    const uint32_t cnt = (uint32_t)(phi - plo);
    const int32_t *ids = keys + plo;
    uint32_t head = (uint32_t)((16 - (reinterpret_cast<uintptr_t>(ids) & 15)) & 15) / 4;
    if (head > cnt) head = cnt;
    const uint32_t nv = (cnt - head) / 4, tail0 = head + 4 * nv;
    constexpr uint32_t kV = 4;
    for (uint32_t v0 = threadIdx.x; v0 < nv; v0 += kV * kOwnThreads) {
        uint4 v[kV];
#pragma unroll
        for (uint32_t u = 0; u < kV; ++u)
            if (v0 + u * kOwnThreads < nv) v[u] = gload16(ids + head + 4 * (v0 + u * kOwnThreads));
#pragma unroll
        for (uint32_t u = 0; u < kV; ++u)
            if (v0 + u * kOwnThreads < nv) {
                mark_id(v[u].x);
                mark_id(v[u].y);
                mark_id(v[u].z);
                mark_id(v[u].w);
            }
    }
    const uint32_t rest = head + (cnt - tail0);  // at most 6
    if (threadIdx.x < rest) mark_id((uint32_t)ids[threadIdx.x < head ? threadIdx.x : tail0 + threadIdx.x - head]);
    if (bad && sl == 0) atomicOr(g.err, ERR_RANGE);
    __syncthreads();
    if (parts > 1) {  // block-uniform
        const int64_t words = (int64_t)g.total_bm_blocks * kWordsPerBlock;
        uint4 *dst = reinterpret_cast<uint4 *>(g.part_bm + part * words + (int64_t)tb.bm_block0 * kWordsPerBlock +
                                               (int64_t)sl * kOwnSliceWords);
        for (int k = threadIdx.x; k < nq; k += kOwnThreads) dst[k] = s_bm[k];
        return;
    }
    uint4 *gbm = reinterpret_cast<uint4 *>(tb.bitmap + (int64_t)sl * kOwnSliceWords);
    for (int k = threadIdx.x; k < nq; k += kOwnThreads) {
        const uint4 v = s_bm[k];
        if (v.x | v.y | v.z | v.w) gbm[k] = v;
        int c = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) c += __shfl_xor(c, m);
        // a wave's 64 uint4 words lie in one bitmap block of 256 uint4 words
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(&s_cnt[k / (kWordsPerBlock / 4)], c);
    }
    __syncthreads();
    if (threadIdx.x < sblk) g.blocksum[tb.bm_block0 + sl * kOwnSliceBlocks + threadIdx.x] = s_cnt[threadIdx.x];
}

// Mark the resident rows of every table (for the sorted dump).
__global__ void __launch_bounds__(kBlock) k_mark_resident(DGlobal g) {
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < tb.cap;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = tb.slot_row[k];
        if (r >= 0) atomicOr(tb.bitmap + (r >> 5), 1u << (r & 31));
    }
}

// The table of bitmap block blk (T <= blockDim.x), or -1 if the error word is set
// (read once per block, see block_err): every table's bounds are tested at once,
// where a binary search would chain its loads.  Ends with a barrier.
__device__ __forceinline__ int block_table(const DGlobal &g, int blk) {
    __shared__ int s_t, s_err;
    const int t = threadIdx.x;
    if (t == 0) s_err = *g.err;
    if (t < g.T && g.bm_block_start[t] <= blk && blk < g.bm_block_start[t + 1]) s_t = t;
    __syncthreads();
    return s_err ? -1 : s_t;
}

__global__ void __launch_bounds__(kBlock) k_bm_count(DGlobal g) {
    __shared__ int tmp[16];
    const int blk = blockIdx.x;
    const int t = block_table(g, blk);
    if (t < 0) return;  // block-uniform
    const DTable &tb = g.tabs[t];
    const int64_t w0 = (int64_t)(blk - tb.bm_block0) * kWordsPerBlock + threadIdx.x * kWordsPerThread;
    const uint4 w = *reinterpret_cast<const uint4 *>(tb.bitmap + w0);
    const int c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    const int s = block_sum(c, tmp);
    if (threadIdx.x == 0) g.blocksum[blk] = s;
}

// The parts' copies of a bitmap block put together: its non-zero words to the
// (all-zero) bitmap, their popcount to blocksum.
__global__ void __launch_bounds__(kBlock) k_bm_merge(DGlobal g, int parts) {
    __shared__ int tmp[16];
    const int blk = blockIdx.x;
    const int t = block_table(g, blk);
    if (t < 0) return;  // block-uniform
    const DTable &tb = g.tabs[t];
    const int64_t words = (int64_t)g.total_bm_blocks * kWordsPerBlock;
    const uint32_t *src = g.part_bm + (int64_t)blk * kWordsPerBlock + threadIdx.x * kWordsPerThread;
    uint4 v[kMarkMaxParts];
#pragma unroll
    for (int k = 0; k < kMarkMaxParts; ++k) v[k] = k < parts ? gload16(src + k * words) : make_uint4(0u, 0u, 0u, 0u);
    uint4 w = v[0];
#pragma unroll
    for (int k = 1; k < kMarkMaxParts; ++k) w.x |= v[k].x, w.y |= v[k].y, w.z |= v[k].z, w.w |= v[k].w;
    if (w.x | w.y | w.z | w.w)
        *reinterpret_cast<uint4 *>(tb.bitmap + (int64_t)(blk - tb.bm_block0) * kWordsPerBlock +
                                   threadIdx.x * kWordsPerThread) = w;
    const int s = block_sum(__popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w), tmp);
    if (threadIdx.x == 0) g.blocksum[blk] = s;
}

// One block per table: exclusive scan of the table's block counts (for tables
// of more blocks than k_bm_emit adds up by itself).
__global__ void __launch_bounds__(1024) k_bm_scan(DGlobal g) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    const int t = blockIdx.x;
    const int b0 = g.bm_block_start[t], nb = g.bm_block_start[t + 1] - b0;
    int carry = 0;
    for (int base = 0; base < nb; base += blockDim.x) {
        const int k = base + threadIdx.x;
        const int v = k < nb ? g.blocksum[b0 + k] : 0;
        int tot;
        const int ex = block_excl_scan(v, tmp, &tot);
        if (k < nb) g.blockoff[b0 + k] = carry + ex;
        carry += tot;
    }
}

// Write the distinct ids in ascending order (U, PU or the resident dump), one
// bitmap word per thread.  SCANNED: the block's first rank comes from k_bm_scan;
// else the block adds up the counts of the table's blocks before it (at most
// kEmitThreads), which costs less than a kernel between marking and emitting.
// The table's last block writes its total to counts[t * count_stride]; a block
// without a set bit ends before it reads its words.
constexpr int kEmitThreads = kWordsPerBlock;
template <int MODE, bool SCANNED>
__global__ void __launch_bounds__(kEmitThreads) k_bm_emit(DGlobal g, int32_t *counts, int count_stride, int32_t stamp) {
    __shared__ int tmp[16];
    const int blk = blockIdx.x;
    const int t = block_table(g, blk);
    if (t < 0) return;  // block-uniform
    const DTable &tb = g.tabs[t];
    const int b0 = tb.bm_block0, own = g.blocksum[blk];
    int first;
    if (SCANNED) first = g.blockoff[blk];
    else first = block_sum((int)threadIdx.x < blk - b0 ? g.blocksum[b0 + threadIdx.x] : 0, tmp);
    if (threadIdx.x == 0 && blk == b0 + tb.bm_nblk - 1) counts[(int64_t)t * count_stride] = first + own;
    if (own == 0) return;  // block-uniform
    const int64_t word = (int64_t)(blk - b0) * kWordsPerBlock + threadIdx.x;
    uint32_t *bmw = tb.bitmap + word;
    uint32_t bits = *bmw;
    int32_t *out;
    if (MODE == EMIT_FORWARD) out = g.U + g.tstart[t];
    else if (MODE == EMIT_PREFETCH) out = g.PU + g.pstart[t];
    else out = g.dump + tb.cap_off;
    const int32_t nsets = tb.nsets, qbits = tb.qbits;
    uint4 *rank = tb.rank + word;
    int tot;
    int u = first + block_excl_scan(__popc(bits), tmp, &tot);
    if (!bits) return;
    if (MODE == EMIT_FORWARD) *rank = make_uint4((uint32_t)u, bits, (uint32_t)stamp, 0u);
    *bmw = 0;
    while (bits) {
        const int b = __ffs(bits) - 1;
        bits &= bits - 1;
        const uint32_t pos = (uint32_t)(word * 32 + b);
        out[u++] = MODE == EMIT_DUMP ? (int32_t)pos : bm_row(nsets, qbits, pos);
    }
}

// ------------------------------------------------------------------- launchers

static inline unsigned grid_for(int64_t n, int per_block, unsigned cap) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (int64_t)cap) b = cap;
    return (unsigned)b;
}

// One kernel does it where every table is marked in LDS; larger tables' ids
// are marked by k_mark, from the starts that it has written.
template <int MODE>
static void mark(const DGlobal &g, const int32_t *keys, const int64_t *offs, int32_t B, int64_t n, int32_t have_fwd,
                 const int64_t *starts, hipStream_t s) {
    const unsigned slices = g.own_slices > 0 ? (unsigned)g.own_slices : 1u;
    // Parts: about 16,000 ids each, from 48,000 ids per table on; below, the
    // merge's launch costs what the split saves (some 5 us).  26 resident tables of
    // 123,000 ids: marking 26 -> 6 us and merging 5; the 290,000 prefetch ids of
    // each of 4 tables 60 -> 17 us in all.
    const int64_t per = n / g.T;
    const int parts = per < kMarkSplitIds ? 1 : (int)std::min<int64_t>(g.mark_parts, per / 16384);
    k_mark_own<MODE><<<dim3(slices, (unsigned)g.T, (unsigned)parts), kOwnThreads, 0, s>>>(g, keys, offs, B, n, have_fwd);
    if (parts > 1) k_bm_merge<<<g.total_bm_blocks, kBlock, 0, s>>>(g, parts);
    if (g.own_tables < g.T) k_mark<<<grid_for(n, kBlock * 8, 4096), kBlock, 0, s>>>(g, keys, starts, n);
}

void launch_mark_forward(const DGlobal &g, const int32_t *indices, const int64_t *offsets, int32_t B, int64_t n,
                         hipStream_t s) {
    mark<EMIT_FORWARD>(g, indices, offsets, B, n, 0, g.tstart, s);
}

void launch_mark_prefetch(const DGlobal &g, const int32_t *rows, const int64_t *poff, int64_t np, int32_t have_fwd,
                          hipStream_t s) {
    mark<EMIT_PREFETCH>(g, rows, poff, 1, np, have_fwd, g.pstart, s);
}

void launch_mark_resident(const DGlobal &g, int32_t max_cap, hipStream_t s) {
    if (max_cap <= 0) return;
    dim3 grid(grid_for(max_cap, kBlock * 4, 4096), g.T);
    k_mark_resident<<<grid, kBlock, 0, s>>>(g);
}

void launch_dedup(const DGlobal &g, int mode, int32_t *counts, int count_stride, int32_t stamp, int32_t max_nblk,
                  hipStream_t s) {
    // k_mark_own has counted the owned tables' blocks (not those of the resident dump)
    if (mode == EMIT_DUMP || g.own_tables < g.T) k_bm_count<<<g.total_bm_blocks, kBlock, 0, s>>>(g);
    const bool scanned = max_nblk > kEmitThreads;
    if (scanned) k_bm_scan<<<g.T, 1024, 0, s>>>(g);
    const dim3 grid((unsigned)g.total_bm_blocks), blk(kEmitThreads);
#define RECMG_EMIT(M)                                                                        \
    if (scanned) k_bm_emit<M, true><<<grid, blk, 0, s>>>(g, counts, count_stride, stamp);    \
    else k_bm_emit<M, false><<<grid, blk, 0, s>>>(g, counts, count_stride, stamp);
    if (mode == EMIT_FORWARD) {
        RECMG_EMIT(EMIT_FORWARD)
    } else if (mode == EMIT_PREFETCH) {
        RECMG_EMIT(EMIT_PREFETCH)
    } else {
        RECMG_EMIT(EMIT_DUMP)
    }
#undef RECMG_EMIT
}

}  // namespace recmg

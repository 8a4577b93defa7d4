// Placement between batches: the batched form of Alg. 1 (load_embeddings)
// and Alg. 2 (gpu_buffer_populate), Sec. VI-B.
//
// Per table t the candidate set is K = R ∪ M ∪ set(P): resident slots, the
// last batch's misses (already in HBM staging) and the prefetch list.  Every
// member gets a score (aging, touch, prefetch, below), and the cache keeps the
// min(Cap, |K|) largest keys (score, row).  Instead of one victim scan per
// insertion, one radix select per placement finds the threshold key: 11-bit
// digits from the top, each pass a histogram kernel whose digit, the one holding
// the Cap-th largest key, the next kernel picks.  Keys are
// distinct (rows are distinct), so exactly min(Cap, |K|) keys are >= the
// threshold.
//
// Scores:  LRU_BATCH  touched by the last batch: lru_touch; prefetched:
//                     max(score, pscore) with pscore = lru_touch + 1
//          LFU_BATCH  every row's score is its batch count (last_batch_share adds
//                     the last batch); a prefetch does not change it
//          PRIORITY   residents first age by one, saturating at 0 (Alg. 2);
//                     touched: caching bit + ES (Alg. 1); prefetched:
//                     max(score, ES); a touched resident loses its prefetch flag.
//
// Kernels on the stream: the dedup of P with the placement's preparation
// (dedup.hip; k_plc_prep or k_plc_last if P is empty), k_plc_classify,
// k_plc_update (scores + histogram of pass 0), k_plc_select per further pass
// (which first picks the digit of the pass before), k_plc_evict (which picks the
// last), k_plc_admit, k_plc_end, k_plc_fill.  A map with too many deleted entries
// is rebuilt on the way (map_clear_share).  Placements of few rows run all but
// the end in one kernel (small.hip).
#include <hip/hip_ext.h>

#include "launch.h"
#include "placement_device.h"

namespace recmg {

// The start of a placement with an empty prefetch list (others start in the
// first kernel of the list's dedup): one block per table.
__global__ void k_plc_prep(DGlobal g, const int64_t *__restrict__ poff, int64_t np, int32_t have_fwd) {
    placement_prep(g, blockIdx.x, poff, np, have_fwd);
}

// The last batch's bits or counts alone (an empty prefetch list has no kernel
// for them to ride with), and the placement's start.
__global__ void __launch_bounds__(kBlock) k_plc_last(DGlobal g, const int64_t *__restrict__ poff, int64_t np,
                                                     const uint8_t *__restrict__ bits, int64_t n) {
    const bool err = block_err(g);
    const bool bad = list_malformed(g, poff, np);  // a malformed call changes nothing
    if ((int)blockIdx.x < g.T) placement_prep(g, blockIdx.x, poff, np, 1);
    if (!err && !bad) last_batch_share(g, bits, n);
}

// Classify every distinct prefetch row of the fully associative tables (Alg.
// 1's prefetch loop taken as a set): resident -> flag the slot; missed by the
// last batch -> flag the miss; otherwise a new candidate, appended to NP.  The
// distinct rows are laid end to end, one per thread and round; a round reserves
// its new candidates with one atomic per table (one per wave queued on the
// table states: 1.16 million rows of 4 tables took 300 us, now 69).
// Set-associative tables play their prefetch rows as events in k_sa_place,
// which also counts the resident ones.
// last_n > 0: then the last batch's bits or counts.
__global__ void __launch_bounds__(kRound) k_plc_classify(DGlobal g, int32_t last_stamp, const uint8_t *__restrict__ bits,
                                                         int64_t last_n) {
    __shared__ int s_err;  // read once per block (block_err), behind the barriers of lay_tables
    if (threadIdx.x == 0) s_err = *g.err;
    __shared__ int32_t s_pre[RECMG_MAX_TABLES + 1];
    __shared__ int64_t s_ps[RECMG_MAX_TABLES];
    __shared__ int s_res[RECMG_MAX_TABLES], s_new[RECMG_MAX_TABLES];
    __shared__ int tmp[16];
    if ((int)threadIdx.x < g.T) {
        s_res[threadIdx.x] = s_new[threadIdx.x] = 0;
        s_ps[threadIdx.x] = g.pstart[threadIdx.x];
    }
    const int32_t n = lay_tables(g.T, [&](int t) { return g.tabs[t].ways ? 0 : g.st[t].pcount; }, s_pre, tmp);
    if (s_err) return;  // block-uniform
    int32_t lo, hi;
    round_share(n, kRound, &lo, &hi);
    for (int64_t base = lo; base < hi; base += kRound) {  // block-uniform; 64 bits: hi may be 2^31 - 1
        const bool in = base + threadIdx.x < hi;
        const int32_t i = in ? (int32_t)(base + threadIdx.x) : (int32_t)base;
        const int t = find_seg32(s_pre, g.T, i);
        int64_t at = 0;
        int32_t row = 0, k = -1;
        // rows of one table (nearly every wave): its descriptor is read through scalar loads
        auto classify = [&](const DTable &tb) {
            at = s_ps[t] + (i - s_pre[t]);
            bool isnew = false, resident = false;
            if (in) {
                row = g.PU[at];
                const int32_t slot = map_find(tb, row);
                if (slot >= 0) {
                    // distinct prefetch rows name distinct slots: plain read-modify-write
                    tb.slot_flags[slot] |= F_INP;
                    resident = true;
                    g.puref[at] = slot;
                } else {
                    // distinct rows of the last batch carry its stamp in the rank word
                    const uint4 rk = gload16(tb.rank + ((uint32_t)row >> 5));
                    const uint32_t bit = 1u << (row & 31);
                    if ((int32_t)rk.z == last_stamp && (rk.y & bit)) {
                        const int64_t ts = g.tstart[t];
                        const int32_t u = (int32_t)rk.x + __popc(rk.y & (bit - 1u));
                        const int64_t m = -(int64_t)g.slotU[ts + u] - 1;
                        g.mflags[ts + m] |= F_INP;  // distinct rows, distinct misses
                        g.puref[at] = ring_ref_miss((int32_t)m);
                    } else {
                        isnew = true;
                    }
                }
            }
            wave_count_lds(resident, t, s_res);  // counts only
            k = wave_append(isnew, t, s_new, 1);
        };
        const int t0 = __builtin_amdgcn_readfirstlane(t);
        if (__ballot(t != t0) == 0) classify(g.tabs[t0]);
        else classify(g.tabs[t]);
        __syncthreads();
        int *cnt = s_new + threadIdx.x;  // counts -> first candidate of this round
        if ((int)threadIdx.x < g.T && *cnt) *cnt = atomicAdd(&g.st[threadIdx.x].npcount, *cnt);
        __syncthreads();
        if (k >= 0) {
            k += s_new[t];
            g.NP[s_ps[t] + k] = row;
            g.puref[at] = ring_ref_new(k);
        }
        __syncthreads();
        if ((int)threadIdx.x < g.T) *cnt = 0;
        __syncthreads();
    }
    if ((int)threadIdx.x < g.T && s_res[threadIdx.x]) atomicAdd(&g.st[threadIdx.x].p_res, s_res[threadIdx.x]);
    if (last_n > 0) last_batch_share(g, bits, last_n);
}

// ----------------------------------------------------------------- ranking

// Merge the block's histogram into the table's global one (non-zero bins).
// No fence and no "last block" here: on this GPU an agent-scope fence writes
// back the XCD's whole L2, and a histogram kernel has many blocks; the digit
// is picked after the kernel boundary instead (pass_threshold).
__device__ __forceinline__ int *pass_hist(const DGlobal &g, int pass, int t) {
    return g.hist + ((int64_t)pass * g.T + t) * kRadix;
}
__device__ __forceinline__ void hist_merge(const DGlobal &g, int pass, int t, const int *s_hist) {
    int *gh = pass_hist(g, pass, t);
    for (int b = threadIdx.x; b < kRadix; b += blockDim.x)
        if (s_hist[b]) atomicAdd(&gh[b], s_hist[b]);
}

// The threshold prefix after pass `pass`, from the table's finished histogram
// of that pass: by every block of the kernel that follows, for itself (8 KiB
// from L2 and a scan, about 2 us beside the block's other loads; a kernel of its
// own per pass cost 6 to 7 us).  Each pass has its own histogram, so none is
// cleared here, and writes its result to its own place: block 0 of the table
// does it for the next pass's kernel, and no block of this kernel reads it.
// s_hist is used up.  Every thread calls.
__device__ __forceinline__ uint64_t pass_threshold(const DGlobal &g, TState &st, int t, int pass, int keep, int *s_hist,
                                                   int *tmp) {
    const int *gh = pass_hist(g, pass, t);
    for (int b = threadIdx.x; b < kRadix; b += blockDim.x) s_hist[b] = gh[b];
    const int need = pass == 0 ? keep : st.pass_need[pass - 1];
    const uint64_t before = pass == 0 ? 0 : st.pass_prefix[pass - 1] << kRadixBits;
    __syncthreads();
    int digit, rest;
    pick_digit(s_hist, need, tmp, &digit, &rest);
    const uint64_t prefix = before | (uint64_t)digit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st.pass_prefix[pass] = prefix;
        st.pass_need[pass] = rest;
    }
    return prefix;
}

// Scores of every candidate (written back) and the first select pass.
__global__ void __launch_bounds__(kBlock) k_plc_update(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int s_hist[kRadix];
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    TState &st = g.st[t];
    if (tb.ring_cap) return;  // ranked in ring.hip
    const Counts c = table_counts(tb, st, p);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st.sel_mode = tb.ways ? SEL_NONE : c.mode;  // set-associative tables place in setassoc.hip
        st.plc_nm = c.nm;
    }
    if (tb.ways) return;
    const bool sel = c.mode == SEL_SELECT;
    if (sel)
        for (int b = threadIdx.x; b < kRadix; b += blockDim.x) s_hist[b] = 0;
    __syncthreads();
    update_items(g, p, tb, c, t, s_hist, sel, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
                 (int64_t)gridDim.x * blockDim.x, FlagInp());
    __syncthreads();
    if (sel) hist_merge(g, 0, t, s_hist);
}

__global__ void __launch_bounds__(kBlock) k_plc_select(DGlobal g, PlcParams p, int pass) {
    if (block_err(g)) return;
    __shared__ int s_hist[kRadix];
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    TState &st = g.st[t];
    if (tb.ring_cap || st.sel_mode != SEL_SELECT) return;  // uniform over the table's blocks
    const Counts c = table_counts(tb, st, p);
    __shared__ int tmp[16];
    const uint64_t prefix = pass_threshold(g, st, t, pass - 1, c.keep, s_hist, tmp);
    for (int b = threadIdx.x; b < kRadix; b += blockDim.x) s_hist[b] = 0;
    __syncthreads();
    select_items(g, p, tb, c, t, s_hist, pass, prefix, (int64_t)blockIdx.x * blockDim.x + threadIdx.x,
                 (int64_t)gridDim.x * blockDim.x);
    __syncthreads();
    hist_merge(g, pass, t, s_hist);
}

// Small tables: the whole ranking of a table in one block (scores, then every
// pass's histogram in LDS and its digit), one launch instead of 2 per pass.
constexpr int kRankSmallThreads = 1024;
__global__ void __launch_bounds__(kRankSmallThreads) k_plc_rank_small(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int s_hist[kRadix];
    __shared__ int tmp[16];
    const int t = blockIdx.x;
    const DTable &tb = g.tabs[t];
    TState &st = g.st[t];
    if (tb.ring_cap) return;
    const Counts c = table_counts(tb, st, p);
    if (threadIdx.x == 0) {
        st.sel_mode = tb.ways ? SEL_NONE : c.mode;
        st.plc_nm = c.nm;
    }
    if (tb.ways) return;
    const uint64_t thr = rank_block(g, p, tb, c, t, s_hist, tmp, FlagInp());
    if (threadIdx.x == 0 && c.mode == SEL_SELECT) st.prefix = thr;
}

// ----------------------------------------------------------------- evict / admit

// Slots a block collects in LDS before it reserves free-stack space for
// them: one atomic on the table's stack top per block in the common case (a
// few hundred evictions per block), instead of one per 256 slots scanned (a
// full cache of 19.5 million slots would queue some 76,000 of those on one
// word per table).  Freed slots enter the stack in no fixed order; slot
// numbers are not observable.
constexpr int kEvictBuf = 2048;

// last_pass: the radix select's last pass, whose digit gives the threshold key
// (-1: k_plc_rank_small has found it).
__global__ void __launch_bounds__(kBlock) k_plc_evict(DGlobal g, PlcParams p, int last_pass) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    __shared__ int s_base, s_n;
    __shared__ int32_t s_free[kEvictBuf];
    static_assert(kEvictBuf >= kRadix, "the last pass's histogram takes the buffer's place first");
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    if (tb.ways || tb.ring_cap) return;
    TState &st = g.st[t];
    const int mode = st.sel_mode;
    uint64_t thr = 0;
    if (mode == SEL_SELECT) {  // block-uniform
        if (last_pass < 0) thr = st.prefix;
        else {
            thr = pass_threshold(g, st, t, last_pass, table_counts(tb, st, p).keep, s_free, tmp);
            if (blockIdx.x == 0 && threadIdx.x == 0) st.prefix = thr;  // for admission
        }
    }
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    // reserve stack space for the collected slots with one atomic and write
    // them out; every thread calls (s_n is read after a barrier)
    auto flush = [&]() {
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
    unsigned long long dig = 0;
    const int64_t cap = tb.cap;
    // four slots per thread; a block's iterations are uniform (its barriers)
    const int64_t ngrp = (cap + 3) / 4, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < ngrp; base += stride) {
        const int64_t q = base + threadIdx.x;
        const int64_t k0 = 4 * q;
        const int64_t lim = q < ngrp ? cap : 0;
        int32_t row[4], sc[4];
        slot_quad(tb.slot_row, k0, lim, -1, row);
        slot_quad(tb.slot_score, k0, lim, 0, sc);
        bool evs[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool keep = row[i] >= 0 && kept(mode, make_key(sc[i], row[i], p.rowbits), thr);
            if (keep) dig += mix64(((unsigned long long)t << 40) | (unsigned long long)row[i]);
            evs[i] = row[i] >= 0 && !keep;
        }
        if (!reb) map_delete_n<4>(tb, row, evs);  // their first probes in flight together
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t k = k0 + i;
            const bool ev = evs[i];
            if (ev) {
                tb.slot_row[k] = -1;
                tb.slot_flags[k] = 0;
            }
            // append the wave's freed slots to the block's list (one LDS atomic per wave)
            const uint64_t m = __ballot(ev);
            int wb = 0;
            if (lane == 0 && m) wb = atomicAdd(&s_n, __popcll(m));
            wb = __shfl(wb, 0);
            if (ev) s_free[wb + __popcll(m & ((1ull << lane) - 1ull))] = (int32_t)k;
        }
        if (list_past(&s_n, kEvictBuf - 4 * (int)blockDim.x)) flush();  // room for one more pass of the block
    }
    __syncthreads();
    flush();
    __shared__ unsigned long long s_dig[kBlock / 64];
    const unsigned long long d = block_sum64(dig, s_dig);
    if (threadIdx.x == 0 && d) atomicAdd(&st.digest_acc, d);
}

// Candidates kept: slots from the free stack's top, map entries, the fill list.
// A block takes Q candidates per thread and round with their loads (and first
// map attempts) in flight together, and reserves its slots with one atomic.
// Q = 4 where the candidates are many: a chain of five dependent accesses and an
// atomic per 256 of them took 133 us for 487,000 rows of 4 tables, 71 now.  Q = 1
// below kAdmitMany per table, where blocks are few (6,600 candidates in each of
// 13 tables: 16 us, 26 with Q = 4).
constexpr int64_t kAdmitMany = 65536;
template <int Q>
__global__ void __launch_bounds__(kBlock) k_plc_admit(DGlobal g, PlcParams p) {
    if (block_err(g)) return;
    __shared__ int tmp[16];
    __shared__ int s_base;
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    if (tb.ways) return;
    TState &st = g.st[t];
    const Counts c = table_counts(tb, st, p);
    const int mode = st.sel_mode;
    const uint64_t thr = st.prefix;
    const bool reb = st.rebuild != 0;  // k_plc_end inserts every resident
    const int32_t top = st.free_top, cap = tb.cap;
    const int64_t ts = g.ftstart[t], ps = g.pstart[t];
    const int64_t items = (int64_t)c.nm + c.nnp;
    const bool ring = tb.ring_cap != 0, staged = tb.staged != 0;
    const int32_t *stack = tb.free_stack;
    int n_adm_miss = 0, n_pdrop = 0, n_reuse = 0;
    unsigned long long dig = 0;
    for (int64_t base = (int64_t)blockIdx.x * (Q * kBlock); base < items; base += (int64_t)gridDim.x * (Q * kBlock)) {
        int32_t row[Q], sc[Q], slot[Q];
        bool adm[Q], inp[Q];
        int mine = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t k = base + q * kBlock + threadIdx.x;
            row[q] = sc[q] = 0;
            inp[q] = true;
            if (k < c.nm) {
                row[q] = (int32_t)gload4(g.M + ts + k);
                sc[q] = (int32_t)gload4(g.mscore + ts + k);
                inp[q] = (gload4(g.mflags + ts + k) & F_INP) != 0;
            } else if (k < items) {
                row[q] = (int32_t)gload4(g.NP + ps + (k - c.nm));
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t k = base + q * kBlock + threadIdx.x;
            if (k >= c.nm && k < items) sc[q] = new_prefetch_score(p, tb, row[q]);
            adm[q] = k < items && kept(mode, make_key(sc[q], row[q], p.rowbits), thr);
            mine += adm[q] ? 1 : 0;
        }
        int tot;
        const int ex = block_excl_scan(mine, tmp, &tot);
        if (threadIdx.x == 0 && tot) s_base = atomicAdd(&st.popped, tot);
        __syncthreads();
        int32_t at[Q];
        int nth = s_base + ex;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            at[q] = nth;
            nth += adm[q] ? 1 : 0;
            const int64_t fi = (int64_t)top - 1 - at[q], fj = ts + ps + at[q];  // fj: this row's entry in the fill list
            slot[q] = adm[q] && fi >= 0 && fi < cap && fj >= 0 && fj < g.fill_cap ? (int32_t)gload4(stack + fi) : -1;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t k = base + q * kBlock + threadIdx.x;
            const bool is_miss = k < c.nm;
            if (adm[q] && (uint32_t)slot[q] >= (uint32_t)cap) {
                atomicOr(g.err, ERR_INTERNAL);
                adm[q] = false;
            }
            if (!adm[q]) {
                n_pdrop += k < items && inp[q] ? 1 : 0;
                continue;
            }
            tb.slot_row[slot[q]] = row[q];
            if (!ring) tb.slot_score[slot[q]] = sc[q];  // a ring's order holds its scores
            // (the slot's touch stamp, of a forward before this placement, is
            // older than any a later placement asks for)
            tb.slot_flags[slot[q]] = inp[q] ? F_PF : 0u;
            // the fill list: admitted row j of this table, its source and slot: a
            // miss's staging row; a prefetch row's host row, or for a STAGED table
            // the staged row of its candidate (the host gathered NP[ps + i] into
            // row ps + i)
            const int64_t fj = ts + ps + at[q];
            g.fill_src[fj] = is_miss ? (int32_t)k : staged ? -(int32_t)(ps + (k - c.nm)) - 1 : -(row[q] + 1);
            g.fill_slot[fj] = slot[q];
            if (ring) {  // where ring.hip finds the admitted rows' slots
                if (is_miss) g.mslot[ts + k] = slot[q];
                else g.npslot[ps + (k - c.nm)] = slot[q];
            }
            dig += mix64(((unsigned long long)t << 40) | (unsigned long long)row[q]);
            n_adm_miss += is_miss ? 1 : 0;
        }
        if (!reb) n_reuse += map_insert_n<Q>(tb, row, slot, adm);
        __syncthreads();  // before s_base is set again
    }
    const int a = block_sum(n_adm_miss, tmp), pd = block_sum(n_pdrop, tmp), ru = block_sum(n_reuse, tmp);
    __shared__ unsigned long long s_dig[kBlock / 64];
    const unsigned long long d = block_sum64(dig, s_dig);
    if (threadIdx.x == 0) {
        if (d) atomicAdd(&st.digest_acc, d);
        if (a) atomicAdd(&st.adm_miss, a);
        if (pd) atomicAdd(&st.p_drop, pd);
        if (ru) atomicAdd(&st.reused, ru);
    }
}

// The fill by the first nb blocks of a grid: first_of(t), count_of(t) give
// table t's entries in the fill list, miss0_of(t) the base of its admitted
// misses in staging.
template <class First, class Count, class Miss0>
__device__ __forceinline__ void fill_rows(const DGlobal &g, int phase, int64_t nb, First first_of, Count count_of,
                                          Miss0 miss0_of) {
    // admit and the set-associative placement checked the entries that they wrote
    copy_flat(
        g,
        [&](int t) {
            const int64_t base = first_of(t), n = count_of(t);
            const bool mine = (g.tabs[t].staged != 0) == (phase == FILL_STAGED);
            return mine && base >= 0 && n >= 0 && base + n <= g.fill_cap ? (int32_t)n : 0;
        },
        [&](int64_t) { return nb; },
        [&](int t, const DTable &tb, int64_t j) -> const char * {
            const int32_t src = g.fill_src[first_of(t) + j];
            if (src >= 0) return g.staging + (miss0_of(t) + src) * g.stage_stride;  // admitted miss
            return tb.staged ? g.fstage + (int64_t)(-src - 1) * g.stage_stride  // prefetch row, host-staged
                             : tb.host + (int64_t)(-src - 1) * tb.row_bytes;    // prefetch row, zero-copy
        },
        [&](int t, const DTable &tb, int64_t j) { return tb.pool + (int64_t)g.fill_slot[first_of(t) + j] * tb.row_bytes; });
}

// Publishes table t's counters and moves its state past this placement; one
// thread.  log_slot >= 0: the counters also go to that call's record of the
// stats log (the forward group of the record stays zero).
__device__ __forceinline__ void publish_placement(const DGlobal &g, int t, int64_t *fdesc, int64_t log_slot) {
    TState &st = g.st[t];
    const DTable &tb = g.tabs[t];
    if (fdesc) {
        fdesc[4 * t] = g.ftstart[t] + g.pstart[t];
        fdesc[4 * t + 1] = st.popped;
        fdesc[4 * t + 2] = g.ftstart[t];
    }
    int32_t n_res = st.n_res, evicted = st.evicted, fill = st.p_fill, m_drop = st.m_drop;
    const int32_t adm_miss = st.adm_miss;
    if (!tb.ways) {  // set-associative tables count these as they place
        const int32_t before = st.free_top, popped = st.popped, top = before - popped;  // popped stays: the fill reads it
        evicted = before - st.free0;
        fill = popped - adm_miss;
        m_drop = st.plc_nm - adm_miss;
        st.free_top = top;
        n_res = tb.cap - top;
        st.n_res = n_res;
        const int32_t tomb = st.rebuild ? 0 : st.tomb + evicted - st.reused;
        st.tomb = tomb;
        st.rebuild_next = (int64_t)tomb * 4 > (int64_t)tb.map_mask + 1 ? 1u : 0u;
    }
    if (tb.ring_cap) {  // the ring's new front and back, the new pending list
        int32_t head;
        if (st.r_compact) {  // the live entries moved to the front of the other buffer
            st.r_buf ^= 1;
            st.r_tail = 0;
            head = st.r_moved + st.z1_len;
            st.r_compact = 0;
        } else {
            st.r_tail = st.r_cut;
            head = st.r_head + st.z1_len;
        }
        st.r_head = head;
        st.pend_n = st.pcount;
        st.pend_off = g.pstart[t];
        const int32_t stale = (int32_t)(uint32_t)st.touched, run = (int32_t)(st.appended >> 32);
        const int32_t valid = st.r_valid - stale - (evicted - st.z_evicted) + run;
        st.r_valid = valid;
        if (valid + (int32_t)(uint32_t)st.appended != n_res || head > tb.ring_cap) atomicOr(g.err, ERR_INTERNAL);
    }
    int64_t v[kPlcStats];
    v[0] = evicted;
    v[1] = adm_miss;
    v[2] = fill;
    v[3] = st.p_res;
    v[4] = st.p_drop;
    v[5] = m_drop;
    v[6] = n_res;
    v[7] = (int64_t)fill * tb.row_bytes;
    v[8] = st.pcount;
    for (int k = 0; k < kPlcStats; ++k) {
        st.last[kFwdStats + k] = v[k];
        st.total[kFwdStats + k] += v[k];
    }
    st.digest = st.digest_acc;
    if (log_slot >= 0) {
        int64_t *rec = g.stat_log + (log_slot * g.T + t) * (kNumStats + 1);
        for (int k = 0; k < kNumStats; ++k) rec[k] = k < kFwdStats ? 0 : v[k - kFwdStats];
        rec[kNumStats] = (int64_t)st.digest_acc;
    }
}

// Copy admitted rows into their slots: misses from HBM staging, prefetch
// fills from pinned host memory over the host link (ZERO_COPY tables) or from
// rows the host staged and copied in (STAGED tables).  One launch per miss
// mode present (phase): the zero-copy tables' at once, the STAGED tables'
// after the host has staged their rows.  May run on a side stream,
// concurrently with the next forward and with the next placement: it reads
// only its own placement's fill list and descriptor (both double-buffered, see
// k_plc_end) and the staging buffer of the forward before that placement,
// which the next forward does not use.
__global__ void __launch_bounds__(kBlock) k_plc_fill(DGlobal g, const int64_t *__restrict__ fdesc, int phase) {
    if (block_err(g)) return;
    // the blocks that copy: zero-copy fills as many as k_plc_end chose
    // (fdesc[3]), HBM-to-HBM copies of STAGED rows the whole grid
    const int64_t nb = phase == FILL_STAGED ? (int64_t)gridDim.x
                       : fdesc[3] < 1 ? 1 : fdesc[3] > (int64_t)gridDim.x ? (int64_t)gridDim.x : fdesc[3];
    if ((int64_t)blockIdx.x >= nb) return;  // block-uniform
    fill_rows(g, phase, nb, [&](int t) { return fdesc[4 * t]; }, [&](int t) { return fdesc[4 * t + 1]; },
              [&](int t) { return fdesc[4 * t + 2]; });
}

#ifndef RECMG_FILL_BLOCKS
#define RECMG_FILL_BLOCKS 112  // zero-copy fill alone on the host link
#endif
#ifndef RECMG_FILL_BLOCKS_SHARED
#define RECMG_FILL_BLOCKS_SHARED 256  // zero-copy fill beside the next forward's on-demand fetch
#endif
#ifndef RECMG_FILL_BLOCKS_BIG
#define RECMG_FILL_BLOCKS_BIG 512  // zero-copy fill beside a fetch of a few hundred MB
#endif
#ifndef RECMG_FILL_BLOCKS_HUGE
#define RECMG_FILL_BLOCKS_HUGE 768  // ... and of more
#endif
constexpr int kStagedFillBlocks = 1024;
// on-demand fetch bytes above which the next fetch is taken to share the link
// with the fill (below it, the fetch takes a few microseconds of link time)
constexpr unsigned long long kSharedFetchBytes = 1ull << 20;
// ... above which the two hold the link together for milliseconds
constexpr unsigned long long kBigFetchBytes = 1ull << 28;
// ... and for most of the step
constexpr unsigned long long kHugeFetchBytes = 1ull << 29;
constexpr int max_of(int a, int b) { return a > b ? a : b; }
constexpr int kFillGridBlocks = max_of(max_of(RECMG_FILL_BLOCKS, RECMG_FILL_BLOCKS_SHARED),
                                       max_of(RECMG_FILL_BLOCKS_BIG, RECMG_FILL_BLOCKS_HUGE));

// The end of a placement.  Blocks by role:
//   [0, nfill)         the fill, where it runs with the placement (small batches:
//                      see recmg_apply_placement); else nfill = 0
//   [nfill, + T)       table blockIdx.x - nfill: a set-associative table's counts
//                      added up (sa_sum), its counters published, its fill
//                      descriptor written (fdesc, where the fill runs apart)
//   the rest           the maps that this placement cleared, refilled
// fdesc (per table: first fill-list entry, entry count, base of its admitted
// misses in staging) is what a fill on another stream reads instead of state
// the next placement resets.  fdesc[3] (a spare word of table 0's entry) is the
// number of blocks such a fill copies with: zero-copy fills take more when the
// last forward fetched at least 1 MB on demand, since the next forward's fetch
// will then share the host link (with fewer waves of its own the fill gets less
// of it), more still when it fetched at least 256 MB or 512 MB (the two then
// hold the link for milliseconds or tens of them, and the kernels beside them
// are a small part of the step), and fewer when the fill has the link to itself, so that it
// takes no more CUs than it needs from the kernels beside it.
// Table blocks also clear the radix select's histograms.
__global__ void __launch_bounds__(kBlock) k_plc_end(DGlobal g, int64_t *fdesc, int64_t log_slot, int32_t nfill,
                                                    int32_t nsa, int32_t passes) {
    if (block_err(g)) return;
    __shared__ long long tmp[16];
    if ((int)blockIdx.x < nfill) {  // block-uniform, as the other roles
        fill_rows(g, FILL_ZERO_COPY, nfill, [&](int t) { return g.ftstart[t] + g.pstart[t]; },
                  [&](int t) { return (int64_t)g.st[t].popped; }, [&](int t) { return g.ftstart[t]; });
        return;
    }
    const int r = (int)blockIdx.x - nfill;
    if (r >= g.T) {
        const int nb = (int)gridDim.x - nfill - g.T;
        const bool mine = (int)threadIdx.x < g.T && g.st[threadIdx.x].rebuild != 0;
        if (!__syncthreads_or(mine)) return;
        for (int t = 0; t < g.T; ++t)
            if (g.st[t].rebuild) map_refill_share(g.tabs[t], r - g.T, nb);
        return;
    }
    if (nsa > 0 && g.tabs[r].ways) sa_sum_table(g, r, nsa, tmp);
    if (passes > 0 && g.st[r].sel_mode == SEL_SELECT && !g.tabs[r].ways && !g.tabs[r].ring_cap)
        for (int k = 0; k < passes; ++k) {
            int *h = pass_hist(g, k, r);
            for (int b = threadIdx.x; b < kRadix; b += blockDim.x) h[b] = 0;
        }
    if (r == 0 && fdesc) {
        long long mb = 0, tot;  // bytes of the last forward's on-demand misses
        if ((int)threadIdx.x < g.T) {
            const int32_t m = g.st[threadIdx.x].mcount;
            mb = (long long)(m > 0 ? m : 0) * g.tabs[threadIdx.x].row_bytes;
        }
        (void)block_excl_scan64(mb, tmp, &tot);
        if (threadIdx.x == 0)
            fdesc[3] = (unsigned long long)tot >= kHugeFetchBytes     ? RECMG_FILL_BLOCKS_HUGE
                       : (unsigned long long)tot >= kBigFetchBytes    ? RECMG_FILL_BLOCKS_BIG
                       : (unsigned long long)tot >= kSharedFetchBytes ? RECMG_FILL_BLOCKS_SHARED
                                                                      : RECMG_FILL_BLOCKS;
    }
    if (threadIdx.x == 0) publish_placement(g, r, fdesc, log_slot);
}

// Initial state: every slot free, the free stack handing out slot 0 first.
__global__ void __launch_bounds__(kBlock) k_init_state(DGlobal g) {
    const int t = blockIdx.y;
    const DTable &tb = g.tabs[t];
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < tb.cap; k += (int64_t)gridDim.x * blockDim.x)
        tb.free_stack[k] = tb.cap - 1 - (int32_t)k;
    if (blockIdx.x == 0 && threadIdx.x == 0) g.st[t].free_top = tb.cap;
}

// ----------------------------------------------------------------- launchers

static inline unsigned grid_for(int64_t n, int per_block, unsigned cap) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (int64_t)cap) b = cap;
    return (unsigned)b;
}

void launch_plc_prep(const DGlobal &g, const int64_t *poff, int64_t np, int32_t have_fwd, hipStream_t s) {
    k_plc_prep<<<g.T, 64, 0, s>>>(g, poff, np, have_fwd);
}

void launch_plc_last(const DGlobal &g, const int64_t *poff, int64_t np, const uint8_t *bits, int64_t last_n,
                     hipStream_t s) {
    const unsigned blocks = grid_for(last_n, kBlock * 4, 8192);
    k_plc_last<<<blocks < (unsigned)g.T ? (unsigned)g.T : blocks, kBlock, 0, s>>>(g, poff, np, bits, last_n);
}

void launch_plc_classify(const DGlobal &g, int32_t last_stamp, int64_t np, const uint8_t *bits, int64_t last_n,
                         hipStream_t s) {
    k_plc_classify<<<grid_for(np > last_n / 4 ? np : last_n / 4, kRound, 1024), kRound, 0, s>>>(g, last_stamp, bits, last_n);
}

static bool rank_in_block(const DGlobal &g, int64_t item_bound) {
    return g.hist_sets == 0 || item_bound <= kRankSmallItems;
}

void launch_plc_rank(const DGlobal &g, const PlcParams &p, int64_t item_bound, hipStream_t s) {
    if (rank_in_block(g, item_bound)) {  // a table's slots and candidates fit one block's loop
        k_plc_rank_small<<<g.T, kRankSmallThreads, 0, s>>>(g, p);
        return;
    }
    // few blocks per table, as each merges its non-zero histogram bins into
    // global memory: 32 items per thread where that gives some 512 blocks in all,
    // fewer items where it would leave the chip idle (13 tables of up to 60,000
    // slots were 117 blocks)
    const int64_t want = item_bound * g.T / (kBlock * 512) + 1;
    const int ipt = (int)(want < 4 ? 4 : want > 32 ? 32 : want);
    const dim3 grid(grid_for(item_bound, kBlock * ipt, 512), g.T);
    k_plc_update<<<grid, kBlock, 0, s>>>(g, p);
    for (int pass = 1; pass < p.passes; ++pass) k_plc_select<<<grid, kBlock, 0, s>>>(g, p, pass);
}

void launch_plc_evict(const DGlobal &g, const PlcParams &p, int32_t max_cap, int64_t item_bound, hipStream_t s) {
    const int last = rank_in_block(g, item_bound) ? -1 : p.passes - 1;
    // each block picks the last digit for itself (2 us), so it takes four rounds
    // of slots where there are that many
    k_plc_evict<<<dim3(grid_for(max_cap, kBlock * (max_cap > 1 << 16 ? 16 : 4), 2048), g.T), kBlock, 0, s>>>(g, p, last);
}

void launch_plc_admit(const DGlobal &g, const PlcParams &p, int64_t cand_bound, hipStream_t s) {
    if (cand_bound > kAdmitMany) k_plc_admit<4><<<dim3(grid_for(cand_bound, kBlock * 4, 2048), g.T), kBlock, 0, s>>>(g, p);
    else k_plc_admit<1><<<dim3(grid_for(cand_bound, kBlock, 2048), g.T), kBlock, 0, s>>>(g, p);
}

void launch_plc_fill(const DGlobal &g, const int64_t *fdesc, int phase, hipStream_t s, hipEvent_t ev0,
                     hipEvent_t ev1) {
    // Zero-copy fills read the host: about a hundred blocks of 4-deep 16-byte
    // loads keep the host link full (about 2 MB in flight) when the fill has
    // it to itself.  Host reads hold a CU's L1 miss slots for microseconds, so
    // a larger grid slows every kernel that shares its CUs: with 512 blocks the
    // next forward's dedup, running alongside, took 0.88 ms on configuration 2
    // instead of 0.28 ms.  Measured on configuration 2 (no on-demand misses):
    // 80-96 blocks leave the link short, 160 and more slow the placement that
    // runs beside the fill (192: -8% lookups/s).  On configuration 3 the fill
    // shares the link with the next forward's fetch of about 330,000 misses
    // (85 MB), and 256 blocks gave +4% (512: -6%).  On configuration 5 the
    // fetch moves about 750 MB per batch beside a 3.8 GB fill for most of the
    // step: 768 blocks with the fetch's 288 (see launch_fetch) 82.4 ms per step,
    // 512 and 96 blocks 83.7, 256 and 96 85.9, 1,024 and 96 84.0; with 32-way sets
    // 41.7, 43.6 with 512 and 96.  The grid holds
    // the largest count; k_plc_end writes how many of its blocks copy.
    // STAGED fills copy within HBM and take a full grid.
    const int blocks = phase == FILL_STAGED ? kStagedFillBlocks : kFillGridBlocks;
    if (ev0 || ev1) hipExtLaunchKernelGGL(k_plc_fill, dim3(blocks), dim3(kBlock), 0, s, ev0, ev1, 0, g, fdesc, phase);
    else k_plc_fill<<<blocks, kBlock, 0, s>>>(g, fdesc, phase);
}

void launch_plc_end(const DGlobal &g, int64_t *fdesc, int64_t log_slot, bool fill, int32_t max_fa_cap, int32_t nsa,
                    int32_t passes, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int32_t nfill = fill ? RECMG_FILL_BLOCKS : 0;
    const unsigned refill = max_fa_cap > 0 ? grid_for(max_fa_cap, kBlock * 4, 256) : 0;
    const dim3 grid((unsigned)nfill + (unsigned)g.T + refill);
    if (ev0 || ev1) hipExtLaunchKernelGGL(k_plc_end, grid, dim3(kBlock), 0, s, ev0, ev1, 0, g, fdesc, log_slot, nfill, nsa, passes);
    else k_plc_end<<<grid, kBlock, 0, s>>>(g, fdesc, log_slot, nfill, nsa, passes);
}

void launch_init_state(const DGlobal &g, int32_t max_cap, hipStream_t s) {
    k_init_state<<<dim3(grid_for(max_cap, kBlock * 4, 2048), g.T), kBlock, 0, s>>>(g);
}

}  // namespace recmg

// Forward of one batch: pooled embedding-bag lookup over the two-tier store.
//
// Order of work on the stream (dedup and probe live in dedup.hip):
//   k_mark_own (and k_mark), k_bm_emit   bag offsets checked, each table's
//                index range recorded, distinct rows sorted
//   k_fwd_probe  map probe of the distinct rows, prefetch coverage
//   k_fetch      ZERO_COPY: copy each distinct missing row once from pinned
//                host memory to HBM staging (GPU reads over the host link); one
//                block publishes the counters, further blocks write per index
//                where its row lives (slot or staging row), through the rank of
//                the row among the distinct rows.  (k_fwd_src writes the
//                locations ahead of it where a placement on another stream may
//                want them; k_fwd_finalize publishes a forward of no indices.)
//   k_pool       per bag, sum of its rows in fp32 (Sec. II, pooling by sum)
// A forward of few ids per table runs the part before the fetch in one kernel
// (k_fwd_small, small.hip).
#include <type_traits>

#include <hip/hip_ext.h>

#include "launch.h"

namespace recmg {

// A forward of no indices: offsets checked, counters zero (one block per table;
// other forwards do this in the first kernel of their dedup).
__global__ void __launch_bounds__(kBlock) k_fwd_prep(DGlobal g, const int64_t *__restrict__ offsets, int32_t B,
                                                     int64_t n) {
    forward_prep(g, blockIdx.x, offsets, B, n);
}

// Many bags: their offsets are checked over the whole chip, before the forward's
// first kernel (one block per table took 70 us for 262,144).
__global__ void __launch_bounds__(kBlock) k_bag_offsets(DGlobal g, const int64_t *__restrict__ offsets, int64_t bags) {
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < bags; i += (int64_t)gridDim.x * kBlock)
        bad |= offsets[i] > offsets[i + 1];
    if (bad) atomicOr(g.err, ERR_OFFSETS);
}

// Cache probe of every distinct row (row -> slot map, or a scan of the row's
// set in a set-associative table): hits are stamped and counted, misses are
// numbered (their staging row).  The tables' distinct rows are laid end to end
// and dealt to the blocks in contiguous shares, so no block is spent on the
// repeats of the index space; a round of one row per thread reserves its misses
// with one atomic per table (an atomic per wave queued on the state's few
// lines).  Small blocks of one round each: this kernel runs beside the fill,
// whose host reads hold the L1s of the CUs they run on, and blocks of 1,024
// threads or of four rows per thread then waited at their barriers for their
// slowest wave (259 and 293 us on 402,000 rows, 61 with 256 threads).
// Then coverage (Eq. coverage): how many distinct rows of the last placement's
// prefetch list (PU, still in place) this batch touches: a row is in the batch
// iff its rank word carries this forward's stamp and its bit.
constexpr int kProbeRound = 256;
__global__ void __launch_bounds__(kProbeRound) k_fwd_probe(DGlobal g, int32_t stamp, int cover) {
    __shared__ int s_err;  // read once per block (block_err), behind the barriers of lay_tables
    if (threadIdx.x == 0) s_err = *g.err;
    __shared__ int32_t s_pre[RECMG_MAX_TABLES + 1];
    __shared__ int64_t s_ts[RECMG_MAX_TABLES];
    __shared__ int s_hits[RECMG_MAX_TABLES], s_hits_pf[RECMG_MAX_TABLES], s_miss[RECMG_MAX_TABLES];
    __shared__ int tmp[16];
    if ((int)threadIdx.x < g.T) {
        s_hits[threadIdx.x] = s_hits_pf[threadIdx.x] = s_miss[threadIdx.x] = 0;
        s_ts[threadIdx.x] = g.tstart[threadIdx.x];
    }
    const int32_t n = lay_tables(g.T, [&](int t) { return g.st[t].ucount; }, s_pre, tmp);
    if (s_err) return;  // block-uniform
    int32_t lo, hi;
    round_share(n, kProbeRound, &lo, &hi);
    for (int64_t base = lo; base < hi; base += kProbeRound) {  // block-uniform; 64 bits: hi may be 2^31 - 1
        const bool in = base + threadIdx.x < hi;
        const int32_t i = in ? (int32_t)(base + threadIdx.x) : (int32_t)base;
        int t = find_seg32(s_pre, g.T, i);
        int64_t at = 0;
        int32_t row = 0, m = -1;
        // rows of one table (nearly every wave): its descriptor is read through scalar loads
        auto probe = [&](const DTable &tb) {
            at = s_ts[t] + (i - s_pre[t]);
            bool hit = false, pf = false;
            if (in) {
                row = g.U[at];
                const int32_t slot = find_slot(tb, row);
                hit = slot >= 0;
                if (hit) {
                    g.slotU[at] = slot;
                    tb.slot_touch[slot] = stamp;
                    pf = (tb.slot_flags[slot] & F_PF) != 0;
                }
            }
            wave_count_lds(hit, t, s_hits);  // counts only
            wave_count_lds(pf, t, s_hits_pf);
            m = wave_append(in && !hit, t, s_miss, 1);
        };
        const int t0 = __builtin_amdgcn_readfirstlane(t);
        if (__ballot(t != t0) == 0) probe(g.tabs[t0]);
        else probe(g.tabs[t]);
        __syncthreads();
        int *cnt = s_miss + threadIdx.x;  // counts -> first miss number of this round
        if ((int)threadIdx.x < g.T && *cnt) *cnt = atomicAdd(&g.st[threadIdx.x].mcount, *cnt);
        __syncthreads();
        if (m >= 0) {
            m += s_miss[t];
            const int64_t a = s_ts[t] + m;
            g.slotU[at] = -(m + 1);
            g.M[a] = row;
            g.mflags[a] = 0;
            g.mcbit[a] = 0;
        }
        __syncthreads();
        if ((int)threadIdx.x < g.T) *cnt = 0;
        __syncthreads();
    }
    if ((int)threadIdx.x < g.T) {
        if (s_hits[threadIdx.x]) atomicAdd(&g.st[threadIdx.x].hits, s_hits[threadIdx.x]);
        if (s_hits_pf[threadIdx.x]) atomicAdd(&g.st[threadIdx.x].hits_pf, s_hits_pf[threadIdx.x]);
    }
    if (!cover) return;
    __syncthreads();
    int *s_cov = s_hits;
    if ((int)threadIdx.x < g.T) {
        s_cov[threadIdx.x] = 0;
        s_ts[threadIdx.x] = g.pstart[threadIdx.x];
    }
    const int32_t np = lay_tables(g.T, [&](int t) { return g.st[t].pcount; }, s_pre, tmp);
    round_share(np, kProbeRound, &lo, &hi);
    for (int64_t base = lo; base < hi; base += kProbeRound) {
        int t = 0;
        bool hit = false;
        if (base + threadIdx.x < hi) {
            const int32_t i = (int32_t)(base + threadIdx.x);
            t = find_seg32(s_pre, g.T, i);
            const DTable &tb = g.tabs[t];
            const uint32_t pos = bm_pos(tb, g.PU[s_ts[t] + (i - s_pre[t])]);
            const uint4 rk = gload16(tb.rank + (pos >> 5));
            hit = (int32_t)rk.z == stamp && (rk.y >> (pos & 31) & 1u);
        }
        wave_count_lds(hit, t, s_cov);  // counts only
    }
    __syncthreads();
    if ((int)threadIdx.x < g.T && s_cov[threadIdx.x]) atomicAdd(&g.st[threadIdx.x].covered, s_cov[threadIdx.x]);
}

// inverse map: where every index's row lives (slot, or -(miss + 1)).  The pooled
// kernels make addresses of it themselves: an 8-byte address per index beside
// the location was 38 MB of the 3.2 million indices' traffic here and there.
__device__ __forceinline__ void src_share(const DGlobal &g, const int32_t *__restrict__ indices, int64_t n,
                                          int64_t first_block) {
    __shared__ int64_t s_start[RECMG_MAX_TABLES + 1];
    __shared__ const uint4 *s_rank[RECMG_MAX_TABLES];
    __shared__ int32_t s_ns[RECMG_MAX_TABLES], s_qb[RECMG_MAX_TABLES];
    for (int t = threadIdx.x; t <= g.T; t += blockDim.x) {
        s_start[t] = g.tstart[t];
        if (t < g.T) {
            s_rank[t] = g.tabs[t].rank;
            s_ns[t] = g.tabs[t].nsets;
            s_qb[t] = g.tabs[t].qbits;
        }
    }
    __syncthreads();
    // contiguous shares: a block meets one or two tables
    int64_t lo, hi;
    block_share(n, &lo, &hi, first_block);
    if (lo >= hi) return;
    int t = find_seg(s_start, g.T, lo);
    constexpr int Q = 4;
    for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += Q * kBlock) {
        int tq[Q];
        uint32_t pos[Q];
        uint4 rk[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t i = i0 + q * kBlock;
            if (i >= hi) break;
            while (i >= s_start[t + 1]) ++t;
            tq[q] = t;
            pos[q] = bm_pos(s_ns[t], s_qb[t], indices[i]);
            rk[q] = gload16(s_rank[t] + (pos[q] >> 5));
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (i0 + q * kBlock >= hi) break;
            const int32_t u = (int32_t)rk[q].x + __popc(rk[q].y & ((1u << (pos[q] & 31)) - 1u));
            g.src[i0 + q * kBlock] = g.slotU[s_start[tq[q]] + u];
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_fwd_src(DGlobal g, const int32_t *__restrict__ indices, int64_t n) {
    if (!block_err(g)) src_share(g, indices, n, 0);
}

// Publishes the forward's counters; log_slot >= 0: also as that call's record
// of the stats log (the placement group of the record stays zero).
__device__ __forceinline__ void publish_forward(const DGlobal &g, int64_t log_slot) {
    for (int t = threadIdx.x; t < g.T; t += blockDim.x) {
        TState &st = g.st[t];
        const DTable &tb = g.tabs[t];
        int64_t v[kFwdStats];
        v[0] = g.tstart[t + 1] - g.tstart[t];
        v[1] = st.ucount;
        v[2] = st.hits;
        v[3] = st.hits_pf;
        v[4] = st.mcount;
        v[5] = (int64_t)st.mcount * tb.row_bytes;
        v[6] = st.covered;
        for (int k = 0; k < kFwdStats; ++k) {
            st.last[k] = v[k];
            st.total[k] += v[k];
        }
        if (log_slot >= 0) {
            int64_t *rec = g.stat_log + (log_slot * g.T + t) * (kNumStats + 1);
            for (int k = 0; k <= kNumStats; ++k) rec[k] = k < kFwdStats ? v[k] : 0;
        }
    }
}

// ----------------------------------------------------------------- miss fetch

// ZERO_COPY miss fetch: each distinct miss of a zero-copy table is read once
// from pinned host memory (device-visible mapping) and written to its staging
// row (STAGED tables' misses are staged by the host).  The block after the
// copying ones publishes the forward's counters, which are complete before this
// kernel starts: that costs no launch of its own (k_fwd_finalize took 3.4 us and a
// dispatch after the pooled kernel of every forward).  n > 0: the blocks after
// that one write the n locations (k_fwd_src's work), which then hides behind the
// host link's time (a step of 8 32-way LFU tables of 25,000
// indices 172 -> 164 us, a forward of 655,000 fp32 indices 434 -> 423), or, where
// the host gathers every table's rows, behind that.
#ifndef RECMG_FETCH_BLOCKS
#define RECMG_FETCH_BLOCKS 96
#endif
#ifndef RECMG_FETCH_BLOCKS_HUGE
#define RECMG_FETCH_BLOCKS_HUGE 288
#endif
constexpr int64_t kHugeFetchUnits = int64_t(1) << 25;  // 512 MiB in 16-byte units
__global__ void __launch_bounds__(kBlock) k_fetch(DGlobal g, int64_t log_slot, int32_t nb,
                                                  const int32_t *__restrict__ indices, int64_t n) {
    if (block_err(g)) return;
    if ((int32_t)blockIdx.x > nb) {  // block-uniform
        src_share(g, indices, n, nb + 1);
        return;
    }
    if ((int32_t)blockIdx.x == nb) {  // block-uniform
        publish_forward(g, log_slot);
        return;
    }
    copy_flat(
        g, [&](int t) { return g.tabs[t].staged ? 0 : g.st[t].mcount; },
        [&](int64_t units) { return units >= kHugeFetchUnits ? nb : nb < RECMG_FETCH_BLOCKS ? nb : RECMG_FETCH_BLOCKS; },
        [&](int t, const DTable &tb, int64_t j) {
            return tb.host + (int64_t)g.M[g.tstart[t] + j] * tb.row_bytes;
        },
        [&](int t, const DTable &tb, int64_t j) { return g.staging + (g.tstart[t] + j) * g.stage_stride; });
}

// ----------------------------------------------------------------- pooling

template <int DT>
struct Elem;
template <>
struct Elem<RECMG_F32> {
    static constexpr int bytes = 4;
    __device__ static float widen(uint32_t x) { return __builtin_bit_cast(float, x); }
};
template <>
struct Elem<RECMG_F16> {
    static constexpr int bytes = 2;
    __device__ static float widen(uint32_t x) { return f16_to_f32(x & 0xffffu); }
};
template <>
struct Elem<RECMG_BF16> {
    static constexpr int bytes = 2;
    __device__ static float widen(uint32_t x) { return bf16_to_f32(x & 0xffffu); }
};

// 16-byte vector of elements -> VE floats added into acc
template <int DT>
__device__ __forceinline__ void accum_vec(float *acc, const uint4 v) {
    if constexpr (DT == RECMG_F32) {
        acc[0] += __builtin_bit_cast(float, v.x);
        acc[1] += __builtin_bit_cast(float, v.y);
        acc[2] += __builtin_bit_cast(float, v.z);
        acc[3] += __builtin_bit_cast(float, v.w);
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (DT == RECMG_BF16) {
                acc[2 * k] += __builtin_bit_cast(float, w[k] << 16);
                acc[2 * k + 1] += __builtin_bit_cast(float, w[k] & 0xffff0000u);
            } else {
                acc[2 * k] += f16_to_f32(w[k] & 0xffffu);
                acc[2 * k + 1] += f16_to_f32(w[k] >> 16);
            }
        }
    }
}

template <int DT, bool VEC>
struct Lane {
    static constexpr int VE = VEC ? 16 / Elem<DT>::bytes : 1;
    using V = typename std::conditional<VEC, uint4, typename std::conditional<Elem<DT>::bytes == 4, uint32_t,
                                                                               uint16_t>::type>::type;
    __device__ static V load(const char *p) {
        if constexpr (VEC) return gload16(p);
        else if constexpr (Elem<DT>::bytes == 4) return gload4(p);
        else return gload2(p);
    }
    __device__ static void add(float *acc, const V v) {
        if constexpr (VEC) accum_vec<DT>(acc, v);
        else acc[0] += Elem<DT>::widen((uint32_t)v);
    }
};

// One group of G lanes sums one bag.  Lookup p of the bag goes to
// accumulator p mod 4; the four partial sums are combined pairwise at the end.
// The order is fixed per bag, so the result does not depend on which tier
// served each row.  The group keeps up to 16 row loads in flight and loads the
// next chunk of locations while the current chunk's rows are in flight.
template <int DT, bool VEC>
__device__ __forceinline__ void pool_table(const DGlobal &g, const DTable &tb, int t, int32_t B,
                                           const int64_t *__restrict__ offsets, float *__restrict__ out,
                                           int blk_in_table) {
    using L = Lane<DT, VEC>;
    using V = typename L::V;
    constexpr int VE = L::VE;
    constexpr int EB = Elem<DT>::bytes;
#ifndef RECMG_POOL_UNROLL
#define RECMG_POOL_UNROLL 8
#endif
#ifndef RECMG_POOL_UNROLL_HALF
#define RECMG_POOL_UNROLL_HALF 8
#endif
    // row loads in flight per group (fp32 / 2-byte storage): measured best on
    // gfx950, where more depth costs more in occupancy than it gains
    constexpr int UNROLL = EB == 4 ? RECMG_POOL_UNROLL : RECMG_POOL_UNROLL_HALF;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int G = tb.gsz;
    const int gl = lane & (G - 1);
    const int gi = lane / G;
    const int bpw = 64 / G;
    const int j = (blk_in_table * (kBlock / 64) + wave) * bpw + gi;
    if (j >= B) return;
    const int64_t a = offsets[(int64_t)t * B + j], e = offsets[(int64_t)t * B + j + 1];
    const int D = tb.dim;
    const int64_t rb = tb.row_bytes;
    const char *__restrict__ pool = tb.pool;
    const int64_t sstride = g.stage_stride;
    const char *__restrict__ stg = g.staging + g.tstart[t] * sstride;
    const int32_t *__restrict__ src = g.src;
    float *orow = out + (int64_t)B * tb.out_elem_off + (int64_t)j * D;

    for (int ch = 0; ch < tb.nchunk; ++ch) {
        const int e0 = (ch * G + gl) * VE;
        const bool lane_ok = e0 < D;
        const int64_t eoff = lane_ok ? (int64_t)e0 * EB : 0;
        // slot s >= 0: the HBM pool; s < 0: staging row -(s + 1); no branch
        auto row_ptr = [&](int s) -> const char * {
            const bool hit = s >= 0;
            const char *base = hit ? pool : stg;
            const int64_t idx = hit ? s : -(int64_t)s - 1;
            return base + idx * (hit ? rb : sstride) + eoff;
        };
        float acc[4][VE];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int x = 0; x < VE; ++x) acc[k][x] = 0.f;

        int my = (a + gl < e) ? (int)gload4(src + a + gl) : 0;
        for (int64_t c = a; c < e; c += G) {
            const int n = (int)((e - c) < G ? (e - c) : G);
            const int nxt = (c + G + gl < e) ? (int)gload4(src + c + G + gl) : 0;  // next chunk, in flight meanwhile
            int q = 0;
            for (; q + UNROLL <= n; q += UNROLL) {
                int sv[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) sv[u] = __shfl(my, q + u, G);
                V v[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) v[u] = L::load(row_ptr(sv[u]));
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) L::add(acc[u & 3], v[u]);
            }
            for (; q < n; q += 4) {
                int sv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) sv[u] = __shfl(my, q + u < n ? q + u : q, G);
                V v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (q + u < n) v[u] = L::load(row_ptr(sv[u]));
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (q + u < n) L::add(acc[u], v[u]);
            }
            my = nxt;
        }
        if (lane_ok) {
            float r[VE];
#pragma unroll
            for (int x = 0; x < VE; ++x) r[x] = (acc[0][x] + acc[1][x]) + (acc[2][x] + acc[3][x]);
            float *o = orow + e0;
            if (VE % 4 == 0 && (((uintptr_t)o) & 15) == 0) {
#pragma unroll
                for (int x = 0; x < VE; x += 4)
                    *reinterpret_cast<float4 *>(o + x) = make_float4(r[x], r[x + 1], r[x + 2], r[x + 3]);
            } else {
#pragma unroll
                for (int x = 0; x < VE; ++x) o[x] = r[x];
            }
        }
    }
}

// Workgroups are dealt round-robin to the 8 XCDs; give each XCD one
// contiguous range of a launch's blocks so a table's hot rows stay in one L2.
__device__ __forceinline__ int xcd_block(int nb) {
#ifndef RECMG_POOL_NO_XCD_MAP
    const int x = (int)blockIdx.x & 7, q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + ((int)blockIdx.x >> 3);
#else
    return (int)blockIdx.x;
#endif
}

// Group-per-bag kernel for the tables the wave-per-bag kernel does not take.
// Each launch covers the blocks [boff, boff + nblk) of one class; block lb
// belongs to table btab[k] for the k with bstart[k] <= lb < bstart[k + 1].
template <int DT, bool VEC>
__global__ void __launch_bounds__(kBlock) k_pool(DGlobal g, const int64_t *__restrict__ offsets, int32_t B,
                                                 float *__restrict__ out, const int32_t *__restrict__ bstart,
                                                 const int32_t *__restrict__ btab, int32_t nt, int32_t boff,
                                                 int32_t nblk) {
    const int lb = boff + xcd_block(nblk);
    __shared__ int s_k, s_err;  // the error word is read once per block (block_err)
    if (threadIdx.x == 0) {
        s_err = *g.err;
        s_k = find_seg32(bstart, nt, lb);
    }
    __syncthreads();
    if (s_err) return;  // block-uniform
    const int k = s_k, t = btab[k];
    pool_table<DT, VEC>(g, g.tabs[t], t, B, offsets, out, lb - bstart[k]);
}

// ------------------------------------------------- wave-per-bag pooled sum
//
// One wave sums kWaveBags consecutive bags, one bag at a time.  Each lane
// adds its LW-byte slice of every row; a row's address comes from its index's
// location, written before it, so the kernel does no lookups.
//   R == 1 (rows of 1024 bytes or whole multiples): all lanes read the same
//     row, so its address is wave-uniform and comes in through scalar loads.
//   R > 1 (shorter rows): the wave splits into R groups of 64 / R lanes that
//     read R different rows per load instruction, group h taking the lookups
//     p with p mod R = h.  Each lane makes one address of a window of 64
//     lookups; a ds_bpermute hands every group its row's address.
// Either way lookup p goes to partial sum p mod 4 and the four are combined
// as (S0 + S1) + (S2 + S3): a fixed order per bag, whichever tier served a row.

template <int LW>
struct WVec;
template <>
struct WVec<4> {
    using V = uint32_t;
    __device__ static void words(const V v, uint32_t *w) { w[0] = v; }
};
template <>
struct WVec<8> {
    using V = u32x2_t;
    __device__ static void words(const V v, uint32_t *w) {
        w[0] = v.x;
        w[1] = v.y;
    }
};
template <>
struct WVec<16> {
    using V = u32x4_t;
    __device__ static void words(const V v, uint32_t *w) {
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    }
};

// acc + the fp16 value in the low / high half of w: one mixed-precision FMA
// (x * 1 + acc) converts exactly and rounds once, like convert-then-add
__device__ __forceinline__ float add_f16_lo(float acc, uint32_t w) {
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(acc));
    return r;
}
__device__ __forceinline__ float add_f16_hi(float acc, uint32_t w) {
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(acc));
    return r;
}

template <int DT, int LW>
__device__ __forceinline__ void wadd(float *acc, const typename WVec<LW>::V v) {
    uint32_t w[LW / 4];
    WVec<LW>::words(v, w);
#pragma unroll
    for (int k = 0; k < LW / 4; ++k) {
        if constexpr (DT == RECMG_F32) {
            acc[k] += __builtin_bit_cast(float, w[k]);
        } else if constexpr (DT == RECMG_BF16) {
            acc[2 * k] += __builtin_bit_cast(float, w[k] << 16);
            acc[2 * k + 1] += __builtin_bit_cast(float, w[k] & 0xffff0000u);
        } else {
            acc[2 * k] = add_f16_lo(acc[2 * k], w[k]);
            acc[2 * k + 1] = add_f16_hi(acc[2 * k + 1], w[k]);
        }
    }
}

// LW-byte load at global address base + off
template <class V>
__device__ __forceinline__ V wload(uint64_t base, uint32_t off) {
    typedef const __attribute__((address_space(1))) char gchar;
    return *(const __attribute__((address_space(1))) V *)((gchar *)base + off);
}

// The lane offset is passed through an empty asm in every block of loads so
// that its zero extension is visible where the loads are selected: a uniform
// 64-bit base plus a 32-bit lane offset then becomes the scalar-base form of
// global_load, with no vector address arithmetic at all.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Combine the NA partial sums of each of the R groups in the order
// (S0 + S1) + (S2 + S3) and store the bag's NE floats of this lane (group 0).
template <int NE, int R, int NA>
__device__ __forceinline__ void wstore(float (&acc)[NA][NE], int h, float *o) {
    float r[NE];
#pragma unroll
    for (int x = 0; x < NE; ++x) {
        if constexpr (R == 1) {
            r[x] = (acc[0][x] + acc[1][x]) + (acc[2][x] + acc[3][x]);
        } else if constexpr (R == 2) {
            // group 0 holds S0, S2 and group 1 holds S1, S3
            const float o0 = __shfl_xor(acc[0][x], 32), o1 = __shfl_xor(acc[1][x], 32);
            r[x] = (acc[0][x] + o0) + (acc[1][x] + o1);
        } else {
            // group h holds S_h
            const float s01 = acc[0][x] + __shfl_xor(acc[0][x], 16);
            r[x] = s01 + __shfl_xor(s01, 32);
        }
    }
    if (h != 0) return;
    // a table's output block starts at B * (sum of the earlier dims) floats,
    // so vector stores need a run-time alignment check
    const uintptr_t oa = reinterpret_cast<uintptr_t>(o);
    if (NE % 4 == 0 && (oa & 15) == 0) {
#pragma unroll
        for (int x = 0; x + 3 < NE; x += 4)
            *reinterpret_cast<float4 *>(o + x) = make_float4(r[x], r[x + 1], r[x + 2], r[x + 3]);
    } else if (NE == 2 && (oa & 7) == 0) {
        *reinterpret_cast<float2 *>(o) = make_float2(r[0], r[NE - 1]);
    } else {
#pragma unroll
        for (int x = 0; x < NE; ++x) o[x] = r[x];
    }
}

// the bag offsets of the wave's bags, clamped to the last one present
template <int BPW>
__device__ __forceinline__ void wave_offsets(int64_t (&offs)[BPW + 1], const int64_t *__restrict__ ob, int nbags) {
#pragma unroll
    for (int b = 0; b <= BPW; ++b) offs[b] = ob[b < nbags ? b : nbags];
}

// A table's rows: slot s >= 0 in the slot pool, s < 0 staging row -(s + 1).
struct Rows {
    uint64_t pool, staging;  // addresses of slot 0 and of the table's first staging row
    uint32_t row_bytes, stride;
    __device__ uint64_t at(int32_t s) const {
        const bool hit = s >= 0;
        return (hit ? pool : staging) + (uint64_t)(uint32_t)(hit ? s : ~s) * (hit ? row_bytes : stride);
    }
};
__device__ __forceinline__ Rows table_rows(const DGlobal &g, const DTable &tb, int64_t tstart) {
    Rows r;
    r.pool = (uint64_t)tb.pool;
    r.staging = (uint64_t)(g.staging + tstart * g.stage_stride);
    r.row_bytes = (uint32_t)tb.row_bytes;
    r.stride = (uint32_t)g.stage_stride;
    return r;
}

// R == 1.  Software pipeline: the scalar loads of the next block's U row
// locations (this bag's, else the next non-empty bag's first) are in flight
// while the current block's row loads are.  A block may run past the bag and
// past the batch (the location array has kSrcPad entries of padding); the
// addresses made of such entries are never dereferenced.
template <int DT, int LW>
__device__ __forceinline__ void pool_wave_s(const int32_t *__restrict__ src, const Rows rows,
                                            const int64_t *__restrict__ ob, int nbags, int wnch, int D,
                                            float *__restrict__ obase) {
    using V = typename WVec<LW>::V;
    constexpr int EB = Elem<DT>::bytes, NE = LW / EB;
    constexpr int U = 8;  // rows in flight per wave (8 KB)
    constexpr int BPW = kWaveBags;
    const int lane = threadIdx.x & 63;
    int64_t offs[BPW + 1];
    wave_offsets<BPW>(offs, ob, nbags);
    for (int ch = 0; ch < wnch; ++ch) {
        const uint32_t eoff = (uint32_t)((ch * 64 + lane) * LW);
        int32_t nx[U];
        // first block of the first non-empty bag after bag b (all indices
        // static, so offs and nx stay in scalar registers)
        auto next_bag_addrs = [&](int b) {
            bool found = false;
#pragma unroll
            for (int b2 = 0; b2 < BPW; ++b2)
                if (b2 > b && !found && b2 < nbags && offs[b2 + 1] > offs[b2]) {
#pragma unroll
                    for (int k = 0; k < U; ++k) nx[k] = src[offs[b2] + k];
                    found = true;
                }
        };
        next_bag_addrs(-1);
#pragma unroll
        for (int b = 0; b < BPW; ++b) {
            if (b >= nbags) continue;
            const int64_t a = offs[b];
            const int n = (int)(offs[b + 1] - a);
            float acc[4][NE];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int x = 0; x < NE; ++x) acc[k][x] = 0.f;
            int p = 0;
            for (; p + U <= n; p += U) {
                V v[U];
                const uint32_t eo = opaque(eoff);
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = wload<V>(rows.at(nx[u]), eo);
                // the barrier keeps the next block's scalar loads after the
                // row loads above, so one block of addresses is live at a time
                asm volatile("" ::: "memory");
                if (p + U < n) {
#pragma unroll
                    for (int k = 0; k < U; ++k) nx[k] = src[a + p + U + k];
                } else {
                    next_bag_addrs(b);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) wadd<DT, LW>(acc[u & 3], v[u]);
            }
            if (p < n) {
                // partial block, in quads of loads; a lookup past the bag's end
                // re-reads the quad's first row and is not added
                V v[U];
#pragma unroll
                for (int q = 0; q < U; q += 4)
                    if (p + q < n) {
                        const uint32_t eo = opaque(eoff);
#pragma unroll
                        for (int u = q; u < q + 4; ++u) v[u] = wload<V>(rows.at(p + u < n ? nx[u] : nx[q]), eo);
                    }
                asm volatile("" ::: "memory");
                next_bag_addrs(b);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (p + u < n) wadd<DT, LW>(acc[u & 3], v[u]);
            }
            wstore<NE, 1, 4>(acc, 0, obase + (int64_t)b * D + ch * 64 * NE + lane * NE);
        }
    }
}

#ifndef RECMG_WPOOL_KB
#define RECMG_WPOOL_KB 8
#endif

// R > 1.  Lane i holds the address of lookup w + i of a window of 64 lookups
// of the bag starting at w (a whole bag when it has at most 64); the next
// window's locations (this bag's, else the next non-empty bag's first) are loaded
// while the current one's rows are read.  Window entries past the bag, and past
// the batch (kSrcPad entries of padding), are never dereferenced.
template <int DT, int LW, int R>
__device__ __forceinline__ void pool_wave_v(const int32_t *__restrict__ src, const Rows rows,
                                            const int64_t *__restrict__ ob, int nbags, int D,
                                            float *__restrict__ obase) {
    using V = typename WVec<LW>::V;
    constexpr int EB = Elem<DT>::bytes, NE = LW / EB, GL = 64 / R, NA = 4 / R;
    constexpr int U0 = RECMG_WPOOL_KB * 16 / LW;  // load instructions per sub-block (KB of rows in flight)
    constexpr int U = U0 * R > 64 ? 64 / R : U0;  // a sub-block stays inside its window
    constexpr int UR = U * R;                    // lookups per sub-block, divides 64
    static_assert(64 % UR == 0 && U % NA == 0, "sub-blocks tile a window; slot = u mod NA");
    constexpr int BPW = kWaveBags;
    const int lane = threadIdx.x & 63, h = lane / GL, gl = lane % GL;
    const uint32_t eoff = (uint32_t)(gl * LW);
    int64_t offs[BPW + 1];
    wave_offsets<BPW>(offs, ob, nbags);
    int32_t wnext = 0;
    auto next_bag_window = [&](int b) {
        bool found = false;
#pragma unroll
        for (int b2 = 0; b2 < BPW; ++b2)
            if (b2 > b && !found && b2 < nbags && offs[b2 + 1] > offs[b2]) {
                wnext = RECMG_GLOBAL(int32_t, src + offs[b2] + lane);
                found = true;
            }
    };
    next_bag_window(-1);
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
        if (b >= nbags) continue;
        const int64_t a = offs[b];
        const int n = (int)(offs[b + 1] - a);
        float acc[NA][NE];
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int x = 0; x < NE; ++x) acc[k][x] = 0.f;
        for (int p = 0; p < n; p += 64) {
            const uint64_t wcur = rows.at(wnext);
            const int m = n - p < 64 ? n - p : 64;  // lookups in this window
            const int wlo = (int)(uint32_t)wcur, whi = (int)(uint32_t)(wcur >> 32);
            // one sub-block of U load instructions; FULL: all UR lookups are
            // in the bag (no masking).  The two forms are separate code paths
            // so that no loaded value has to be merged (and waited for) early.
            auto sub_block = [&](int s, auto full_tag) {
                constexpr bool FULL = decltype(full_tag)::value;
                V v[U];
                const int bidx = (s + h) * 4;  // bpermute byte index of lookup s + h
                if constexpr (FULL) {
                    uint32_t lo[U], hi[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        lo[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(bidx + u * R * 4, wlo);
                        hi[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(bidx + u * R * 4, whi);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = wload<V>(((uint64_t)hi[u] << 32) | lo[u], eoff);
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (s + u * R < m) {
                            const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(bidx + u * R * 4, wlo);
                            const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(bidx + u * R * 4, whi);
                            if (s + u * R + h < m) v[u] = wload<V>(((uint64_t)hi << 32) | lo, eoff);
                        }
                }
                if (s == 0) {
                    // the next window, issued after this sub-block's row loads
                    asm volatile("" ::: "memory");
                    if (p + 64 < n) wnext = RECMG_GLOBAL(int32_t, src + a + p + 64 + lane);
                    else next_bag_window(b);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (FULL || s + u * R + h < m) wadd<DT, LW>(acc[u % NA], v[u]);
            };
            int s = 0;
            for (; s + UR <= m; s += UR) sub_block(s, std::true_type{});
            if (s < m) sub_block(s, std::false_type{});
        }
        wstore<NE, R, NA>(acc, h, obase + (int64_t)b * D + gl * NE);
    }
}

#ifndef RECMG_WPOOL_OCC
#define RECMG_WPOOL_OCC 1
#endif

// RECMG_WPOOL_OCC: waves per SIMD the register allocation must allow
// nbt > 0: every table of the launch has nbt blocks, so block lb belongs to
// table btab[k0 + (lb - boff) / nbt] (no search; one wave's prologue is a
// chain of dependent loads, and the search would add four to it).
template <int DT, int LW, int R>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(RECMG_WPOOL_OCC))) k_pool_w(DGlobal g, const int64_t *__restrict__ offsets,
                                                   const int32_t *__restrict__ src, int32_t B,
                                                   float *__restrict__ out, const int32_t *__restrict__ bstart,
                                                   const int32_t *__restrict__ btab, int32_t nt, int32_t boff,
                                                   int32_t nblk, int32_t k0, int32_t nbt) {
    const int lb = boff + xcd_block(nblk);
    int k, b0;
    if (nbt > 0) {
        k = k0 + (lb - boff) / nbt;
        b0 = boff + (k - k0) * nbt;
    } else {
        k = find_seg32(bstart, nt, lb);
        b0 = bstart[k];
    }
    const int t = btab[k];
    const int err = *g.err;
    const DTable &tb = g.tabs[t];
    const int D = tb.dim;
    const int64_t ooff = (int64_t)B * tb.out_elem_off;
    if (err) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int j0 = ((lb - b0) * (kBlock / 64) + wave) * kWaveBags;
    if (j0 >= B) return;
    const int nbags = B - j0 < kWaveBags ? B - j0 : kWaveBags;
    const int64_t *ob = offsets + (int64_t)t * B + j0;
    float *ob_out = out + ooff + (int64_t)j0 * D;
    const Rows rows = table_rows(g, tb, offsets[(int64_t)t * B]);
    if constexpr (R == 1) pool_wave_s<DT, LW>(src, rows, ob, nbags, tb.wnch, D, ob_out);
    else pool_wave_v<DT, LW, R>(src, rows, ob, nbags, D, ob_out);
}

// The pooled sums of tables of several kinds in one launch: a block takes its
// table's own form.  For batches of few bags, where a launch per kind leaves most
// of the chip idle each time (13 tables of five kinds with 1,000 bags each: 29 us
// in five launches, 15 in one); the registers of the largest form would cost the
// others waves where there are many.
template <int DT>
__device__ __forceinline__ void pool_any(const DGlobal &g, const DTable &tb, int t, int32_t B,
                                         const int64_t *__restrict__ offsets, const int32_t *__restrict__ src,
                                         float *__restrict__ out, int blk) {
    if (!tb.wlw) {
        if (tb.vec) pool_table<DT, true>(g, tb, t, B, offsets, out, blk);
        else pool_table<DT, false>(g, tb, t, B, offsets, out, blk);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int j0 = (blk * (kBlock / 64) + wave) * kWaveBags;
    if (j0 >= B) return;
    const int nbags = B - j0 < kWaveBags ? B - j0 : kWaveBags, D = tb.dim;
    const int64_t *ob = offsets + (int64_t)t * B + j0;
    float *o = out + (int64_t)B * tb.out_elem_off + (int64_t)j0 * D;
    const Rows rows = table_rows(g, tb, offsets[(int64_t)t * B]);
    if (tb.wlw == 4) pool_wave_v<DT, 4, 4>(src, rows, ob, nbags, D, o);
    else if (tb.wlw == 8) pool_wave_v<DT, 8, 4>(src, rows, ob, nbags, D, o);
    else if (tb.wr == 4) pool_wave_v<DT, 16, 4>(src, rows, ob, nbags, D, o);
    else if (tb.wr == 2) pool_wave_v<DT, 16, 2>(src, rows, ob, nbags, D, o);
    else pool_wave_s<DT, 16>(src, rows, ob, nbags, tb.wnch, D, o);
}

__global__ void __launch_bounds__(kBlock) k_pool_any(DGlobal g, const int64_t *__restrict__ offsets,
                                                     const int32_t *__restrict__ src, int32_t B,
                                                     float *__restrict__ out, const int32_t *__restrict__ bstart,
                                                     const int32_t *__restrict__ btab, int32_t nt, int32_t nblk) {
    const int lb = xcd_block(nblk);
    __shared__ int s_k, s_err;  // the error word is read once per block (block_err)
    if (threadIdx.x == 0) s_err = *g.err;
    // (blocks of the tables in btab order; a table without blocks matches none)
    if ((int)threadIdx.x < nt && bstart[threadIdx.x] <= lb && lb < bstart[threadIdx.x + 1]) s_k = threadIdx.x;
    __syncthreads();
    if (s_err) return;  // block-uniform
    const int k = __builtin_amdgcn_readfirstlane(s_k);
    const int t = btab[k], blk = lb - bstart[k];
    const DTable &tb = g.tabs[t];
    if (tb.dtype == RECMG_F32) pool_any<RECMG_F32>(g, tb, t, B, offsets, src, out, blk);
    else if (tb.dtype == RECMG_F16) pool_any<RECMG_F16>(g, tb, t, B, offsets, src, out, blk);
    else pool_any<RECMG_BF16>(g, tb, t, B, offsets, src, out, blk);
}

// The counters of a forward of no indices (others publish in k_fetch).
__global__ void k_fwd_finalize(DGlobal g, int64_t log_slot) {
    if (*g.err) return;
    publish_forward(g, log_slot);
}

// ----------------------------------------------------------------- launchers

static inline unsigned grid_for(int64_t n, int per_block, unsigned cap) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > (int64_t)cap) b = cap;
    return (unsigned)b;
}

void launch_bag_offsets(const DGlobal &g, const int64_t *offsets, int32_t B, hipStream_t s) {
    const int64_t bags = (int64_t)g.T * B;
    if (B > kPrepBags) k_bag_offsets<<<grid_for(bags, kBlock * 4, 4096), kBlock, 0, s>>>(g, offsets, bags);
}

void launch_fwd_prep(const DGlobal &g, const int64_t *offsets, int32_t B, int64_t n, hipStream_t s) {
    k_fwd_prep<<<g.T, kBlock, 0, s>>>(g, offsets, B, n);
}

void launch_fwd_probe(const DGlobal &g, int32_t stamp, int64_t n, int64_t np, hipStream_t s) {
    // one round per block if all ids were distinct
    k_fwd_probe<<<grid_for(n > np ? n : np, kProbeRound, 8192), kProbeRound, 0, s>>>(g, stamp, np > 0 ? 1 : 0);
}

static unsigned src_blocks(int64_t n) { return grid_for(n, kBlock * items_per_thread(n, 4), 16384); }

void launch_fwd_src(const DGlobal &g, const int32_t *indices, int64_t n, hipStream_t s) {
    if (n > 0) k_fwd_src<<<src_blocks(n), kBlock, 0, s>>>(g, indices, n);
}

// As for the prefetch fill, which runs at the same time on the copy stream: a
// modest grid fills the host link and leaves most CUs' L1s to other kernels
// (the next placement runs beside it).  Measured on configuration 3 (64-256
// blocks): 96 is best with 32-way sets (k_sa_place's critical path runs
// alongside) and within 1% of the best without prefetch.  From 512 MiB on the
// fetch shares the link with a large fill for most of a step and takes
// RECMG_FETCH_BLOCKS_HUGE.  Configuration 5 with 768 fill blocks, ms per step, fully
// associative (750 MB fetched beside a 3.8 GB fill) and with 32-way sets (more
// fetched than filled): 96 blocks 83.4 and 42.2, 112 82.4 .. 84.6 and 42.7, 160 82.2
// and 43.5, 224 82.4 and 42.5, 256 82.4 .. 82.9 and 42.0, 288 82.4 and 41.7.  (A step
// that fetches some 270 MB: 7.49 ms with larger counts, 7.31 with 96 and 512.)  The
// kernel knows how much it copies; the grid holds the larger count.
void launch_fetch(const DGlobal &g, bool copies, int64_t log_slot, const int32_t *indices, int64_t n, hipStream_t s,
                  hipEvent_t ev0, hipEvent_t ev1) {
    const int32_t nb = copies ? RECMG_FETCH_BLOCKS_HUGE : 0;
    const dim3 grid(nb + 1 + (n > 0 ? src_blocks(n) : 0));
    if (ev0 || ev1) hipExtLaunchKernelGGL(k_fetch, grid, dim3(kBlock), 0, s, ev0, ev1, 0, g, log_slot, nb, indices, n);
    else k_fetch<<<grid, kBlock, 0, s>>>(g, log_slot, nb, indices, n);
}

int pool_kind(int dtype, int vec, int wlw, int wr) {
    if (wlw == 0) return dtype * 2 + vec;
    const int v = wlw == 16 ? (wr == 1 ? 0 : wr == 2 ? 1 : 2) : wlw == 8 ? 3 : 4;
    return kPoolKindsGroup + dtype * 5 + v;
}

// Blocks up to which tables of several kinds share a launch.  12 tables of four
// kinds, whole forwards: 512 bags each (1,536 blocks) 42 us shared, 57 apart;
// 2,048 bags (6,144 blocks) 63 and 59; 8,192 bags 162 and 116.
#ifndef RECMG_POOL_ANY
#define RECMG_POOL_ANY 3072
#endif

// ev0 / ev1 (may be null): recorded by the first / last dispatch itself, so
// they bracket the kernels' execution without the dispatch gap.
void launch_pool(const DGlobal &g, const int64_t *offsets, int32_t B, float *out, const int32_t *bstart,
                 const int32_t *btab, int32_t nt, const PoolLaunch *ls, int nl, hipEvent_t ev0, hipEvent_t ev1,
                 hipStream_t s) {
    using KG = void (*)(DGlobal, const int64_t *, int32_t, float *, const int32_t *, const int32_t *, int32_t,
                        int32_t, int32_t);
    using KW = void (*)(DGlobal, const int64_t *, const int32_t *, int32_t, float *, const int32_t *,
                        const int32_t *, int32_t, int32_t, int32_t, int32_t, int32_t);
    static const KG kg[kPoolKindsGroup] = {k_pool<RECMG_F32, false>,  k_pool<RECMG_F32, true>,
                                           k_pool<RECMG_F16, false>,  k_pool<RECMG_F16, true>,
                                           k_pool<RECMG_BF16, false>, k_pool<RECMG_BF16, true>};
#define RECMG_WK(DT) k_pool_w<DT, 16, 1>, k_pool_w<DT, 16, 2>, k_pool_w<DT, 16, 4>, k_pool_w<DT, 8, 4>, k_pool_w<DT, 4, 4>
    static const KW kw[kPoolKinds - kPoolKindsGroup] = {RECMG_WK(RECMG_F32), RECMG_WK(RECMG_F16),
                                                        RECMG_WK(RECMG_BF16)};
#undef RECMG_WK
    int32_t blocks = 0;
    for (int i = 0; i < nl; ++i) blocks += ls[i].nblk;
    if (nl > 1 && blocks > 0 && blocks <= RECMG_POOL_ANY) {
        const dim3 grid((unsigned)blocks), blk(kBlock);
        const int32_t *ra = g.src;
        if (ev0 || ev1) hipExtLaunchKernelGGL(k_pool_any, grid, blk, 0, s, ev0, ev1, 0, g, offsets, ra, B, out, bstart, btab,
                                              nt, blocks);
        else k_pool_any<<<grid, blk, 0, s>>>(g, offsets, ra, B, out, bstart, btab, nt, blocks);
        return;
    }
    int first = -1, last = -1;
    for (int i = 0; i < nl; ++i)
        if (ls[i].nblk > 0) {
            if (first < 0) first = i;
            last = i;
        }
    for (int i = 0; i < nl; ++i) {
        const PoolLaunch &L = ls[i];
        if (L.nblk <= 0) continue;
        hipEvent_t a = i == first ? ev0 : nullptr, b = i == last ? ev1 : nullptr;
        const dim3 grid((unsigned)L.nblk), blk(kBlock);
        if (L.kind < kPoolKindsGroup) {
            const KG k = kg[L.kind];
            if (a || b) hipExtLaunchKernelGGL(k, grid, blk, 0, s, a, b, 0, g, offsets, B, out, bstart, btab, nt,
                                              L.boff, L.nblk);
            else k<<<grid, blk, 0, s>>>(g, offsets, B, out, bstart, btab, nt, L.boff, L.nblk);
        } else {
            const KW k = kw[L.kind - kPoolKindsGroup];
            const int32_t *ra = g.src;
            if (a || b) hipExtLaunchKernelGGL(k, grid, blk, 0, s, a, b, 0, g, offsets, ra, B, out, bstart, btab, nt,
                                              L.boff, L.nblk, L.k0, L.nbt);
            else k<<<grid, blk, 0, s>>>(g, offsets, ra, B, out, bstart, btab, nt, L.boff, L.nblk, L.k0, L.nbt);
        }
    }
}

void launch_fwd_finalize(const DGlobal &g, int64_t log_slot, hipStream_t s) {
    k_fwd_finalize<<<1, kBlock, 0, s>>>(g, log_slot);
}

}  // namespace recmg

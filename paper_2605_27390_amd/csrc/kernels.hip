// HIP kernels (gfx950 / CDNA4) for the active-vocabulary LM head of the EvoSpec paper:
// Eq. 1 (Softmax(h W_LM^T)) evaluated on the active set V_t of Eq. 3 / Algorithm 1, with the
// log-normaliser and the top-k of the draft phase fused in, plus the row insertion that
// keeps the compact matrix W_act in step with the dynamic buffer.
//
// Wavefronts are 64 wide.  The contraction uses v_mfma_f32_16x16x32_bf16 (bf16 in, fp32
// accumulate): the A operand is a 16-row group of W_act, the B operand 16 draft rows of h,
// so an accumulator register holds z[vocab row 4*(lane/16)+j][draft row lane%16].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include <type_traits>

#include "common.hpp"
#include "plan.hpp"
#include "slab.hpp"

namespace evospec {

// ---------------------------------------------------------------------------------------
// Row insertion  W_act[slot] <- W_lm[id], act_ids[slot] <- id  (bit copy, 16 B per lane).
// One workgroup per row.  Into a packed W_act the row's pieces go to their places in the operand
// tiles (16-byte stores 256 bytes apart) and the pieces between d and the padded row length are
// zeroed.  PAST: the stores bypass the caches (see update_past_caches).
template <bool PAST>
__device__ __forceinline__ void copy_row(const GatherArgs& g, int32_t id, int32_t s) {
    auto put = [](u32x4 v, u32x4* p) {
        if constexpr (PAST) __builtin_nontemporal_store(v, p);
        else *p = v;
    };
    const u32x4* src = static_cast<const u32x4*>(g.W_lm) + (size_t)id * g.row_vec;
    const int nt = blockDim.x;
    if (g.packed) {
        const int dp_vec = packed_d(g.row_vec * 8) / 8;
        u32x4* dst = static_cast<u32x4*>(g.W_act) + (size_t)(s >> 4) * (kPackRows * (size_t)dp_vec) + (s & 15);
        for (int c0 = 0; c0 < dp_vec; c0 += 4 * nt) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * nt + threadIdx.x;
                v[u] = u32x4{0u, 0u, 0u, 0u};
                if (c < g.row_vec) v[u] = src[c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * nt + threadIdx.x;
                if (c < dp_vec) put(v[u], dst + (c >> 2) * 64 + (c & 3) * 16);
            }
        }
    } else {
        u32x4* dst = static_cast<u32x4*>(g.W_act) + (size_t)s * g.row_vec;
        for (int c0 = 0; c0 < g.row_vec; c0 += 4 * nt) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * nt + threadIdx.x;
                if (c < g.row_vec) v[u] = src[c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = c0 + u * nt + threadIdx.x;
                if (c < g.row_vec) put(v[u], dst + c);
            }
        }
    }
}
__device__ __forceinline__ void gather_row(const GatherArgs& g, int32_t id, int32_t s) {
    if (id < 0 || id >= g.V || s < 0 || s >= g.V_act) return;      // uniform per workgroup
    if (g.past_caches) copy_row<true>(g, id, s);
    else copy_row<false>(g, id, s);
    if (threadIdx.x == 0) g.act_ids[s] = id;
}
__device__ __forceinline__ void gather_one_row(const GatherArgs& g, int i) {
    gather_row(g, g.src_ids[i], g.slots ? g.slots[i] : i);
}

// grid-stride over the n rows of the update
__global__ void __launch_bounds__(256)
gather_rows_kernel(GatherArgs g) {
    for (int i = blockIdx.x; i < g.n; i += gridDim.x) gather_one_row(g, i);
}

// A small update whose (slot, id) pairs travel in the kernel arguments: a caller that has them on
// the host (the failure event of Path A) needs no upload and no wait for one.
__global__ void __launch_bounds__(256)
gather_rows_inline_kernel(GatherArgs g, InlineRows r) {
    gather_row(g, r.id[blockIdx.x], r.slot[blockIdx.x]);
}

// Rebuild of a row-major W_act (slot i = i): four rows per workgroup and round, so that every lane has
// eight 16-byte loads in flight, and stores that bypass the cache (the rows are not read again soon;
// measured on MI355X for 36,864 rows of 8 KB: 95 us against 119 us with one row per round and cached
// stores).
__global__ void __launch_bounds__(256)
gather_rebuild_rows_kernel(GatherArgs g) {
    constexpr int RPB = 4;
    for (int i0 = blockIdx.x * RPB; i0 < g.n; i0 += gridDim.x * RPB) {
        const uint4* src[RPB];
        bool ok[RPB];
#pragma unroll
        for (int r = 0; r < RPB; ++r) {
            const int i = i0 + r;
            const int32_t id = i < g.n ? g.src_ids[i] : -1;
            ok[r] = id >= 0 && id < g.V && i < g.V_act;                   // uniform per workgroup
            src[r] = static_cast<const uint4*>(g.W_lm) + (size_t)(ok[r] ? id : 0) * g.row_vec;
            if (ok[r] && threadIdx.x == 0) g.act_ids[i] = id;
        }
        for (int c0 = 0; c0 < g.row_vec; c0 += 512) {
            u32x4 v[RPB][2];
#pragma unroll
            for (int r = 0; r < RPB; ++r)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = c0 + u * 256 + threadIdx.x;
                    if (ok[r] && c < g.row_vec) v[r][u] = *(gvec_ptr)(src[r] + c);
                }
#pragma unroll
            for (int r = 0; r < RPB; ++r)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int c = c0 + u * 256 + threadIdx.x;
                    if (ok[r] && c < g.row_vec)
                        __builtin_nontemporal_store(v[r][u], reinterpret_cast<u32x4*>(g.W_act) + (size_t)(i0 + r) * g.row_vec + c);
                }
        }
    }
}

// Rebuild of a packed W_act (slot i = i): one workgroup per tile of 16 slots, whole 128-byte lines on
// both sides.  Lane 8 r + p of a wavefront reads piece 8 q + p of row r (rows 0..7 of the tile in one
// load, rows 8..15 in a second one): 8 rows x 128 bytes per load.  Piece (row, c) belongs to operand
// block c / 4 at slot (c % 4) * 16 + row, so the eight lanes that hold the same piece of rows 0..7
// write 128 contiguous bytes.  The stores bypass the cache.  (Measured for 36,864 rows of 8 KB: 99 us
// against 129 us for half-line loads with cached stores.)
__global__ void __launch_bounds__(256)
gather_tiles_kernel(GatherArgs g) {
    constexpr int UNR = 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r8 = lane >> 3, p = lane & 7;
    const int dp_vec = packed_d(g.row_vec * 8) / 8;
    const int npairs = dp_vec / 8;                       // line pairs per row (dp_vec is a multiple of 32)
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    for (int t = blockIdx.x; t * kPackRows < g.n; t += gridDim.x) {
        const int ia = t * kPackRows + r8, ib = ia + 8;
        const int32_t ida = ia < g.n ? g.src_ids[ia] : -1, idb = ib < g.n ? g.src_ids[ib] : -1;
        const bool oka = ida >= 0 && ida < g.V && ia < g.V_act, okb = idb >= 0 && idb < g.V && ib < g.V_act;
        const uint4* sa = static_cast<const uint4*>(g.W_lm) + (size_t)(oka ? ida : 0) * g.row_vec;
        const uint4* sb = static_cast<const uint4*>(g.W_lm) + (size_t)(okb ? idb : 0) * g.row_vec;
        u32x4* d = reinterpret_cast<u32x4*>(g.W_act) + (size_t)t * (kPackRows * (size_t)dp_vec) + (p >> 2) * 64 + (p & 3) * 16 + r8;
        for (int q0 = w; q0 < npairs; q0 += 4 * UNR) {
            u32x4 va[UNR], vb[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int c = 8 * (q0 + 4 * u) + p;      // pieces past the row's end are zero padding
                va[u] = zero4; vb[u] = zero4;
                if (oka && c < g.row_vec) va[u] = *(gvec_ptr)(sa + c);
                if (okb && c < g.row_vec) vb[u] = *(gvec_ptr)(sb + c);
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int q = q0 + 4 * u;
                if (q < npairs) {
                    if (oka) __builtin_nontemporal_store(va[u], d + (size_t)q * 128);
                    if (okb) __builtin_nontemporal_store(vb[u], d + (size_t)q * 128 + 8);
                }
            }
        }
        if (w == 0 && p == 0) {
            if (oka) g.act_ids[ia] = ida;
            if (okb) g.act_ids[ib] = idb;
        }
    }
}

// ---------------------------------------------------------------------------------------
// Debug check of an id list: range and uniqueness (Eq. 3 is a set union).  O(n^2 / tile).
__device__ int g_validate_flag;

__global__ void __launch_bounds__(256)
validate_ids_kernel(const int32_t* __restrict__ ids, int n, int V, int* flag) {
    __shared__ int32_t tile[1024];
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int32_t mine = i < n ? ids[i] : -1;
    bool bad = i < n && (mine < 0 || mine >= V);
    for (int t0 = 0; t0 < n; t0 += 1024) {
        __syncthreads();
        for (int u = threadIdx.x; u < 1024; u += 256) tile[u] = (t0 + u < n) ? ids[t0 + u] : -2;
        __syncthreads();
        if (i < n) {
            for (int u = 0; u < 1024; ++u)
                if (tile[u] == mine && t0 + u != i) bad = true;
        }
    }
    if (bad) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------------------
// Wavefronts to a SIMD that the slab kernel's registers must leave room for: those of two workgroups to a compute unit, which launches of several rounds
// want, where 128 registers are nearly enough anyway (seven wavefronts of 132 cost the second one: packed, 24 rows, 51,446 x 512 26.7 us instead of
// 23.9, x 2,048 48.8 instead of 45.6.  One block of draft rows does without: nine wavefronts held to 96 70,000 x 5,120 at 8 rows 119.9, otherwise 117.5).
constexpr int slab_waves(int tw, int ks, int mb, bool packed, int segs) {
    if (ks == 1 && mb == 2 && (tw == 7 || tw == 8) && (packed || segs == 2)) return 4;
    return (tw * ks + 3) / 4;                          // (one workgroup)
}

// Pass 1 of the restricted head, one slab to a workgroup (slab.hpp).  Grid: (slabs, chunks of the batch, twice as many where
// their draft rows are split).  CORE: with a core beside the extensions (always front to back: KS and SEGS 1), one
// dimension: the core's slabs pass by pass, then the chunks'.  (Kernels of their own: as a case of one kernel, whose other launches then carried
// the core's arguments too, these lost up to 0.4 us: row-major 12,000 x 768 at 12 rows 15.9 and 16.3, packed 26,044 x 1,024 at 14 19.1 and 19.2.)
template <int TW, int KS, int RC, int MB, bool FULLK, bool PACKED, bool ONCE, int SEGS, bool CORE>
__global__ void __launch_bounds__(TW * KS * 64, slab_waves(TW, KS, MB, PACKED, SEGS))
lmhead_partials_kernel(const uint16_t* __restrict__ h_all, ChunkBatch cb, std::conditional_t<CORE, CoreSet, int> core_or_split, int seq_rows,
                       size_t chunk_keys, size_t chunk_stats, int d,
                       const uint16_t* __restrict__ W_all, const int32_t* __restrict__ ids_all,
                       int V_act, int k, int GL,
                       u64* __restrict__ keys_all, float2* __restrict__ stats_all) {
    static_assert(!CORE || (KS == 1 && SEGS == 1), "two sets: every logit's sum front to back");
    extern __shared__ __align__(16) unsigned char smem[];
    // this workgroup's problem: chunk `ci` of the batch (its draft rows, its sequence's
    // rows of a per-sequence matrix, its own piece of the partials), or a pass of the core
    // (split = 1: its draft rows go to two workgroups, the first kSplitRows and the others)
    constexpr bool kMaySplit = !CORE && MB == mb_for_rows(kSplitRows) && KS == 1;
    int slab = blockIdx.x, ci = blockIdx.y, row_first = 0;
    bool of_core = false;
    if constexpr (CORE) {
        of_core = slab < core_or_split.blocks;
        slab = of_core ? slab : slab - core_or_split.blocks;
        const int n = of_core ? core_or_split.n_slabs : core_or_split.chunk_slabs;
        ci = slab / n;
        slab -= ci * n;
    } else if constexpr (kMaySplit) {
        ci = blockIdx.y >> core_or_split;
        row_first = (blockIdx.y & core_or_split) * kSplitRows;
    }
    const int c_rows = cb.rows[of_core ? 0 : ci], c_m0 = cb.m0[of_core ? 0 : ci], c_seq = cb.seq[of_core ? 0 : ci];      // (asked for together)
    SlabProblem pr;
    if (CORE && of_core) {
        if constexpr (CORE) {
            const CoreSet& core = core_or_split;
            pr.rows = min(core.M - ci * kMTile, kMTile);
            pr.h = h_all + (size_t)ci * kMTile * d;
            pr.W = static_cast<const uint16_t*>(core.W);
            pr.ids = core.ids;
            pr.V_act = core.V;
            pr.keys = static_cast<u64*>(core.keys) + ci * core.pass_keys;
            pr.stats = static_cast<float2*>(core.stats) + ci * core.pass_stats;
        }
    } else {
        pr.rows = c_rows;
        if constexpr (kMaySplit) {
            if (core_or_split) pr.rows = min(pr.rows - row_first, kSplitRows);
            if (pr.rows <= 0) return;                                         // (uniform)
        }
        const size_t seq_row0 = (size_t)c_seq * seq_rows;
        pr.h = h_all + (size_t)(c_m0 + row_first) * d;
        // (a packed matrix pads every sequence's rows to whole tiles and its rows to whole chunks)
        pr.W = W_all + (PACKED ? (size_t)c_seq * packed_rows(seq_rows) * packed_d(d) : seq_row0 * d);
        pr.ids = ids_all ? ids_all + seq_row0 : nullptr;
        pr.V_act = V_act;
        pr.keys = keys_all + (size_t)ci * chunk_keys + row_first * k;
        pr.stats = stats_all + (size_t)ci * chunk_stats + row_first;
    }
    slab_partials<TW, KS, RC, MB, FULLK, PACKED, ONCE, SEGS>(pr, slab, d, k, GL, smem);
}

// ---------------------------------------------------------------------------------------
// Pass 2: one workgroup per draft row merges the slab partials:
//   logZ = M + log(sum_t s_t * exp(m_t - M)),  M = max_t m_t
//   top-k = the k largest of all slab candidates (keys are unique, so the order is total).
// Candidates come from up to two partial sets (a shared core and a per-sequence extension in the
// batched variant).
//
// The kernel is bound by latency, so it is built around ONE trip to memory: every thread fetches its
// candidates at once (the first kEager keys of a sorted list, or eight whole 16-byte pieces of the
// unsorted lists, which lie one after the other and are read a line at a time).  The largest of the
// 64 per-thread maxima of a wavefront, found bit by bit with ballots, give a bound that k candidates
// reach; what reaches it (some 20 keys of 2,560 at 256 lists of 10) goes to a list in LDS and is ranked
// by counting.  Only a thread whose last fetched key still reaches the bound goes back to memory.
// Measured on MI355X against ordering the list heads with sorting networks and reading the qualifying
// lists afterwards (a second trip): 60 rows x 256 lists of 10 7.3 -> 6.8 us, 37 x 251 of 20 11.8 -> 7.0,
// 60 x 950 of 10 19.3 -> 13.2, 960 x (256 unsorted + 15 sorted) 26.7 -> 14.8.  What is left at the
// first size: 1.4 us launch, 0.6 arguments, 2.0 memory, 0.6 bound, 2 exchange, ranking and stores.

// An unranked list slot holds (logit bits << 32) | id; all ones = empty.
__device__ __forceinline__ u64 pair_key(uint32_t zbits, uint32_t id) {
    return id == 0xffffffffu ? 0ull : make_key(__uint_as_float(zbits), (int32_t)id);
}

// The q-th largest (1 <= q <= 64) of the 64 keys of a wavefront: the largest value that q keys reach
// (0 if fewer than q lanes hold a key).  The high words first; when a single lane holds the word that
// was found, its key is the answer, else the low words decide among the lanes that share it.
__device__ __forceinline__ u64 wave_kth_key(u64 key, int q) {
    const uint32_t hi = (uint32_t)(key >> 32), lo = (uint32_t)key;
    uint32_t th = 0;
#pragma unroll
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t c = th | (1u << bit);
        if (__popcll(__ballot(hi >= c)) >= q) th = c;            // (uniform)
    }
    const u64 same = __ballot(hi == th);
    if (__popcll(same) == 1)
        return ((u64)th << 32) | (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)__builtin_ctzll(same));
    const int need = q - __popcll(__ballot(hi > th));            // >= 1: fewer than q lanes lie above th
    uint32_t tl = 0;
#pragma unroll
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t c = tl | (1u << bit);
        if (__popcll(__ballot(hi == th && lo >= c)) >= need) tl = c;
    }
    return ((u64)th << 32) | tl;
}

constexpr int kEager = 4;              // keys of a sorted list that a thread fetches up front
constexpr int kPieces = 8;             // 16-byte pieces (two slots) of unsorted lists, likewise

template <int NT>
__global__ void __launch_bounds__(NT)
lmhead_merge_kernel(PartialSet A, PartialSet B, ChunkBatch cb, size_t a_pass_keys, size_t a_pass_stats,
                    size_t b_chunk_keys, size_t b_chunk_stats, int k, int parts_log2, int deal, int pend_cap,
                    float* __restrict__ out_vals, int32_t* __restrict__ out_ids,
                    float* __restrict__ out_logz, GatherArgs upd) {
    // The blocks of grid row cb.n (present only when an update rides along) insert the rows of a
    // dynamic-buffer update into the compact matrix: the partials that this launch merges were
    // computed by an earlier launch, so nothing reads those rows any more.
    if ((int)blockIdx.y == cb.n) {
        if ((int)blockIdx.x < upd.n) gather_one_row(upd, blockIdx.x);
        return;
    }
    constexpr int NWV = NT / 64;
    extern __shared__ __align__(16) unsigned char merge_smem[];
    u64* pend = reinterpret_cast<u64*>(merge_smem);      // candidates that reach the bound
    __shared__ u64 run[kKMax];                           // the k best of earlier rounds, descending
    __shared__ u64 wave_tau[NWV];
    __shared__ float wave_m[NWV], wave_s[NWV];
    __shared__ int npend, count_s;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // row blockIdx.x of chunk blockIdx.y: where its partials sit in the two sets
    const int chunk = blockIdx.y;
    if ((int)blockIdx.x >= cb.rows[chunk]) return;                 // uniform: the grid spans the longest chunk
    const int out_row = cb.m0[chunk] + blockIdx.x;
    const int slotA = A.row_base + cb.a_slot[chunk] + blockIdx.x, slotB = B.row_base + blockIdx.x;
    const u64* keysA = A.keys + (size_t)cb.a_pass[chunk] * a_pass_keys + (size_t)slotA * A.key_row;
    const u64* keysB = B.keys + (size_t)chunk * b_chunk_keys + (size_t)slotB * B.key_row;
    const float2* statsA = A.stats + (size_t)cb.a_pass[chunk] * a_pass_stats + (size_t)slotA * A.stat_row;
    const float2* statsB = B.stats + (size_t)chunk * b_chunk_stats + (size_t)slotB * B.stat_row;
    const int total = A.n_slabs + B.n_slabs;

    // Sorted lists (set B, and set A unless it is unsorted), 2^parts_log2 threads to a list: thread
    // part p takes the entries p, p + P, ..., which descend.
    const int parts = 1 << parts_log2;
    const int sortedA = A.sorted ? A.n_slabs : 0, n_sorted = sortedA + B.n_slabs;
    // Unsorted lists (set A only): contiguous, taken as one array of 16-byte pieces.
    const int n_pieces = A.sorted ? 0 : A.n_slabs * (A.list_len / 2);
    // Where they do not fill the threads, the launcher has the lists (the pieces, a line at a time) dealt out to the wavefronts
    // in turn.
    auto dealt = [&](int log2_run) { return (((lane >> log2_run) * NWV + w) << log2_run) | (lane & ((1 << log2_run) - 1)); };
    const int unit_s = deal & 1 ? dealt(parts_log2) : tid, unit_p = deal & 2 ? dealt(3) : tid;
    const int part = unit_s & (parts - 1);
    const int step_sorted = NT >> parts_log2, step_pieces = NT * kPieces;

    int len = 0;
    const u64* lst = nullptr;                            // this thread's sorted list of the round, from its own part on
    u64 se[kEager];
    u32x4 up[kPieces];
    auto fetch = [&](int round) {
        const int L = round * step_sorted + (unit_s >> parts_log2);
        const bool inA = L < sortedA;
        lst = (inA ? keysA + (size_t)L * A.key_slab : keysB + (size_t)(L - sortedA) * B.key_slab) + part;
        len = L < n_sorted ? (inA ? A.list_len : B.list_len) - part : 0;       // entries are lst[0], lst[parts], ... below len
#pragma unroll
        for (int j = 0; j < kEager; ++j) se[j] = (j << parts_log2) < len ? lst[j << parts_log2] : 0ull;
        if (n_pieces) {
#pragma unroll
            for (int j = 0; j < kPieces; ++j) {
                const int q = round * step_pieces + j * NT + unit_p;
                up[j] = u32x4{~0u, ~0u, ~0u, ~0u};
                if (q < n_pieces) up[j] = *(gvec_ptr)(keysA + 2 * (size_t)q);
            }
        }
    };
    fetch(0);

    // ---- log-normaliser: online (max, scaled sum) per thread, fixed-shape reduction
    {
        float mx = -INFINITY, sm = 0.f;
        for (int t = tid; t < total; t += NT) {
            const float2 st = t < A.n_slabs ? statsA[(size_t)t * A.stat_slab] : statsB[(size_t)(t - A.n_slabs) * B.stat_slab];
            const float nm = fmaxf(mx, st.x);
            sm = (mx == -INFINITY ? 0.f : sm * __expf(mx - nm)) + st.y * __expf(st.x - nm);
            mx = nm;
        }
        // wavefront: the maximum first, then one rescale per lane and a plain sum
        const float wm_ = wave_max(mx, lane);
        sm = mx == -INFINITY ? 0.f : sm * __expf(mx - wm_);
        sm = wave_sum(sm, lane);
        if (lane == 0) { wave_m[w] = wm_; wave_s[w] = sm; }
    }

    // ---- top-k
    // The bound: the q-th largest per-thread maximum of every wavefront; with q * kSets >= k, the kSets-th
    // largest of these values is reached by k candidates.  (Half of the wavefronts: some 20 candidates
    // reach it at k = 10, whatever the number of wavefronts; with one wavefront's k-th largest alone it is
    // 30 for four wavefronts and 110 for sixteen.)
    constexpr int kSets = NWV / 2;
    const int q = (k + kSets - 1) / kSets;
    const int rounds_s = (n_sorted + step_sorted - 1) / step_sorted, rounds_p = (n_pieces + step_pieces - 1) / step_pieces;
    const int rounds = rounds_s > rounds_p ? rounds_s : rounds_p;
    int nrun = 0;
    for (int round = 0; round < rounds; ++round) {
        if (round > 0) fetch(round);
        // (1) the bound: k candidates of some wavefront reach it
        u64 best = se[0];
        if (n_pieces) {
            // any large candidate of the thread serves: plain float compares (false for empty slots: NaN)
            float bz = -INFINITY;
            uint32_t bid = ~0u;
#pragma unroll
            for (int j = 0; j < kPieces; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float z = __uint_as_float(up[j][2 * h + 1]);
                    const bool up_ = z > bz;
                    bz = up_ ? z : bz;
                    bid = up_ ? up[j][2 * h] : bid;
                }
            const u64 kb = pair_key(__float_as_uint(bz), bid);
            best = kb > best ? kb : best;
        }
        const u64 wt = wave_kth_key(best, q);
        if (lane == 0) wave_tau[w] = wt;
        if (tid == 0) npend = 0;
        __syncthreads();
        u64 tau;
        {
            const u64 mine = lane < NWV ? wave_tau[lane] : 0ull;
            int ge = 0;
#pragma unroll
            for (int i = 0; i < NWV; ++i) ge += wave_tau[i] >= mine ? 1 : 0;
            const u64 hit = __ballot(lane < NWV && mine != 0ull && ge == kSets);     // (keys are distinct: at most one lane)
            const int src = hit ? (int)__builtin_ctzll(hit) : 63;
            tau = hit ? ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(mine >> 32), src) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, src)
                      : 0ull;
            if (nrun == k && run[k - 1] > tau) tau = run[k - 1];
        }
        // (2) what reaches the bound goes to pend; use(key) sees every candidate of the thread that does
        auto each = [&](u64 t, auto use) {
            bool more = true;                            // sorted entries: stop at the first one below t
#pragma unroll
            for (int j = 0; j < kEager; ++j) {
                more = more && se[j] != 0ull && se[j] >= t;
                if (more) use(se[j]);
            }
            for (int j = kEager << parts_log2; more && j < len; j += parts) {
                const u64 key = lst[j];
                more = key != 0ull && key >= t;
                if (more) use(key);
            }
            if (n_pieces) {
                const float tz = t ? ordered_to_f32((uint32_t)(t >> 32)) : -INFINITY;
#pragma unroll
                for (int j = 0; j < kPieces; ++j)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // (a NaN logit is no smaller than anything, as in the keys)
                        if (!(__uint_as_float(up[j][2 * h + 1]) < tz) && up[j][2 * h] != ~0u) {
                            const u64 key = pair_key(up[j][2 * h + 1], up[j][2 * h]);
                            if (key >= t) use(key);
                        }
                    }
            }
            if (tid < nrun && run[tid] >= t) use(run[tid]);
        };
        auto collect = [&](u64 t) {
            // room for all of a thread's candidates with one atomic add, then stores that wait for nothing
            int n = 0;
            each(t, [&](u64) { ++n; });
            if (n == 0) return;
            int p = atomicAdd(&npend, n);
            each(t, [&](u64 key) { if (p < pend_cap) pend[p] = key; ++p; });
        };
        collect(tau);
        __syncthreads();
        if (npend > pend_cap) {
            // More candidates than the list holds (they crowd into few lists, many wavefronts over, with a
            // large k): the exact k-th largest, one bit at a time, leaves k of them.
            u64 t = tau;
            u64 found = 0;
            for (int bit = 63; bit >= 0; --bit) {
                const u64 c = found | (1ull << bit);
                __syncthreads();
                if (tid == 0) count_s = 0;
                __syncthreads();
                int mine = 0;
                each(c > t ? c : t, [&](u64 key) { mine += key >= c ? 1 : 0; });
                if (mine) atomicAdd(&count_s, mine);
                __syncthreads();
                if (count_s >= k) found = c;
            }
            tau = found > t ? found : t;
            __syncthreads();
            if (tid == 0) npend = 0;
            __syncthreads();
            collect(tau);
            __syncthreads();
        }
        // (3) exact order among pend: the rank of a key is the number of larger ones
        const int np = npend < pend_cap ? npend : pend_cap;
        const bool last = round + 1 == rounds;
        if (!last) __syncthreads();                      // (run has been read: it is rewritten below)
        for (int e = tid; e < np; e += NT) {
            const u64 mine = pend[e];
            int r = 0, j = 0;
            for (; j < np; j += 8) {                     // (the list is a whole number of eights long; past np: stale, not counted)
                ulonglong2 q[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) q[u] = *reinterpret_cast<const ulonglong2*>(pend + j + 2 * u);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    r += (q[u].x > mine && j + 2 * u < np ? 1 : 0) + (q[u].y > mine && j + 2 * u + 1 < np ? 1 : 0);
            }
            if (r < k) {
                if (last) {
                    out_vals[(size_t)out_row * k + r] = key_value(mine);
                    out_ids[(size_t)out_row * k + r] = key_id(mine);
                } else {
                    run[r] = mine;
                }
            }
        }
        nrun = np < k ? np : k;
        if (!last) __syncthreads();
    }
    // the log-normaliser over the wavefronts, by the one that has least to rank
    if (w == NWV - 1) {
        const float m_ = lane < NWV ? wave_m[lane] : -INFINITY, gm_ = wave_max(m_, lane);
        const float gs = wave_sum(m_ == -INFINITY ? 0.f : wave_s[lane] * __expf(m_ - gm_), lane);
        if (lane == 0) out_logz[out_row] = gm_ + __logf(gs);
    }
    for (int j = nrun + tid; j < k; j += NT) {           // fewer than k candidates in all
        out_vals[(size_t)out_row * k + j] = -INFINITY;
        out_ids[(size_t)out_row * k + j] = -1;
    }
}

}  // namespace evospec

// =======================================================================================
// Host launchers (argument shapes are validated by the C ABI layer before these run).
#include "launch.hpp"

namespace evospec {

namespace {
constexpr int kMaxDevices = 64;

template <int TW, int KS, int RC, int MB, bool FULLK, bool PACKED, bool ONCE, int SEGS, bool CORE>
hipError_t launch_partials_k(const Plan& p, const void* h, const ChunkBatch& cb, const CoreSet& core, const BatchLayout& bl, int d,
                             const void* W, const int32_t* ids, int V_act, int k, void* keys, void* stats,
                             hipStream_t stream) {
    auto kern = lmhead_partials_kernel<TW, KS, RC, MB, FULLK, PACKED, ONCE, SEGS, CORE>;
    static std::atomic<bool> attr_set[kMaxDevices] = {};      // concurrent first calls may both set the (idempotent) attribute
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices || !attr_set[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev].store(true, std::memory_order_release);
    }
    const dim3 grid = CORE ? dim3(core.blocks + p.n_slabs * cb.n) : dim3(p.n_slabs, bl.split ? 2 * cb.n : cb.n);
    std::conditional_t<CORE, CoreSet, int> core_or_split;
    if constexpr (CORE) core_or_split = core;
    else core_or_split = bl.split ? 1 : 0;
    hipLaunchKernelGGL(kern, grid, dim3(TW * KS * 64), p.lds_bytes, stream,
                       static_cast<const uint16_t*>(h), cb, core_or_split, bl.seq_rows, bl.chunk_bytes / 8, bl.chunk_bytes / 8, d,
                       static_cast<const uint16_t*>(W), ids,
                       V_act, k, p.gl, static_cast<u64*>(keys), static_cast<float2*>(stats));
    return hipGetLastError();
}

template <int TW, int RC, int KS4, int KS2>
hipError_t launch_partials_shape(const Plan& p, const void* h, const ChunkBatch& cb, const CoreSet& core, const BatchLayout& bl, int d,
                                 const void* W, const int32_t* ids, int V_act, int k, void* keys, void* stats,
                                 hipStream_t stream) {
    const bool full = d % kKC == 0;
    // (passes of a core beside each other share its rows through the caches)
    const bool once = core.blocks > core.n_slabs ? false
                                                 : slab_streams_once((size_t)V_act * (bl.seq_rows ? cb.n : 1) + (core.blocks > 0 ? core.V : 0), d, bl.packed);
#define EVOSPEC_ARGS p, h, cb, core, bl, d, W, ids, V_act, k, keys, stats, stream
#define EVOSPEC_FULL(MB_, KS_, SEGS_, CORE_)                                                                    \
    (bl.packed ? (once ? launch_partials_k<TW, KS_, RC, MB_, true, true, true, SEGS_, CORE_>(EVOSPEC_ARGS)      \
                       : launch_partials_k<TW, KS_, RC, MB_, true, true, false, SEGS_, CORE_>(EVOSPEC_ARGS))    \
               : (once ? launch_partials_k<TW, KS_, RC, MB_, true, false, true, SEGS_, CORE_>(EVOSPEC_ARGS)     \
                       : launch_partials_k<TW, KS_, RC, MB_, true, false, false, SEGS_, CORE_>(EVOSPEC_ARGS)))
#define EVOSPEC_MB(MB_, KS_, CORE_)                                                                             \
    if (p.mb == MB_ && p.ks == KS_ && CORE_ == (core.blocks > 0)) {                                             \
        if (!full)                                                                                              \
            return bl.packed ? launch_partials_k<TW, KS_, RC, MB_, false, true, false, 1, CORE_>(EVOSPEC_ARGS)  \
                             : launch_partials_k<TW, KS_, RC, MB_, false, false, false, 1, CORE_>(EVOSPEC_ARGS); \
        if constexpr (KS_ <= kSegMaxShare && !CORE_) {                                                          \
            if (p.segs == 2) return EVOSPEC_FULL(MB_, KS_, 2, CORE_);                                           \
        }                                                                                                       \
        return EVOSPEC_FULL(MB_, KS_, 1, CORE_);                                                                \
    }
    EVOSPEC_MB(1, 1, false) EVOSPEC_MB(2, 1, false) EVOSPEC_MB(4, 1, false)
    EVOSPEC_MB(1, 1, true) EVOSPEC_MB(2, 1, true) EVOSPEC_MB(4, 1, true)
    if constexpr (KS2 > 1) { EVOSPEC_MB(2, KS2, false) }
    if constexpr (KS4 > 1) { EVOSPEC_MB(4, KS4, false) }
#undef EVOSPEC_MB
#undef EVOSPEC_FULL
#undef EVOSPEC_ARGS
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_partials_batch(const Plan& p, const void* h, const ChunkBatch& cb, const CoreSet& core, const BatchLayout& bl,
                                 int d, const void* W, const int32_t* ids, int V_act, int k, void* keys,
                                 void* stats, hipStream_t stream) {
    if (cb.n < 1 || cb.n > kMaxChunks || bl.chunk_bytes % 8 != 0) return hipErrorInvalidValue;
    if (core.blocks > 0 && (p.ks != 1 || p.segs != 1 || bl.split || core.n_slabs < 1 || core.chunk_slabs != p.n_slabs ||
                            core.blocks % core.n_slabs != 0 || (long)core.n_slabs * p.rt < core.V ||
                            core.blocks / core.n_slabs != (core.M + kMTile - 1) / kMTile))
        return hipErrorInvalidValue;
    if (bl.split && (p.mb != mb_for_rows(kSplitRows) || p.ks != 1)) return hipErrorInvalidValue;      // (the kernels that know it)
    switch (p.nw) {
#define EVOSPEC_SHAPE(TW_, RC_, KS4_, KS2_)                                                     \
    case TW_: return launch_partials_shape<TW_, RC_, KS4_, KS2_>(p, h, cb, core, bl, d, W, ids, V_act, k, keys, stats, stream);
        EVOSPEC_SLAB_SHAPES(EVOSPEC_SHAPE)
#undef EVOSPEC_SHAPE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_partials(const Plan& p, const void* h, int rows, int d, const void* W,
                           const int32_t* ids, int V_act, int k, void* keys, void* stats,
                           hipStream_t stream, bool packed) {
    ChunkBatch cb;
    cb.n = 1; cb.m0[0] = 0; cb.rows[0] = rows; cb.seq[0] = 0; cb.a_pass[0] = 0; cb.a_slot[0] = 0;
    BatchLayout bl;
    bl.packed = packed;
    return launch_partials_batch(p, h, cb, CoreSet{}, bl, d, W, ids, V_act, k, keys, stats, stream);
}

hipError_t launch_merge_batch(const MergeSet& a, size_t a_pass_bytes, const MergeSet& b, size_t b_chunk_bytes,
                              const ChunkBatch& cb, int k, float* out_vals, int32_t* out_ids,
                              float* out_logz, hipStream_t stream, const GatherArgs* update) {
    if (cb.n < 1 || cb.n > kMaxChunks || a_pass_bytes % 8 != 0 || b_chunk_bytes % 8 != 0) return hipErrorInvalidValue;
    int max_rows = 0;
    for (int i = 0; i < cb.n; ++i) max_rows = cb.rows[i] > max_rows ? cb.rows[i] : max_rows;
    GatherArgs upd{};
    if (update && update->n > 0) upd = *update;
    if (max_rows == 0 && upd.n == 0) return hipSuccess;
    if ((a.list_len != 0 && (a.list_len < k || a.list_len > kKMax || (a.list_len & 15))) ||
        (b.list_len != 0 && (b.list_len < k || b.list_len > kKMax || (b.list_len & 15))))
        return hipErrorInvalidValue;
    if (b.list_len != 0 || (a.list_len != 0 && !a.row_major)) return hipErrorInvalidValue;   // unsorted: one contiguous set
    auto as_set = [&](const MergeSet& m) {
        PartialSet p;
        p.keys = static_cast<const u64*>(m.keys);
        p.stats = static_cast<const float2*>(m.stats);
        p.n_slabs = m.n_slabs;
        p.row_base = m.row_base;
        p.list_len = m.list_len ? m.list_len : k;
        p.sorted = m.list_len == 0;
        if (m.row_major) {          // [row][slab][slot]: one row's lists are contiguous
            p.key_slab = (size_t)p.list_len; p.key_row = (size_t)m.n_slabs * p.list_len;
            p.stat_slab = 1; p.stat_row = (size_t)m.n_slabs;
        } else {                    // [slab][row][slot]
            p.key_slab = (size_t)m.row_stride * p.list_len; p.key_row = (size_t)p.list_len;
            p.stat_slab = (size_t)m.row_stride; p.stat_row = 1;
        }
        return p;
    };
    const PartialSet A = as_set(a), B = as_set(b);
    const int gx = max_rows > upd.n ? max_rows : upd.n;
    // Enough threads to take all lists of a row in one round where possible: a thread takes one sorted
    // list, or 16 slots of the unsorted ones.  Fewer sorted lists than threads: several threads share one.
    const int n_sorted = (A.sorted ? A.n_slabs : 0) + B.n_slabs;
    const int n_pieces = A.sorted ? 0 : A.n_slabs * (A.list_len / 2);
    const int units = n_sorted > n_pieces / 8 ? n_sorted : (n_pieces + 7) / 8;
    const int nt = units <= 256 ? 256 : (units <= 512 ? 512 : 1024);
    const int max_len = A.list_len > B.list_len ? A.list_len : B.list_len;
    int parts_log2 = 0;
    while (n_sorted > 0 && parts_log2 < 4 && (n_sorted << (parts_log2 + 1)) <= nt && (2 << parts_log2) <= max_len) ++parts_log2;
    // The kernel's bound is the sets-th largest of the wavefronts' q-th largest candidates (see there).  Lists or pieces
    // that do not fill the threads are dealt out to the wavefronts in turn where each then gets 2 q of them, and where
    // otherwise not even `sets` wavefronts have q, so that everything would be a candidate (16 lists of 5 9.0 us, 64 of 1
    // 8.6; dealt out 5.2 and 5.1; 132 lists of 64, where each wavefront gets q of 33: 43 dealt out, 10 not).
    const int sets = nt / 128, q = (k + sets - 1) / sets;
    auto deals = [&](int units) { return units < nt && (units >= 2 * q * (nt / 64) || units < 64 * (sets - 1) + q); };
    const int deal = (deals(n_sorted << parts_log2) ? 1 : 0) | (deals(n_pieces) ? 2 : 0);
    // room for what usually reaches the bound, up to 32 KB (more is handled, slowly), and the running k
    int pend_cap = nt / 64 * k * (max_len > 16 ? max_len : 16);
    pend_cap = ((pend_cap < 4096 ? pend_cap : 4096) + k + 7) & ~7;
    const dim3 grid(gx, cb.n + (upd.n > 0 ? 1 : 0));
#define EVOSPEC_MERGE(NT_)                                                                                  \
    hipLaunchKernelGGL(lmhead_merge_kernel<NT_>, grid, dim3(NT_), (size_t)pend_cap * 8, stream, A, B, cb,    \
                       a_pass_bytes / 8, a_pass_bytes / 8, b_chunk_bytes / 8, b_chunk_bytes / 8, k, parts_log2, \
                       deal, pend_cap, out_vals, out_ids, out_logz, upd)
    if (nt == 256) EVOSPEC_MERGE(256);
    else if (nt == 512) EVOSPEC_MERGE(512);
    else EVOSPEC_MERGE(1024);
#undef EVOSPEC_MERGE
    return hipGetLastError();
}

hipError_t launch_merge(const MergeSet& a, const MergeSet& b, int k, float* out_vals, int32_t* out_ids,
                        float* out_logz, int out_row0, int nrows, hipStream_t stream, const GatherArgs* update) {
    ChunkBatch cb;
    cb.n = 1; cb.m0[0] = out_row0; cb.rows[0] = nrows; cb.seq[0] = 0; cb.a_pass[0] = 0; cb.a_slot[0] = 0;
    return launch_merge_batch(a, 0, b, 0, cb, k, out_vals, out_ids, out_logz, stream, update);
}

hipError_t launch_gather(const void* W_lm, int V, int d, const int32_t* src_ids, const int32_t* slots,
                         int n, void* W_act, int32_t* act_ids, int V_act, hipStream_t stream, bool packed) {
    const GatherArgs g = gather_args(W_lm, V, d, src_ids, slots, n, W_act, act_ids, V_act, packed);
    if (packed && !slots) {                      // rebuild: whole operand tiles per workgroup
        const int tiles = (n + kPackRows - 1) / kPackRows;
        hipLaunchKernelGGL(gather_tiles_kernel, dim3(tiles < 4096 ? tiles : 4096), dim3(256), 0, stream, g);
        return hipGetLastError();
    }
    if (!packed && !slots && n >= 1024) {        // rebuild of a row-major matrix
        hipLaunchKernelGGL(gather_rebuild_rows_kernel, dim3(4096), dim3(256), 0, stream, g);
        return hipGetLastError();
    }
    const int grid = n < 8192 ? n : 8192;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(grid), dim3(256), 0, stream, g);
    return hipGetLastError();
}

hipError_t launch_gather_inline(const void* W_lm, int V, int d, const int32_t* host_ids, const int32_t* host_slots,
                                int n, void* W_act, int32_t* act_ids, int V_act, hipStream_t stream, bool packed) {
    if (n < 0 || n > kInlineRows) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    const GatherArgs g = gather_args(W_lm, V, d, nullptr, nullptr, n, W_act, act_ids, V_act, packed);
    InlineRows r{};
    for (int i = 0; i < n; ++i) { r.slot[i] = host_slots[i]; r.id[i] = host_ids[i]; }
    hipLaunchKernelGGL(gather_rows_inline_kernel, dim3(n), dim3(256), 0, stream, g, r);
    return hipGetLastError();
}

hipError_t run_validate_ids(const int32_t* ids, int n, int V, hipStream_t stream, int* bad) {
    // one flag per device: calls from several threads take turns (the call waits for its kernel anyway)
    static std::mutex flag_mutex;
    std::lock_guard<std::mutex> lock(flag_mutex);
    int* flag = nullptr;
    hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&flag), HIP_SYMBOL(g_validate_flag));
    if (e != hipSuccess) return e;
    int zero = 0;
    e = hipMemcpyAsync(flag, &zero, sizeof(int), hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(validate_ids_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, ids, n, V, flag);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(bad, flag, sizeof(int), hipMemcpyDeviceToHost, stream);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(stream);
}

}  // namespace evospec

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
// Pass 1 of the restricted head: one workgroup streams one slab of RT = 16*TW rows of
// W_act (KS wavefronts to a tile of 16 rows, its elements loaded from HBM straight into MFMA operand layout
// with 128-bit loads), contracts it with up to 16*MB draft rows of h (K-chunks of h staged
// in LDS, double buffered, shared by all waves), and reduces the slab's logits, which stay in
// the accumulators, to
//   part_stats[slab][m] = (max_i z, sum_i exp(z - max))         over the slab's rows
//   part_keys[slab][m][0..k) = the slab's k best keys, descending (0 = none)
// Logits never leave the CU.
// ONCE (see slab_streams_once): the weights bypass the caches, 60.0 -> 54.3 us at 36,864 x 4,096 and 60 rows.  On a
// row-major matrix a load otherwise takes half lines of 16 rows, the other half of which must be found in the caches again; past
// them it takes whole lines of 8 rows, permuted into operands within 16 lanes: full vocabulary 253 -> 244 us.  (Whole lines
// through the caches gain nothing: 254.5, 32,256 x 2,048 37.0 -> 37.3, 24 rows, 36,864 x 4,096 62.1 -> 64.1.)
template <int TW, int KS, int RC, int MB, bool FULLK, bool PACKED, bool ONCE, int SEGS>
__global__ void __launch_bounds__(TW * KS * 64)
lmhead_partials_kernel(const uint16_t* __restrict__ h_all, ChunkBatch cb, int split, int seq_rows,
                       size_t chunk_keys, size_t chunk_stats, int d,
                       const uint16_t* __restrict__ W_all, const int32_t* __restrict__ ids_all,
                       int V_act, int k, int GL,
                       u64* __restrict__ keys_all, float2* __restrict__ stats_all) {
    // this workgroup's problem: chunk blockIdx.y of the batch (its draft rows, its sequence's
    // rows of a per-sequence matrix, its own piece of the partials)
    // (split = 1: its draft rows go to two workgroups, the first kSplitRows and the others)
    constexpr bool kMaySplit = MB == mb_for_rows(kSplitRows) && KS == 1;
    const int ci = kMaySplit ? blockIdx.y >> split : blockIdx.y, row_first = kMaySplit ? (blockIdx.y & split) * kSplitRows : 0;
    int rows = cb.rows[ci];
    if constexpr (kMaySplit) {
        if (split) rows = min(rows - row_first, kSplitRows);
        if (rows <= 0) return;                                                // (uniform)
    }
    const size_t seq_row0 = (size_t)cb.seq[ci] * seq_rows;
    const uint16_t* __restrict__ h = h_all + (size_t)(cb.m0[ci] + row_first) * d;
    // (a packed matrix pads every sequence's rows to whole tiles and its rows to whole chunks)
    const int dp = packed_d(d);
    const uint16_t* __restrict__ W = PACKED ? W_all + (size_t)cb.seq[ci] * packed_rows(seq_rows) * dp
                                            : W_all + seq_row0 * d;
    const int32_t* __restrict__ ids = ids_all ? ids_all + seq_row0 : nullptr;
    u64* __restrict__ part_keys = keys_all + (size_t)ci * chunk_keys + row_first * k;
    float2* __restrict__ part_stats = stats_all + (size_t)ci * chunk_stats + row_first;
    constexpr int NW = TW * KS;                    // wavefronts: KS of them share a tile, each a part of every chunk's k-steps
    constexpr int NT = NW * 64;
    constexpr int RT = 16 * TW;
    static_assert(MB % KS == 0, "after the stream each wavefront of a tile keeps MB / KS blocks of draft rows");
    constexpr int MBW = MB / KS;
    constexpr int MR = 16 * MB;
    constexpr int KC = kKC;
    constexpr int KSTEPS = KC / 32 / KS;           // k-steps of a chunk that a wavefront takes
    static_assert(KSTEPS % 2 == 0, "the B operands of two k-steps alternate");
    constexpr int HPIECES = MR * (KC / 8);
    constexpr int HP = (HPIECES + NT - 1) / NT;

    extern __shared__ __align__(16) unsigned char smem[];
    // region U: h chunks during the contraction, the survivors' keys afterwards
    uint16_t* Hs = reinterpret_cast<uint16_t*>(smem);
    u64* list = reinterpret_cast<u64*>(smem);                                 // [MR][LS]
    constexpr int LS = list_stride(RT);
    constexpr size_t hs_bytes = 2ull * MR * kHStride * 2;
    constexpr size_t list_bytes = (size_t)MR * list_stride(RT) * 8;
    // (with two segments, the sums of the other one behind the h chunks: [NW][MB][64] f32x4)
    constexpr size_t h_lev_bytes = hs_bytes + slab_level_bytes(NW, MB, SEGS);
    constexpr size_t u_bytes = align_up(h_lev_bytes > list_bytes ? h_lev_bytes : list_bytes, 16);
    const bool fine = fine_groups(k, TW);                                     // (then GL is 0)
    const int NGS = fine ? 8 * TW : 4 * TW;                                   // row stride of gm
    float* gm = reinterpret_cast<float*>(smem + u_bytes);                     // [MR][NGS] group maxima
    float* wsum = gm + (size_t)MR * NGS;                                      // [TW][MR] sum-exp of each tile
    int32_t* Ids = reinterpret_cast<int32_t*>(wsum + (size_t)TW * MR);        // [RT]
    float* tau = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(Ids) + align_up((size_t)RT * 4, 16));  // [MR]
    float* vmax = tau + MR;                                                   // [MR]
    int* cnt = reinterpret_cast<int*>(vmax + MR);                             // [MR]

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = (tid >> 6) / KS, kq = KS > 1 ? (tid >> 6) % KS : 0;          // this wavefront's tile, and its part of the k-steps
    const int s0 = kq * KSTEPS;                                               // first of its k-steps in a chunk of h in LDS
    const int n16 = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.x * RT;
    const int n_valid = min(RT, V_act - row0);

    // full-vocabulary id of slab row `tid` (RT <= NT): loaded first, parked in LDS once the operand
    // loads of the first chunks have been issued
    static_assert(RT <= NT, "one slab row per thread");
    int id_reg = 0x7fffffff;
    if (tid < RT && row0 + tid < V_act) id_reg = ids ? ids[row0 + tid] : row0 + tid;

    // Row-major rows past the caches: a load must take whole 128-byte lines (the other half of a line would be fetched
    // again).  The first load of two k-steps takes the line of rows 0..7, the second that of rows 8..15, and permutes within
    // 16 lanes make the operands (see pick_bank).
    constexpr bool LINES = !PACKED && ONCE;
    static_assert(!LINES || FULLK, "whole lines");
    const uint16_t *wp, *wp8 = nullptr;
    if constexpr (PACKED) {
        // the wavefront's tile: 1 KB operand blocks in k-step order, lane l at byte 16 l
        const int tile = min((row0 >> 4) + w, (V_act - 1) >> 4);   // tail slab: a valid tile, masked later
        wp = W + (size_t)tile * kPackRows * dp + lane * 8;
    } else if constexpr (LINES) {
        const int row = row0 + w * 16 + (n16 & 7), c = 8 * g, c_hi = n16 & 8 ? 32 : 0;     // (row past the end: see below)
        wp = W + (size_t)min(row, V_act - 1) * d + c + c_hi;
        wp8 = W + (size_t)min(row + 8, V_act - 1) * d + c + (32 - c_hi);
    } else {
        wp = W + (size_t)min(row0 + w * 16 + n16, V_act - 1) * d + g * 8;   // tail slab: duplicate a valid row, masked later
    }

    f32x4 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Every workgroup adds up a logit in the same order: equal rows of different slabs must tie exactly.  With two segments
    // (segments_for) the chunks of either (c / 4 even, odd) are summed front to back by themselves and the two sums are added
    // at the end.  A workgroup with cx = 4 takes the chunks c ^ 4, each four of the other segment first: both sums
    // and the last addition are the same to the bit, but it is 2 KB away from the others in its rows.
    const int nchunks = (d + KC - 1) / KC;
    // (Every other workgroup; every other pair where slabs are a power of two high, whose places in memory alternate by themselves:
    // 32,256 x 2,048 in slabs of 128 rows 38.3 to 40.9 us by where the matrix lies, by pairs 38.1; 24,000 x 2,048 in slabs of 96
    // 31.5, by pairs 32.9.)
    constexpr int kTurnBit = (TW & (TW - 1)) == 0 ? 1 : 0;
    const int cx = !PACKED && SEGS == 2 ? ((int)(blockIdx.x >> kTurnBit) & 1) * kSegChunks : 0;
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    // chunks that h is requested ahead of its use (13 to 16 wavefronts have 128 registers each, which three pieces
    // per thread twice over exceed)
    constexpr int HA = KS > 1 && (NT <= 768 || HP <= 2) ? 2 : 1;
    static_assert(RC % HA == 0, "the register set of a chunk's h is known at compile time");
    u32x4 hreg[HA][HP];
    u32x4 wr[RC * KSTEPS];                // ring of W operands: this wavefront's k-steps of RC consecutive chunks

    // this thread's pieces (16 B each) of an h chunk: global source, LDS destination
    gvec_ptr hsrc[HP];
    int hdst[HP], hcol[HP];
#pragma unroll
    for (int p = 0; p < HP; ++p) {
        // threads beyond the last piece wrap around and re-stage an earlier piece (same bytes to
        // the same place), which keeps every load and LDS store unconditional
        const int idc = (tid + p * NT) % HPIECES;
        const int m = idc / (KC / 8), c8 = idc % (KC / 8);
        hcol[p] = c8 * 8;
        hsrc[p] = (gvec_ptr)(h + (size_t)min(m, rows - 1) * d + c8 * 8);
        hdst[p] = m * kHStride + c8 * 8;
    }

    // Loads past the end of a row (only in the last chunk when d is not a multiple of KC: `whole` says that
    // this one is not it) are redirected to the row's last 16 bytes and replaced by zeros, so that no load is
    // conditional.
    auto load_h = [&](u32x4 (&hr)[HP], int c, auto whole) {
#pragma unroll
        for (int p = 0; p < HP; ++p) {
            if constexpr (decltype(whole)::value) {
                hr[p] = hsrc[p][c * (KC / 8)];
            } else {
                const int kk = c * KC + hcol[p];
                const bool in = kk < d;
                const u32x4 v = *(hsrc[p] + ((in ? kk : d - 8) - hcol[p]) / 8);
                hr[p] = in ? v : zero4;
            }
        }
    };
    auto store_h = [&](const u32x4 (&hr)[HP], int buf) {
#pragma unroll
        for (int p = 0; p < HP; ++p)
            *reinterpret_cast<u32x4*>(Hs + (size_t)buf * MR * kHStride + hdst[p]) = hr[p];
    };
    // k-step s (0..KSTEPS-1 of this wavefront) of chunk c goes to ring slot (c % RC) * KSTEPS + s
    auto load_w = [&](gvec_ptr p) { return ONCE ? load_once(p) : *p; };
    auto load_w_step = [&](int slot, int c, int s, auto whole) {
        const int koff = c * KC + (s0 + s) * 32;
        if constexpr (PACKED) {
            wr[slot] = load_w((gvec_ptr)wp + (koff / 32) * 64);          // rows are padded to whole chunks
        } else if constexpr (LINES) {
            wr[slot] = load_w((gvec_ptr)((s & 1 ? wp8 - 32 : wp) + koff));
        } else {
            if constexpr (decltype(whole)::value) {
                wr[slot] = load_w((gvec_ptr)(wp + koff));
            } else {
                const bool in = koff + g * 8 < d;
                const u32x4 v = *(gvec_ptr)(wp + (in ? koff : d - 8 - g * 8));
                wr[slot] = in ? v : zero4;
            }
        }
    };
    auto load_b = [&](bf16x8 (&b)[MB], int buf, int s) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            b[mb] = *reinterpret_cast<const bf16x8*>(Hs + ((size_t)buf * MR + mb * 16 + n16) * kHStride + (s0 + s) * 32 + g * 8);
    };
    auto mfma_step = [&](int slot, const bf16x8 (&b)[MB]) {
        u32x4 x = wr[slot];
        if constexpr (LINES) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[i] = slot & 1 ? pick_bank_ror8(wr[slot & ~1][i], wr[slot | 1][i]) : pick_bank(wr[slot & ~1][i], wr[slot | 1][i]);
        }
        const bf16x8 a = __builtin_bit_cast(bf16x8, x);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[mb], acc[mb], 0, 0, 0);
    };
    // One chunk (KSTEPS k-steps of this wavefront).  Ring part SLOT (= c % RC) holds this chunk's W operands, loaded RC
    // chunks ago; each slot is refilled with the same k-step of chunk c+RC right after the MFMAs
    // that consumed it were issued (packed matrix) or all slots at the end of the chunk (row-major
    // matrix), so up to RC*KSTEPS 16-byte loads per lane stay in flight.
    // The h chunk c+HA is requested meanwhile, and chunk c+1 goes from registers to the other LDS buffer
    // at the end.  (One chunk ahead is enough while a chunk takes longer than a trip to L2, about 1 us.)  In the steady state (chunks c+1 and c+RC exist) there is no branch in here;
    // the last chunks test for them at run time.
    auto chunk = [&](auto slot_c, int c, auto steady) {
        constexpr int SLOT = decltype(slot_c)::value;
        constexpr bool STEADY = decltype(steady)::value;
        const bool pw = STEADY || (c + RC < nchunks);
        const bool ph = STEADY || (c + 1 < nchunks);
        const int buf = c & 1, cw = (c + RC) ^ cx;
        constexpr std::bool_constant<FULLK || STEADY> whole{};
        bf16x8 b0[MB], b1[MB];
        if (STEADY || c + HA < nchunks) load_h(hreg[(SLOT + HA) % HA], (c + HA) ^ cx, whole);
        load_b(b0, buf, 0);
#pragma unroll
        for (int s = 0; s < KSTEPS; s += 2) {
            load_b(b1, buf, s + 1);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step(SLOT * KSTEPS + s, b0);
            if (PACKED && pw) load_w_step(SLOT * KSTEPS + s, cw, s, whole);
            if (s + 2 < KSTEPS) load_b(b0, buf, s + 2);
            __builtin_amdgcn_sched_barrier(0);
            mfma_step(SLOT * KSTEPS + s + 1, b1);
            if (PACKED && pw) load_w_step(SLOT * KSTEPS + s + 1, cw, s + 1, whole);
        }
        if (!PACKED && pw) {
            // row-major rows: the chunk's 8 requests go out together, so that the 512 bytes they
            // take from each row reach the memory side close in time (measured: 3.5 us of 73)
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) load_w_step(SLOT * KSTEPS + s, cw, s, whole);
        }
        if (ph) store_h(hreg[(SLOT + 1) % HA], buf ^ 1);
        lds_barrier();
    };
    // RC consecutive chunks starting at `base` (a multiple of RC), ring parts 0..RC-1
    auto chunk_group = [&](int base, auto steady) {
        constexpr bool STEADY = decltype(steady)::value;
#define EVOSPEC_CHUNK(I)                                                                   \
        if constexpr (I < RC) {                                                            \
            if (STEADY || base + I < nchunks) chunk(std::integral_constant<int, I>{}, base + I, steady); \
        }
        EVOSPEC_CHUNK(0) EVOSPEC_CHUNK(1) EVOSPEC_CHUNK(2) EVOSPEC_CHUNK(3)
#undef EVOSPEC_CHUNK
    };
    static_assert(RC >= 1 && RC <= 4, "ring depth");

    constexpr std::bool_constant<FULLK> first{};
    load_h(hreg[0], 0 ^ cx, first);
#pragma unroll
    for (int i = 0; i < RC; ++i) {
        if (i < nchunks) {
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) load_w_step(i * KSTEPS + s, i ^ cx, s, first);
        }
    }
    for (int i = tid; i < MR * NGS; i += NT) gm[i] = -INFINITY;      // padding of the group-maximum rows
    if (tid < RT) Ids[tid] = id_reg;
    store_h(hreg[0], 0);
    if constexpr (HA > 1) {
        if (nchunks > 1) load_h(hreg[1], 1 ^ cx, first);
    }
    lds_barrier();
    int c = 0;
    const int nwhole = d / KC;
    // between two segments: the sum so far waits behind the h chunks, the other segment's goes on
    f32x4* lev = reinterpret_cast<f32x4*>(smem + hs_bytes) + (size_t)(tid >> 6) * MB * 64 + lane;
    auto turn = [&](int done) {
        if (SEGS == 1 || (done & (kSegChunks - 1)) != 0 || done >= nchunks) return;      // (uniform)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const f32x4 other = done == kSegChunks ? f32x4{0.f, 0.f, 0.f, 0.f} : lev[mb * 64];
            lev[mb * 64] = acc[mb];
            acc[mb] = other;
        }
    };
    static_assert(kSegChunks % RC == 0, "segments end with a turn of the ring");
    for (; c + 2 * RC <= nwhole; c += RC) {                                      // every prefetch target exists, and whole
        chunk_group(c, std::true_type{});
        turn(c + RC);
    }
    for (; c < nchunks; c += RC) {
        chunk_group(c, std::false_type{});
        turn(c + RC);
    }
    if constexpr (SEGS == 2) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] += lev[mb * 64];
    }
    // every wave is past its last read of Hs (the loop ends on a barrier): region U is free

    // ---- the wavefronts of a tile add up: wavefront kq keeps the blocks kq * MBW .. + MBW of draft rows, the
    // parts are added in the order of kq
    if constexpr (KS > 1) {
        f32x4* red = reinterpret_cast<f32x4*>(smem);               // [TW][KS][MB][64] (fits region U)
        static_assert((size_t)TW * KS * MB * 1024 <= hs_bytes, "partial sums fit the h chunks");
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) red[((size_t)(w * KS + kq) * MB + mb) * 64 + lane] = acc[mb];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            f32x4 x = red[((size_t)(w * KS) * MB + kq * MBW + i) * 64 + lane];
#pragma unroll
            for (int q = 1; q < KS; ++q) x += red[((size_t)(w * KS + q) * MB + kq * MBW + i) * 64 + lane];
            acc[i] = x;
        }
    }

    // ---- slab epilogue.  The slab's logits stay in the accumulators: lane (n16, g) holds, for each of its
    // blocks mb of 16 draft rows, 4 logits of draft row mb*16+n16 (rows 4g..4g+3 of the tile).
    const int mb0 = kq * MBW;                                      // this wavefront's first block
    if (n_valid < RT) {                                  // tail slab: rows past V_act never win
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (w * 16 + 4 * g + j >= n_valid) {
#pragma unroll
                for (int i = 0; i < MBW; ++i) acc[i][j] = -INFINITY;
            }
    }
    // (1) group maxima (level GL: lane, lane pair or wave; fine: pairs of a lane's logits)
    const int NG = fine ? 8 * TW : TW << (2 - GL);
    {
        const int gidx = GL == 0 ? w * 4 + g : (GL == 1 ? w * 2 + (g >> 1) : w);
        const bool owner = GL == 0 ? true : (GL == 1 ? (g & 1) == 0 : g == 0);
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            const float l0 = fmaxf(acc[i][0], acc[i][1]), l1 = fmaxf(acc[i][2], acc[i][3]);
            float* gr = gm + ((mb0 + i) * 16 + n16) * NGS;
            if (fine) {                                            // (uniform)
                gr[2 * gidx] = l0;
                gr[2 * gidx + 1] = l1;
                continue;
            }
            float lm = fmaxf(l0, l1);
            if (GL >= 1) lm = fmaxf(lm, __uint_as_float(xor_lane<16>(__float_as_uint(lm), lane)));
            if (GL >= 2) lm = fmaxf(lm, __uint_as_float(xor_lane<32>(__float_as_uint(lm), lane)));
            if (owner) gr[gidx] = lm;
        }
    }
    if (tid < MR) { cnt[tid] = 0; tau[tid] = -INFINITY; }
    __syncthreads();
    // (2) tau[m] = k-th largest group maximum (counting equal values): the group maxima are NG
    //     distinct slab entries, so at least k entries are >= tau and nothing below tau can be among
    //     the slab's k best.  (NG < k: tau stays -inf and everything is ranked.)  vmax[m] = slab
    //     maximum.  Rows of gm are padded with -inf to a multiple of 4 and read 16 bytes at a time.
    {
        const int ng4 = (NG + 3) >> 2;
        for (int p = tid; p < rows * NG; p += NT) {
            const int m = p / NG, j = p - m * NG;
            const float4* gr4 = reinterpret_cast<const float4*>(gm + m * NGS);
            const float mine = gm[m * NGS + j];
            int gt = 0, ge = 0;
            float top = -INFINITY;
            for (int i4 = 0; i4 < ng4; ++i4) {
                const float4 o = gr4[i4];
                gt += (o.x > mine) + (o.y > mine) + (o.z > mine) + (o.w > mine);
                ge += (o.x >= mine) + (o.y >= mine) + (o.z >= mine) + (o.w >= mine);
                top = fmaxf(fmaxf(top, fmaxf(o.x, o.y)), fmaxf(o.z, o.w));
            }
            if (gt < k && ge >= k) tau[m] = mine;            // equal maxima write the same value
            if (j == 0) vmax[m] = top;
        }
    }
    __syncthreads();
    // (3) sum of exponentials; entries >= tau become candidates (key = logit and full-vocabulary id).
    //     One LDS atomic per lane and draft-row block reserves room for the lane's candidates, which
    //     are then stored without branches or dependent loads.
    {
        const int4 id4 = *reinterpret_cast<const int4*>(Ids + w * 16 + 4 * g);
        const int idv[4] = {id4.x, id4.y, id4.z, id4.w};
        uint32_t pick[MBW];
        int base[MBW];
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            const int m = (mb0 + i) * 16 + n16;
            pick[i] = 0;
            if ((mb0 + i) * 16 < rows) {                     // uniform: skip blocks of padding draft rows
                const bool live = m < rows;
                const float t = live ? tau[m] : INFINITY;
                const float vm = live ? vmax[m] : 0.f;
                float se = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = acc[i][j];
                    const int rl = w * 16 + 4 * g + j;
                    se += __expf(x - vm);
                    pick[i] |= (x >= t && rl < n_valid) ? 1u << j : 0u;
                }
                se += __uint_as_float(xor_lane<16>(__float_as_uint(se), lane));
                se += __uint_as_float(xor_lane<32>(__float_as_uint(se), lane));
                if (g == 0) wsum[w * MR + m] = se;
            }
        }
#pragma unroll
        for (int i = 0; i < MBW; ++i)
            base[i] = pick[i] ? atomicAdd(&cnt[(mb0 + i) * 16 + n16], __popc(pick[i])) : 0;
#pragma unroll
        for (int i = 0; i < MBW; ++i) {
            u64* dst = list + (size_t)((mb0 + i) * 16 + n16) * LS + base[i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u64 key = make_key(acc[i][j], idv[j]);
                if (pick[i] >> j & 1u) dst[__popc(pick[i] & ((1u << j) - 1u))] = key;
            }
        }
    }
    __syncthreads();
    // (4) exact order among the candidates of a draft row (NW threads per row); the k best go out.
    //     Keys are distinct because ids are, so a key's rank is the number of larger keys.
    if (tid < rows * NW) {
        const int m = tid / NW, sub = tid - m * NW;
        const int c = cnt[m];
        const u64* lst = list + (size_t)m * LS;
        u64* outk = part_keys + ((size_t)blockIdx.x * kMTile + m) * k;
        for (int q = sub; q < c; q += 2 * NW) {              // two candidates per pass share the reads of the list
            const bool two = q + NW < c;
            const u64 mine0 = lst[q], mine1 = two ? lst[q + NW] : ~0ull;
            int rank0 = 0, rank1 = 0;
            int j = 0;
            for (; j + 4 <= c; j += 4) {
                const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(lst + j);
                const ulonglong2 b2 = *reinterpret_cast<const ulonglong2*>(lst + j + 2);
                rank0 += (a.x > mine0) + (a.y > mine0) + (b2.x > mine0) + (b2.y > mine0);
                rank1 += (a.x > mine1) + (a.y > mine1) + (b2.x > mine1) + (b2.y > mine1);
            }
            for (; j < c; ++j) { const u64 o = lst[j]; rank0 += o > mine0; rank1 += o > mine1; }
            if (rank0 < k) outk[rank0] = mine0;
            if (two && rank1 < k) outk[rank1] = mine1;
        }
        if (sub == 0) {
            for (int j = c; j < k; ++j) outk[j] = 0;               // slab holds fewer than k rows
            float sum = 0.f;
#pragma unroll
            for (int ww = 0; ww < TW; ++ww) sum += wsum[ww * MR + m];
            part_stats[(size_t)blockIdx.x * kMTile + m] = make_float2(vmax[m], sum);
        }
    }
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

template <int TW, int KS, int RC, int MB, bool FULLK, bool PACKED, bool ONCE, int SEGS>
hipError_t launch_partials_k(const Plan& p, const void* h, const ChunkBatch& cb, const BatchLayout& bl, int d,
                             const void* W, const int32_t* ids, int V_act, int k, void* keys, void* stats,
                             hipStream_t stream) {
    auto kern = lmhead_partials_kernel<TW, KS, RC, MB, FULLK, PACKED, ONCE, SEGS>;
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
    hipLaunchKernelGGL(kern, dim3(p.n_slabs, bl.split ? 2 * cb.n : cb.n), dim3(TW * KS * 64), p.lds_bytes, stream,
                       static_cast<const uint16_t*>(h), cb, bl.split ? 1 : 0, bl.seq_rows, bl.chunk_bytes / 8, bl.chunk_bytes / 8, d,
                       static_cast<const uint16_t*>(W), ids,
                       V_act, k, p.gl, static_cast<u64*>(keys), static_cast<float2*>(stats));
    return hipGetLastError();
}

template <int TW, int RC, int KS4, int KS2>
hipError_t launch_partials_shape(const Plan& p, const void* h, const ChunkBatch& cb, const BatchLayout& bl, int d,
                                 const void* W, const int32_t* ids, int V_act, int k, void* keys, void* stats,
                                 hipStream_t stream) {
    const bool full = d % kKC == 0;
    const bool once = slab_streams_once((size_t)V_act * (bl.seq_rows ? cb.n : 1), d, bl.packed);
#define EVOSPEC_ARGS p, h, cb, bl, d, W, ids, V_act, k, keys, stats, stream
#define EVOSPEC_FULL(MB_, KS_, SEGS_)                                                                           \
    (bl.packed ? (once ? launch_partials_k<TW, KS_, RC, MB_, true, true, true, SEGS_>(EVOSPEC_ARGS)             \
                       : launch_partials_k<TW, KS_, RC, MB_, true, true, false, SEGS_>(EVOSPEC_ARGS))           \
               : (once ? launch_partials_k<TW, KS_, RC, MB_, true, false, true, SEGS_>(EVOSPEC_ARGS)            \
                       : launch_partials_k<TW, KS_, RC, MB_, true, false, false, SEGS_>(EVOSPEC_ARGS)))
#define EVOSPEC_MB(MB_, KS_)                                                                                    \
    if (p.mb == MB_ && p.ks == KS_) {                                                                           \
        if (!full)                                                                                              \
            return bl.packed ? launch_partials_k<TW, KS_, RC, MB_, false, true, false, 1>(EVOSPEC_ARGS)         \
                             : launch_partials_k<TW, KS_, RC, MB_, false, false, false, 1>(EVOSPEC_ARGS);       \
        if constexpr (KS_ <= kSegMaxShare) {                                                                    \
            if (p.segs == 2) return EVOSPEC_FULL(MB_, KS_, 2);                                                  \
        }                                                                                                       \
        return EVOSPEC_FULL(MB_, KS_, 1);                                                                       \
    }
    EVOSPEC_MB(1, 1) EVOSPEC_MB(2, 1) EVOSPEC_MB(4, 1)
    if constexpr (KS2 > 1) { EVOSPEC_MB(2, KS2) }
    if constexpr (KS4 > 1) { EVOSPEC_MB(4, KS4) }
#undef EVOSPEC_MB
#undef EVOSPEC_FULL
#undef EVOSPEC_ARGS
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_partials_batch(const Plan& p, const void* h, const ChunkBatch& cb, const BatchLayout& bl,
                                 int d, const void* W, const int32_t* ids, int V_act, int k, void* keys,
                                 void* stats, hipStream_t stream) {
    if (cb.n < 1 || cb.n > kMaxChunks || bl.chunk_bytes % 8 != 0) return hipErrorInvalidValue;
    if (bl.split && (p.mb != mb_for_rows(kSplitRows) || p.ks != 1)) return hipErrorInvalidValue;      // (the kernels that know it)
    switch (p.nw) {
#define EVOSPEC_SHAPE(TW_, RC_, KS4_, KS2_)                                                     \
    case TW_: return launch_partials_shape<TW_, RC_, KS4_, KS2_>(p, h, cb, bl, d, W, ids, V_act, k, keys, stats, stream);
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
    return launch_partials_batch(p, h, cb, bl, d, W, ids, V_act, k, keys, stats, stream);
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

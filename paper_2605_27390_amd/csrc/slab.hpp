// The slab kernel's workgroup: one slab of the active set against up to 64 draft rows (see slab_partials).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "common.hpp"
#include "plan.hpp"

namespace evospec {

// One problem of a launch: draft rows against a matrix, and where the partials go.
struct SlabProblem {
    const uint16_t* h;           // its first draft row
    int rows;                    // 1..64
    const uint16_t* W;
    const int32_t* ids;          // null: identity
    int V_act;
    u64* keys;
    float2* stats;
};

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
__device__ __forceinline__ void slab_partials(const SlabProblem& pr, int slab, int d, int k, int GL, unsigned char* smem) {
    const uint16_t* __restrict__ h = pr.h;
    const uint16_t* __restrict__ W = pr.W;
    const int32_t* __restrict__ ids = pr.ids;
    u64* __restrict__ part_keys = pr.keys;
    float2* __restrict__ part_stats = pr.stats;
    const int rows = pr.rows, V_act = pr.V_act;
    const int dp = packed_d(d);                    // (a packed matrix pads its rows to whole chunks)
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
    const int row0 = slab * RT;
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
    const int cx = !PACKED && SEGS == 2 ? ((slab >> kTurnBit) & 1) * kSegChunks : 0;
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
        hdst[p] = m * kHStride + (c8 ^ (m & 15)) * 8;
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
    // h in LDS: piece c (16 bytes) of draft row m sits in place c ^ (m mod 16) of its row.  A 128-bit read takes the 64 lanes in four turns
    // of 16, {0-3, 12-15, 20-27} the first, which holds every draft row of the block once: 16 different 16-byte columns of 256 bytes, no
    // bank twice.  (Rows padded by 16 bytes had one conflict in every turn, which doubled its time.)
    // ANEW: the places of four k-steps are found in every chunk.  Kept over the chunks they are registers that seven and eight wavefronts with two blocks of draft
    // rows have no room for beside a second workgroup (packed 51,446 x 2,048 at 24 rows 45.6 us, kept 48.8), nor shared tiles in one segment, which
    // spill (row-major 28,000 x 1,024 at 60 26.0 and 27.7); elsewhere they cost nothing and save the flips (full vocabulary row-major 243.2, kept 241.2).
    constexpr bool ANEW = (KS == 1 && MB == 2 && (TW == 7 || TW == 8)) || (KS == 2 && MB == 4 && SEGS == 1);
    const uint16_t* brow = Hs + n16 * kHStride;
    int bcol[4];                                   // this lane's piece of k-steps 0..3 (4..7: 128 elements on), relative to its row
#pragma unroll
    for (int s = 0; s < 4; ++s) bcol[s] = ((4 * (((KS > 1 ? s0 : 0) + s) & 3) + g) ^ n16) * 8;
    // (k-step 0 of this wavefront is k-step 0, or 2 where it has two, of a group of four: the piece of the s-th has 4 s flipped)
    static_assert(KSTEPS == 8 || KSTEPS == 4 || KSTEPS == 2, "groups of four k-steps");
    int flip0 = bcol[0] + s0 / 4 * 128;            // (ANEW)
    auto load_b = [&](bf16x8 (&b)[MB], int buf, int s) {
        const int at = ANEW ? (flip0 ^ (s & 3) * 32) + s / 4 * 128 : bcol[s & 3] + ((KS > 1 ? s0 : 0) + s) / 4 * 128;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) b[mb] = *reinterpret_cast<const bf16x8*>(brow + ((size_t)buf * MR + mb * 16) * kHStride + at);
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
        if constexpr (ANEW) asm volatile("" : "+v"(flip0));
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
        u64* outk = part_keys + ((size_t)slab * kMTile + m) * k;
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
            part_stats[(size_t)slab * kMTile + m] = make_float2(vmax[m], sum);
        }
    }
}

}  // namespace evospec

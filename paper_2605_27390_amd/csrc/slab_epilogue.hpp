// Epilogue shared by the matrix-tile kernels (gemm.hip, tile.hip): one wavefront reduces the logits of a
// slab of 128 active rows and 16 * NMB draft rows, which it holds in accumulators, to one partial per
// draft row: (max, sum-exp) and the logits that can still be among the row's k best, unranked, as (logit,
// id) pairs; the merge kernel ranks them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"
#include "plan.hpp"

namespace evospec {

constexpr int kGFastLen = 16;                 // list length the staged common path of the epilogue handles
// LDS per wavefront: the staged lists and spare slots of the common path, or a block's parked logits; then ids
constexpr int epi_lists(int nmb) {
    const int common = nmb * 16 * kGFastLen * 8 + 64 * 8, rare = 64 * 32 * 4;
    return common > rare ? common : rare;
}
// and the logits of a block, where survivors are picked one by one
constexpr int epi_bytes(int nmb) { return epi_lists(nmb) + 64 * 32 * 4 + kGemmSlab * 4; }

// Accumulators are pinned to the accumulation registers: the register allocator must
// not be left to shuffle them through the other file or among themselves.  (The compiler does not see that
// these are matrix instructions: wait out the last ones before the accumulators are read.)
__device__ __forceinline__ void mfma_acc(f32x4& c, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// The 4 lanes n16, n16+16, n16+32, n16+48 (one per 16-lane row of the wavefront) hold the four
// quarters of a draft row's logits.  v_permlane16_swap exchanges the odd rows of its first operand
// with the even rows of the second, v_permlane32_swap the upper half of the first with the lower
// half of the second: applied to two copies of x they hand every lane both members of its pair of
// rows, then of its pair of halves.
// N independent values at a time, stage by stage (the scheduler is fenced in between).
template <int N>
__device__ __forceinline__ void quad_max(float (&x)[N]) {
    float y[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
        x[i] = __uint_as_float(a[0]); y[i] = __uint_as_float(a[1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = fmaxf(x[i], y[i]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
        x[i] = __uint_as_float(b[0]); y[i] = __uint_as_float(b[1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = fmaxf(x[i], y[i]);
    __builtin_amdgcn_sched_barrier(0);
}
template <int N>
__device__ __forceinline__ void quad_sum(float (&x)[N]) {
    float y[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
        x[i] = __uint_as_float(a[0]); y[i] = __uint_as_float(a[1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += y[i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i]), false, false);
        x[i] = __uint_as_float(b[0]); y[i] = __uint_as_float(b[1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += y[i];
    __builtin_amdgcn_sched_barrier(0);
}
// q[r] = x of the lane in row r (lane n16 + 16 r)
__device__ __forceinline__ void quad_all(uint32_t x, uint32_t (&q)[4]) {
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);      // a[0]: rows {0,0,2,2}, a[1]: rows {1,1,3,3}
    const auto e = __builtin_amdgcn_permlane32_swap(a[0], a[0], false, false);  // e[0]: row 0 everywhere, e[1]: row 2
    const auto o = __builtin_amdgcn_permlane32_swap(a[1], a[1], false, false);  // o[0]: row 1 everywhere, o[1]: row 3
    q[0] = e[0]; q[1] = o[0]; q[2] = e[1]; q[3] = o[1];
}

// The bound of draft row `row` (-inf: none; +inf for rows past the last): see RowBound.
__device__ __forceinline__ float row_bound(const RowBound& b, int row, int M) {
    if (row >= M) return INFINITY;
    int c = 0, first = 0;
    for (int i = 1; i < b.n_chunks; ++i)
        if (b.m0[i] <= row) { c = i; first = b.m0[i]; }
    const u64* p = b.keys + (size_t)c * b.chunk_keys + (size_t)(row - first) * b.k + (b.q - 1);
    uint32_t v[kBoundLists];
#pragma unroll
    for (int i = 0; i < kBoundLists; ++i) v[i] = i < b.n_lists ? (uint32_t)(p[(size_t)i * kMTile * b.k] >> 32) : 0u;
    // Batcher's odd-even merge sort, descending
#pragma unroll
    for (int n = 1; n < kBoundLists; n *= 2)
#pragma unroll
        for (int m = n; m >= 1; m /= 2)
#pragma unroll
            for (int x = 0; x + m < kBoundLists; ++x)
                if (x >= m % n && ((x - m % n) / m) % 2 == 0 && x / (2 * n) == (x + m) / (2 * n)) {
                    const uint32_t hi = v[x] > v[x + m] ? v[x] : v[x + m];
                    v[x + m] = v[x] > v[x + m] ? v[x + m] : v[x];
                    v[x] = hi;
                }
    uint32_t t = 0;
#pragma unroll
    for (int i = 0; i < kBoundLists; ++i) t = i == b.sets - 1 ? v[i] : t;
    // (0: fewer lists hold q keys; above infinity: NaN, which bounds nothing)
    return t != 0u && t <= 0xff800000u ? ordered_to_f32(t) : -INFINITY;
}

// acc[rg][mb]: lane (n16, g) holds the logits of the active rows vrow0 + 16 rg + 4 g + 0..3 and draft row
// mbase + 16 mb + n16.  `my`: epi_bytes(NMB) of LDS of this wavefront alone.  Lists are laid out [draft
// row][slab][slot].  NMB <= 8.  bnd (or null): in LDS, for each of the draft rows a value that k logits elsewhere reach, so
// that none below it can be among the row's k best.
// ACC: the accumulators sit in the accumulation registers.  HAS_BND: bnd may be given.
template <int NMB, bool ACC = true, bool HAS_BND = true>
__device__ __forceinline__ void slab_epilogue(f32x4 (&acc)[8][NMB], unsigned char* my, int vrow0, int mbase, int M, int V_act,
                                              const int32_t* __restrict__ ids, int k, int list_len, int slab, int n_slabs, const float* bnd,
                                              u64* __restrict__ part_keys, float2* __restrict__ part_stats) {
    const int lane = threadIdx.x & 63, n16 = lane & 15, g = lane >> 4;
    const int nvalid = min(kGemmSlab, V_act - vrow0);
    // common path: [NMB][16][16] staged lists of all blocks, then one spare slot per lane;
    // rare path (afterwards, same bytes): [64][32] parked logits of a block
    u64* flist = reinterpret_cast<u64*>(my);
    float* zpark = reinterpret_cast<float*>(my);
    int32_t* Ids = reinterpret_cast<int32_t*>(my + epi_bytes(NMB) - kGemmSlab * 4);   // [128]

#pragma unroll
    for (int i = 0; i < kGemmSlab / 64; ++i) {
        const int r = vrow0 + lane + 64 * i;
        Ids[lane + 64 * i] = r < V_act ? (ids ? ids[r] : r) : 0x7fffffff;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    // lane's entries: active row (within the quadrant) 16 rg + 4 g + j  <->  bit 4 rg + j
    uint32_t vmask = 0;
#pragma unroll
    for (int rg = 0; rg < 8; ++rg)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (rg * 16 + 4 * g + j < nvalid) vmask |= 1u << (4 * rg + j);
    if (nvalid < kGemmSlab) {                                      // ragged last slab: rows past the end never win
#pragma unroll
        for (int rg = 0; rg < 8; ++rg)
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (!((vmask >> (4 * rg + j)) & 1u)) acc[rg][mb][j] = -INFINITY;
    }

    // A wavefront runs alone on its SIMD here, so nothing hides a latency but its own independent
    // work: every phase below runs over all NMB blocks of 16 draft rows before the next one starts.
    // Lane (n16, g) holds, for draft row n16 of block mb, the 32 logits acc[0..7][mb][0..3]; the
    // row's 128 logits are spread over the 4 lanes g = 0..3, which exchange values with the
    // row-swap instructions (no LDS round trip).

    // (an empty statement that "rewrites" the accumulators where they sit: copies read into
    // ordinary registers by one phase are dropped instead of being carried, and spilled, to the next)
    auto repin = [&]() {
#pragma unroll
        for (int rg = 0; rg < 8; ++rg)
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) {
                if constexpr (ACC) asm volatile("" : "+a"(acc[rg][mb]));
                else asm volatile("" : "+v"(acc[rg][mb]));
            }
    };
    repin();
    // Dependent vector instructions of one wavefront issue many cycles apart, so each phase is
    // written as stages over the independent blocks (NMB instructions per stage) and the
    // scheduler is fenced between stages so that it keeps them that way.
#define EVOSPEC_FENCE() __builtin_amdgcn_sched_barrier(0)
#define EVOSPEC_MB(body) _Pragma("unroll") for (int mb = 0; mb < NMB; ++mb) { body; } EVOSPEC_FENCE();

    // -- phase 1: maxima of the 32 groups of 4 logits of every row, and the row maximum
    float t[NMB][8], vm[NMB];
#pragma unroll
    for (int rg = 0; rg < 8; ++rg) {
        float p0[NMB], p1[NMB];
        EVOSPEC_MB(p0[mb] = fmaxf(acc[rg][mb][0], acc[rg][mb][1]))
        EVOSPEC_MB(p1[mb] = fmaxf(acc[rg][mb][2], acc[rg][mb][3]))
        EVOSPEC_MB(t[mb][rg] = fmaxf(p0[mb], p1[mb]))
    }
    {
        float p0[NMB], p1[NMB], p2[NMB], p3[NMB];
        EVOSPEC_MB(p0[mb] = fmaxf(t[mb][0], t[mb][1]))
        EVOSPEC_MB(p1[mb] = fmaxf(t[mb][2], t[mb][3]))
        EVOSPEC_MB(p2[mb] = fmaxf(t[mb][4], t[mb][5]))
        EVOSPEC_MB(p3[mb] = fmaxf(t[mb][6], t[mb][7]))
        EVOSPEC_MB(p0[mb] = fmaxf(p0[mb], p1[mb]))
        EVOSPEC_MB(p2[mb] = fmaxf(p2[mb], p3[mb]))
        EVOSPEC_MB(vm[mb] = fmaxf(p0[mb], p2[mb]))
        quad_max(vm);
    }

    repin();
    // -- phase 2: sum of exponentials, exp(z - vm) = 2^(z log2(e) - vm log2(e)), two running sums per block
    float se[NMB];
    {
        float nvm[NMB], s0[NMB], s1[NMB];
        EVOSPEC_MB(nvm[mb] = -vm[mb] * 1.44269504f; s0[mb] = 0.f; s1[mb] = 0.f)
#pragma unroll
        for (int rg = 0; rg < 8; ++rg) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x[NMB];
                EVOSPEC_MB(x[mb] = __builtin_fmaf(acc[rg][mb][j], 1.44269504f, nvm[mb]))
                EVOSPEC_MB(x[mb] = __builtin_amdgcn_exp2f(x[mb]))
                if (j & 1) { EVOSPEC_MB(s1[mb] += x[mb]) } else { EVOSPEC_MB(s0[mb] += x[mb]) }
            }
        }
        EVOSPEC_MB(se[mb] = s0[mb] + s1[mb])
        quad_sum(se);
    }
    const int mrow0 = mbase + n16;                                 // draft row of block 0
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb)
        if (g == 0 && mrow0 + 16 * mb < M) part_stats[(size_t)(mrow0 + 16 * mb) * n_slabs + slab] = make_float2(vm[mb], se[mb]);

    // -- phase 3: a lower bound of every row's k-th best logit, and what reaches it: at most a list's length.  Three ways to
    // a bound, each tried on all rows of the wavefront where the one before leaves any row more than that:
    // (0) from elsewhere (bnd).  It costs nothing here, and about one logit of a row reaches it if the logits here and there are alike.
    // If they are larger here, most may (16 x 60 rows over 32,768 + 2,048 x 4,096, us for the call without bnd, with it alone and with
    // the next: 305, 296 and 295; extensions of half the size 305, 368 and 311; of a hundredth 306, 491 and 312).
    // (1) The slab's own, up to k = kOwnBoundK: each lane sorts its 8 group maxima; k rounds then take the largest head of the row's 4 lanes and
    // pop it wherever it is the head: at least k group maxima, hence k logits, reach the last value taken.
    // (2) By halving the interval between a value that too many reach and the row's maximum, until between k and a list's length do,
    // some 4 to 8 times: a ragged last slab with too few groups for (1), k past it.  (One row after the other, as all such rows used to
    // go, and by halves, us: 20,000 x 2,048 at 256 rows, k = 16 90 and 53, k = 30 93 and 56, k = 60 126 and 69; 14,877 x 1,024 at
    // 200, a last slab of 29 rows, 39 and 24.)
    // Up to kFewOver such rows in a wavefront go one after the other all the same, which is sooner done: with a bound of (1) one row in a few hundred is left, and
    // halving was 1 us more on a small launch (5,000 x 768 at 400 rows 22.4 us, by halves 23.5; 8,192 x 1,024 at 256 23.7 and 24.7).
    // (Blocks of 128 draft rows to a wavefront have no registers for (2), nor for the longer lists below: such rows go one by one.)
    constexpr bool kRoom = NMB <= 2;
    const int cap = list_len == kGFastLen ? kGFastLen : (kRoom ? list_len : -1);
    constexpr int kFewOver = 3;
    constexpr int kHalvings = 20;                                  // (what is left then has equal logits, or next to equal ones)
    float tau[NMB];
#pragma unroll
    for (int mb = 0; mb < NMB; ++mb) tau[mb] = -INFINITY;
    if (HAS_BND && bnd) {                                          // (uniform)
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) tau[mb] = bnd[16 * mb + n16];
    }
    uint32_t mask[NMB];
    // survivors per lane (<= 32), four blocks to a register; from the 4 lanes of a row: the offset
    // of this lane's survivors in the row's list and the list length L (<= 128), still packed
    constexpr int NPK = (NMB + 3) / 4;
    uint32_t basep[NPK], Lp[NPK];
    auto length = [&](int mb) { return (int)((Lp[mb >> 2] >> (8 * (mb & 3))) & 0xff); };
    // what reaches x: mask, basep and Lp
    auto reach = [&](const float (&x)[NMB]) {
        // survivor masks without a compare per entry: the sign of (logit - bound) is
        // shifted in, last entry first, so that entry i ends up as bit i ("below the bound")
        uint32_t below[NMB];
        EVOSPEC_MB(below[mb] = 0u)
#pragma unroll
        for (int i = 31; i >= 0; --i) {
            float df[NMB];
            EVOSPEC_MB(df[mb] = acc[i >> 2][mb][i & 3] - x[mb])
            EVOSPEC_MB(below[mb] = __builtin_amdgcn_alignbit(below[mb], __float_as_uint(df[mb]), 31))
        }
        EVOSPEC_MB(mask[mb] = ~below[mb] & vmask)
#pragma unroll
        for (int hf = 0; hf < NPK; ++hf) {
            uint32_t pk = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * hf + q < NMB) pk |= (uint32_t)__popc(mask[4 * hf + q]) << (8 * q);
            uint32_t q[4];
            quad_all(pk, q);
            basep[hf] = (g > 0 ? q[0] : 0u) + (g > 1 ? q[1] : 0u) + (g > 2 ? q[2] : 0u);
            Lp[hf] = q[0] + q[1] + q[2] + q[3];
        }
    };
    auto over = [&]() {                                            // rows with more than that (the 4 lanes of a row agree)
        int n = 0;
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) n += __popcll(__ballot(length(mb) > cap));
        return n / 4;
    };
    float lo[NMB], hi[NMB];                                        // (2) the interval of an open row
    uint32_t fixed = 0;                                            // bit mb: the row's bound stands
    for (int it = HAS_BND && bnd ? -1 : 0;; ++it) {                // (uniform)
        if (it == 0 && k <= (kRoom ? kOwnBoundK : 32)) {
            float own[NMB];
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) own[mb] = -INFINITY;
#define EVOSPEC_CE(I, J) { float hi[NMB]; EVOSPEC_MB(hi[mb] = fmaxf(t[mb][I], t[mb][J])) \
                           EVOSPEC_MB(t[mb][J] = fminf(t[mb][I], t[mb][J])) EVOSPEC_MB(t[mb][I] = hi[mb]) }
            EVOSPEC_CE(0, 1) EVOSPEC_CE(2, 3) EVOSPEC_CE(4, 5) EVOSPEC_CE(6, 7)
            EVOSPEC_CE(0, 2) EVOSPEC_CE(1, 3) EVOSPEC_CE(4, 6) EVOSPEC_CE(5, 7)
            EVOSPEC_CE(1, 2) EVOSPEC_CE(5, 6) EVOSPEC_CE(0, 4) EVOSPEC_CE(3, 7)
            EVOSPEC_CE(1, 5) EVOSPEC_CE(2, 6)
            EVOSPEC_CE(1, 4) EVOSPEC_CE(3, 6)
            EVOSPEC_CE(2, 4) EVOSPEC_CE(3, 5)
            EVOSPEC_CE(3, 4)
#undef EVOSPEC_CE
            for (int r = 0; r < k; ++r) {
                EVOSPEC_MB(own[mb] = t[mb][0])
                quad_max(own);
                // pop the head where it is the value just taken: all ones / zero select, no compare chain
                uint32_t pop[NMB];
                EVOSPEC_MB(pop[mb] = t[mb][0] == own[mb] ? ~0u : 0u)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    EVOSPEC_MB(const uint32_t cur = __float_as_uint(t[mb][i]);
                               const uint32_t nxt = i < 7 ? __float_as_uint(t[mb][i + 1]) : 0xff800000u;
                               t[mb][i] = __uint_as_float((pop[mb] & nxt) | (~pop[mb] & cur)))
                }
            }
            EVOSPEC_MB(tau[mb] = fmaxf(tau[mb], own[mb]))
        }
        repin();
        reach(tau);
        if (it >= 0) {
            bnd = nullptr;
            if (!kRoom) break;
        }
        if (it <= 0) {
            const int n = over();
            if (n == 0 || (it == 0 && n <= kFewOver)) break;
            if (it < 0) continue;
        }
        if constexpr (kRoom) {
            if (it == 0) {
                // the least logit of the row, where nothing better is known
                float least[NMB];
                EVOSPEC_MB(least[mb] = -INFINITY)
#pragma unroll
                for (int i = 0; i < 32; ++i) { EVOSPEC_MB(least[mb] = fmaxf(least[mb], (vmask >> i) & 1u ? -acc[i >> 2][mb][i & 3] : -INFINITY)) }
                quad_max(least);
                EVOSPEC_MB(lo[mb] = fmaxf(tau[mb], -least[mb]); hi[mb] = vm[mb]; fixed |= length(mb) <= cap ? 1u << mb : 0u)
            } else {
#pragma unroll
                for (int mb = 0; mb < NMB; ++mb) {
                    const bool open = !((fixed >> mb) & 1u), enough = length(mb) >= k;
                    lo[mb] = open && enough ? tau[mb] : lo[mb];
                    hi[mb] = open && !enough ? tau[mb] : hi[mb];
                    fixed |= enough && length(mb) <= cap ? 1u << mb : 0u;
                }
            }
            // (after the last halving a look at the lower end, which enough reach)
            if (__ballot(fixed != (1u << NMB) - 1u) == 0 || it > kHalvings) break;
            EVOSPEC_MB(tau[mb] = (fixed >> mb) & 1u ? tau[mb] : (it == kHalvings ? lo[mb] : 0.5f * lo[mb] + 0.5f * hi[mb]))
        }
    }
    bool rare = false;

    repin();
    // -- phase 4: the survivors of every row, as (logit, id) pairs in no particular order.  Up to k = 16 they are
    // gathered into the row's 16-slot list in LDS (empty slots: all ones) and the lists copied to the
    // workspace a full line at a time; the merge ranks.  No branch or compare per entry: an entry
    // that is not a survivor goes to the lane's spare slot.
    if (!kRoom || list_len == kGFastLen) {
        const u32x4 ones = {~0u, ~0u, ~0u, ~0u};
#pragma unroll
        for (int it = 0; it < NMB * 16 * kGFastLen * 8 / 1024; ++it)
            *reinterpret_cast<u32x4*>(my + (it * 64 + lane) * 16) = ones;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const uint32_t spare_a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u64*)(flist + NMB * 16 * kGFastLen + lane);
        uint32_t mk[NMB], rel[NMB];                                    // survivor mask; row list start - spare slot (bytes)
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
            const int base = (basep[mb >> 2] >> (8 * (mb & 3))) & 0xff;
            const int L = length(mb);
            rare = rare || L > cap;
            mk[mb] = L <= cap ? mask[mb] : 0u;
            rel[mb] = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) u64*)(flist + (mb * 16 + n16) * kGFastLen + base) - spare_a;
        }
        EVOSPEC_FENCE();
        if (HAS_BND && bnd) {
            // Few survivors (a list's at most, mostly about one to a row): block by block the logits are laid out in LDS, where each lane picks
            // its own survivors one after the other.  (Both this and the bound: 16 x 60 rows over 32,768 + 2,048 rows x 4,096
            // 304 -> 297 us for the call.)
            unsigned char* zl = my + epi_lists(NMB) + lane * 16;       // [8][64] f32x4
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb) {
#pragma unroll
                for (int rg = 0; rg < 8; ++rg) *reinterpret_cast<f32x4*>(zl + rg * 1024) = acc[rg][mb];
                uint32_t m = mk[mb], at = spare_a + rel[mb];
                while (__ballot(m != 0u) != 0) {
                    if (m != 0u) {
                        const int i = __builtin_ctz(m);
                        m &= m - 1;
                        const uint32_t z = *reinterpret_cast<const uint32_t*>(zl + (i >> 2) * 1024 + (i & 3) * 4);
                        const uint32_t id = (uint32_t)Ids[16 * (i >> 2) + 4 * g + (i & 3)];
                        *(__attribute__((address_space(3))) u64*)(uintptr_t)at = ((u64)z << 32) | id;
                        at += 8;
                    }
                }
            }
        } else {
            int32_t idv[32];                                               // full-vocabulary ids of the lane's entries
#pragma unroll
            for (int rg = 0; rg < 8; ++rg) {
                const int4 q = *reinterpret_cast<const int4*>(Ids + rg * 16 + 4 * g);
                idv[4 * rg + 0] = q.x; idv[4 * rg + 1] = q.y; idv[4 * rg + 2] = q.z; idv[4 * rg + 3] = q.w;
            }
            repin();                                               // (or the logits are read out of their registers for both branches at once, and spilled)
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                uint32_t at[NMB], sel[NMB];
                EVOSPEC_MB(at[mb] = mk[mb] & ((1u << i) - 1u))
                EVOSPEC_MB(at[mb] = __popc(at[mb]))
                EVOSPEC_MB(sel[mb] = (uint32_t)__builtin_amdgcn_sbfe((int)mk[mb], i, 1))
                EVOSPEC_MB(at[mb] = rel[mb] + 8u * at[mb])
                EVOSPEC_MB(at[mb] &= sel[mb])
                EVOSPEC_MB(at[mb] += spare_a)
                EVOSPEC_MB(*(__attribute__((address_space(3))) u64*)(uintptr_t)at[mb] =
                               ((u64)__float_as_uint(acc[i >> 2][mb][i & 3]) << 32) | (uint32_t)idv[i])
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // piece p = 64 it + lane of the staged lists: block p / 128, row (p / 8) % 16, 16 bytes p % 8
#pragma unroll
        for (int it = 0; it < 2 * NMB; ++it) {
            const int mb = it >> 1, r16 = ((it & 1) << 3) | (lane >> 3);
            const int m = mbase + 16 * mb + r16;
            const u32x4 q = *reinterpret_cast<const u32x4*>(my + (it * 64 + lane) * 16);
            const int L = __builtin_amdgcn_ds_bpermute(4 * r16, (Lp[mb >> 2] >> (8 * (mb & 3))) & 0xff);     // (lane r16 belongs to row r16)
            if (L <= cap && m < M)
                *reinterpret_cast<u32x4*>(part_keys + ((size_t)m * n_slabs + slab) * kGFastLen + 2 * (lane & 7)) = q;
        }
    } else if constexpr (kRoom) {
        // Longer lists: block by block the logits are laid out in LDS, each lane takes its own survivors to their places one after the
        // other (some k / 4 of them), the four lanes of a row fill the rest of its list.
        unsigned char* zl = my + lane * 16;                            // [8][64] f32x4
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
#pragma unroll
            for (int rg = 0; rg < 8; ++rg) *reinterpret_cast<f32x4*>(zl + rg * 1024) = acc[rg][mb];
            const int L = length(mb), m = mrow0 + 16 * mb;
            rare = rare || L > cap;
            const bool out = L <= cap && m < M;
            u64* dst = part_keys + ((size_t)(out ? m : 0) * n_slabs + slab) * list_len;
            uint32_t mk = out ? mask[mb] : 0u;
            int at = (basep[mb >> 2] >> (8 * (mb & 3))) & 0xff;
            while (__ballot(mk != 0u) != 0) {
                if (mk != 0u) {
                    const int i = __builtin_ctz(mk);
                    mk &= mk - 1;
                    const uint32_t z = *reinterpret_cast<const uint32_t*>(zl + (i >> 2) * 1024 + (i & 3) * 4);
                    const uint32_t id = (uint32_t)Ids[16 * (i >> 2) + 4 * g + (i & 3)];
                    dst[at++] = ((u64)z << 32) | id;
                }
            }
            if (out)
                for (int e = L + g; e < list_len; e += 4) dst[e] = ~0ull;
        }
    }
#undef EVOSPEC_MB
#undef EVOSPEC_FENCE
    if (__ballot(rare) == 0) return;
    repin();

    // -- rows with more survivors than a list holds whatever the bound (equal logits, infinities), one after the other: the whole wavefront takes the row, two logits to a
    // lane, finds its k-th largest bit by bit and keeps what reaches it.  The block's logits are parked in LDS.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // the staged lists have been read
    float* zbuf = zpark + lane * 32;
    for (int mbr = 0; mbr < NMB; ++mbr) {
        const int L = (Lp[mbr >> 2] >> (8 * (mbr & 3))) & 0xff;    // (mbr is no constant)
        uint32_t todo = (uint32_t)__ballot(mrow0 + 16 * mbr < M && L > cap) & 0xffffu;       // (the 4 lanes of a row agree)
        if (todo == 0) continue;
#pragma unroll
        for (int mb = 0; mb < NMB; ++mb) {
            if (mb != mbr) continue;                               // uniform
#pragma unroll
            for (int rg = 0; rg < 8; ++rg) *reinterpret_cast<f32x4*>(zbuf + 4 * rg) = acc[rg][mb];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        while (todo) {
            const int r = __builtin_ctz(todo);
            todo &= todo - 1;
            // entries i0, i0 + 1 of the row's quarter g: active row 16 (i / 4) + 4 g + i % 4
            const int i0 = 2 * n16, a0 = 16 * (i0 >> 2) + 4 * g + (i0 & 3);
            const float2 z = *reinterpret_cast<const float2*>(zpark + (r + 16 * g) * 32 + i0);
            const int2 id = *reinterpret_cast<const int2*>(Ids + a0);
            const uint32_t o0 = a0 < nvalid ? f32_to_ordered(z.x) : 0u, o1 = a0 + 1 < nvalid ? f32_to_ordered(z.y) : 0u;
            // a value that at least q and at most `most` of the 128 reach, if there is one; else the largest that
            // q reach (found bit by bit; between 10 and 16 of 128 it takes some 12 of the 32 steps)
            auto kth = [&](uint32_t x0, uint32_t x1, int q, int most) {
                uint32_t t = 0;
                for (int bit = 31; bit >= 0; --bit) {
                    const uint32_t c = t | (1u << bit);
                    const int n = __popcll(__ballot(x0 >= c)) + __popcll(__ballot(x1 >= c));
                    if (n >= q) {
                        t = c;
                        if (n <= most) break;
                    }
                }
                return t;
            };
            uint32_t th = kth(o0, o1, k, list_len);
            // fewer than k rows: all of them down to -inf (a NaN with its sign set, below that in this order, is no
            // survivor above and no candidate here)
            th = th > 0x007fffffu ? th : 0x007fffffu;
            bool in0 = o0 >= th, in1 = o1 >= th;
            if (__popcll(__ballot(in0)) + __popcll(__ballot(in1)) > list_len) {
                // equal logits at the k-th place: the smallest ids among them
                const int need = k - __popcll(__ballot(o0 > th)) - __popcll(__ballot(o1 > th));
                const uint32_t l0 = o0 == th ? ~(uint32_t)id.x : 0u, l1 = o1 == th ? ~(uint32_t)id.y : 0u;
                const uint32_t tl = kth(l0, l1, need, need);
                in0 = o0 > th || (o0 == th && l0 >= tl);
                in1 = o1 > th || (o1 == th && l1 >= tl);
            }
            const u64 b0 = __ballot(in0), b1 = __ballot(in1);
            const int n0 = __popcll(b0), n = n0 + __popcll(b1);
            auto before = [&](u64 bal) { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u)); };
            u64* dst = part_keys + ((size_t)(mbase + 16 * mbr + r) * n_slabs + slab) * list_len;
            const int p0 = before(b0), p1 = n0 + before(b1);
            if (in0 && p0 < list_len) dst[p0] = ((u64)__float_as_uint(z.x) << 32) | (uint32_t)id.x;
            if (in1 && p1 < list_len) dst[p1] = ((u64)__float_as_uint(z.y) << 32) | (uint32_t)id.y;
            for (int e = n + lane; e < list_len; e += 64) dst[e] = ~0ull;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

}  // namespace evospec

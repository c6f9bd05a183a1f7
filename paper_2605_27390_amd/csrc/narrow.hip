// The restricted head for a few draft rows (Eq. 1 of the EvoSpec paper on the active set of Eq. 3;
// one depth of the draft tree, or the exact search of Path A): M <= 16, one block of MFMA columns.
//
// With so few rows all of h fits the registers of a compute unit, so nothing but W_act has to move
// while the kernel runs.  A workgroup of 8 wavefronts takes a run of 16-row tiles; the hidden
// dimension is dealt out to its wavefronts (unit u, a pair of k-steps = 64 elements, to wavefront
// u % 8), each keeps its units of h in registers for the whole launch and streams its part of
// one tile after the other through a ring of registers.  There is no LDS traffic and no barrier in
// the stream, and all 8 wavefronts read one contiguous run of memory together (a packed tile).
// Bound by HBM: 151,936 x 4,096 row-major at one row 227 -> 185 us (6.7 TB/s; the slab kernel before, which
// stages h in LDS behind a barrier per 256 elements), 18,432 x 4,096 packed at 8 rows 30.1 -> 28.8 us.
// Their partial sums of a tile (1 KB each) meet in LDS; after a group of tiles they are added in
// wavefront order, while the loads of the next group are under way.  The logits of the workgroup
// stay in LDS until its last tile, then one wavefront per draft row takes the maximum, the sum of
// exponentials and the k best.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "plan.hpp"

namespace evospec {

namespace {

constexpr int kNW = kNarrowWaves;
constexpr int kNG = kNarrowGroup;
constexpr int kNJ = kNarrowMaxTiles * 16 / 64;     // logits per lane when one wavefront takes a draft row

}  // namespace

// KU units per wavefront and tile, R tiles in the ring.  A unit of a packed tile is two 1 KB blocks, the
// operands of its two k-steps as they are.  On a row-major matrix the first load of a unit takes whole
// 128-byte lines of the rows 0..7, the second of the rows 8..15 (lane (n, g): row n % 8, 16-byte piece g
// or g + 4 of the line), and permutes within 16 lanes turn them into the same two operands.  (A load per
// operand would take half lines of 16 rows.)  Both layouts add in the same order.
// ONCE: the weights are loaded past the caches (see streams_once).
template <int KU, int R, bool PACKED, bool ONCE>
__global__ void __launch_bounds__(kNW * 64)
lmhead_narrow_kernel(const uint16_t* __restrict__ h, int M, int d, const uint16_t* __restrict__ W,
                     const int32_t* __restrict__ ids, int V_act, int k, int base_tiles, int rem_tiles, int z_stride,
                     u64* __restrict__ part_keys, float2* __restrict__ part_stats) {
    constexpr int U = 2;                                    // k-steps per unit
    extern __shared__ __align__(16) unsigned char smem[];
    float* red = reinterpret_cast<float*>(smem);                                   // [kNG][kNW][16][16] partial sums of a group
    u64* list = reinterpret_cast<u64*>(smem);                                      // afterwards: [kNW][z_stride] candidates
    constexpr size_t red_bytes = (size_t)kNG * kNW * 1024;
    float* Z = reinterpret_cast<float*>(smem + red_bytes);                         // [M][z_stride] logits
    int32_t* Ids = reinterpret_cast<int32_t*>(Z + (size_t)M * z_stride);           // [rows of the workgroup]

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;
    const int b = blockIdx.x, n_wg = gridDim.x;
    const int T = base_tiles + (b < rem_tiles ? 1 : 0);                            // this workgroup's tiles
    // The tiles b, b + n_wg, ...: all workgroups walk through memory side by side.  (Runs of neighbouring
    // tiles instead: 29.7 against 28.8 us at 18,432 x 4,096 and 8 rows.)
    auto row_of = [&](int t) { return (b + t * n_wg) * 16; };
    const int n_valid = (T - 1) * 16 + min(16, V_act - row_of(T - 1));             // only the last tile of all can be ragged
    const u32x4 zero4 = {0u, 0u, 0u, 0u};

    // where this lane finds its part of unit s of tile t, and whether it lies inside the rows (d need not
    // be a multiple of the unit; a packed tile is zero there)
    const int dp = packed_d(d);
    const int pl = PACKED ? 0 : n16 & 7;                    // row-major: row within the 8, piece of the first load
    const int p1 = g + ((n16 >> 3) << 2), p2 = g + (((n16 >> 3) ^ 1) << 2);
    const size_t tile_elems = (size_t)16 * dp;
    const uint16_t* wl = W + lane * 8;                      // packed
    const int n_units = dp / 64;
    auto load_unit = [&](u32x4 (&x)[U], int t, int s) {
        if constexpr (PACKED) {
            const int u = s * kNW + w, uc = min(u, n_units - 1);                   // (only the last s can lie past the end)
            const uint16_t* p = wl + (size_t)(b + t * n_wg) * tile_elems + (size_t)uc * 1024;
            x[0] = ONCE ? load_once((gvec_ptr)p) : *(gvec_ptr)p;
            x[1] = ONCE ? load_once((gvec_ptr)(p + 512)) : *(gvec_ptr)(p + 512);
            if (s == KU - 1 && u != uc) x[0] = x[1] = zero4;
        } else {
            const int c0 = (s * kNW + w) * 64;              // first element of the unit's line
            const int ra = min(row_of(t) + pl, V_act - 1), rb = min(row_of(t) + 8 + pl, V_act - 1);   // past the end: a valid row, masked later
            const int ca = c0 + 8 * p1, cb = c0 + 8 * p2;
            const gvec_ptr pa = (gvec_ptr)(W + (size_t)ra * d + (ca < d ? ca : d - 8)), pb = (gvec_ptr)(W + (size_t)rb * d + (cb < d ? cb : d - 8));
            const u32x4 va = ONCE ? load_once(pa) : *pa, vb = ONCE ? load_once(pb) : *pb;
            x[0] = ca < d ? va : zero4;
            x[1] = cb < d ? vb : zero4;
        }
    };

    // h: operand of k-step q of unit s: draft row n16 (past the last: repeated, never read back), elements 8g..8g+7
    bf16x8 hb[KU][U];
#pragma unroll
    for (int s = 0; s < KU; ++s)
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int e = ((s * kNW + w) * U + q) * 32 + 8 * g;
            const u32x4 v = *(gvec_ptr)(h + (size_t)min(n16, M - 1) * d + (e < d ? e : d - 8));
            hb[s][q] = __builtin_bit_cast(bf16x8, e < d ? v : zero4);
        }
    u32x4 ring[R][KU][U];
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r < T) {
#pragma unroll
            for (int s = 0; s < KU; ++s) load_unit(ring[r][s], r, s);
        }
    for (int i = tid; i < T * 16; i += kNW * 64) {
        const int row = row_of(i >> 4) + (i & 15);
        Ids[i] = row < V_act ? (ids ? ids[row] : row) : 0x7fffffff;
    }

    // one tile out of ring slot r; refill with tile t + R behind the k-steps
    auto tile = [&](auto slot, int t, bool refill) {
        constexpr int r = decltype(slot)::value;
        f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < KU; ++s) {
            if constexpr (PACKED) {
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ring[r][s][0]), hb[s][0], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ring[r][s][1]), hb[s][1], acc[1], 0, 0, 0);
            } else {
                u32x4 a0, a1;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    a0[i] = pick_bank(ring[r][s][0][i], ring[r][s][1][i]);
                    a1[i] = pick_bank_ror8(ring[r][s][0][i], ring[r][s][1][i]);
                }
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), hb[s][0], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), hb[s][1], acc[1], 0, 0, 0);
            }
            if (refill) load_unit(ring[r][s], t + R, s);
        }
        acc[0] += acc[1];
        // z partial of active row 4 g + j, draft row n16
        *reinterpret_cast<f32x4*>(red + ((size_t)((t % kNG) * kNW + w) * 16 + n16) * 16 + 4 * g) = acc[0];
    };
    // after a group: logits = the 8 partial sums, added in wavefront order
    auto reduce = [&](int t0, int n) {
        lds_barrier();
        for (int i = tid; i < n * M * 4; i += kNW * 64) {
            const int tt = i / (M * 4), rest = i - tt * (M * 4), m = rest >> 2, q = rest & 3;
            const float* p = red + (size_t)tt * (kNW * 256) + m * 16 + 4 * q;
            f32x4 x = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
            for (int ww = 1; ww < kNW; ++ww) x += *reinterpret_cast<const f32x4*>(p + ww * 256);
            *reinterpret_cast<f32x4*>(Z + (size_t)m * z_stride + (t0 + tt) * 16 + 4 * q) = x;
        }
        lds_barrier();
    };
    static_assert(kNG % R == 0, "a group is a whole number of ring turns");
#define EVOSPEC_TURN(REFILL)                                                               \
    if constexpr (R > 0) tile(std::integral_constant<int, 0>{}, t, REFILL);                \
    if constexpr (R > 1) tile(std::integral_constant<int, (R > 1 ? 1 : 0)>{}, t + 1, REFILL); \
    if constexpr (R > 2) {                                                                 \
        tile(std::integral_constant<int, (R > 2 ? 2 : 0)>{}, t + 2, REFILL);                 \
        tile(std::integral_constant<int, (R > 2 ? 3 : 0)>{}, t + 3, REFILL);                 \
    }
    int t = 0, group0 = 0;
    for (; t + 2 * R <= T; t += R) {                        // every tile to refill with exists
        EVOSPEC_TURN(true)
        if (t + R - group0 == kNG) { reduce(group0, kNG); group0 += kNG; }
    }
#undef EVOSPEC_TURN
    for (; t < T; t += R) {
#define EVOSPEC_LAST(I)                                                                    \
        if constexpr (R > I) {                                                             \
            if (t + I < T) tile(std::integral_constant<int, (R > I ? I : 0)>{}, t + I, t + I + R < T); \
        }
        EVOSPEC_LAST(0) EVOSPEC_LAST(1) EVOSPEC_LAST(2) EVOSPEC_LAST(3)
#undef EVOSPEC_LAST
        const int done = min(t + R, T);
        if (done - group0 == kNG || done == T) { reduce(group0, done - group0); group0 = done; }
    }

    // ---- one wavefront per draft row: maximum, sum of exponentials, k best
    const int nj = (T * 16 + 63) >> 6;
    for (int m = w; m < M; m += kNW) {
        float z[kNJ];
        float vm = -INFINITY;
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            z[j] = -INFINITY;
            if (j < nj) {                                   // (uniform)
                const int i = j * 64 + lane;
                const float x = Z[(size_t)m * z_stride + (i < n_valid ? i : 0)];
                z[j] = i < n_valid ? x : -INFINITY;         // past the active set: never wins, adds nothing
                vm = fmaxf(vm, z[j]);
            }
        }
        const float lane_max = vm;
        vm = wave_max(vm, lane);
        float se = 0.f;
#pragma unroll
        for (int j = 0; j < kNJ; ++j)
            if (j < nj) se += __expf(z[j] - vm);
        se = wave_sum(se, lane);
        if (lane == 0) part_stats[(size_t)m * n_wg + b] = make_float2(vm, se);
        // the k-th largest of the 64 lane maxima is reached by k logits: what reaches it is ranked by counting
        const uint32_t th = wave_kth_largest(lane < n_valid ? f32_to_ordered(lane_max) : 0u, k);
        u64* lst = list + (size_t)w * z_stride;
        int n = 0;
#pragma unroll
        for (int j = 0; j < kNJ; ++j)
            if (j < nj) {
                const int i = j * 64 + lane;
                const bool in = i < n_valid && z[j] == z[j] && f32_to_ordered(z[j]) >= th;
                const u64 bal = __ballot(in);
                const int p = n + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                if (in) lst[p] = make_key(z[j], Ids[i]);
                n += __popcll(bal);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (this wavefront's own list)
        u64* outk = part_keys + ((size_t)m * n_wg + b) * k;
        for (int e = lane; e < n; e += 64) {
            const u64 mine = lst[e];
            int r = 0;
            for (int f = 0; f < n; f += 4) {                // (z_stride is a multiple of 4: reads past n stay inside the list)
                const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(lst + f), y = *reinterpret_cast<const ulonglong2*>(lst + f + 2);
                r += (x.x > mine ? 1 : 0) + (x.y > mine && f + 1 < n ? 1 : 0) + (y.x > mine && f + 2 < n ? 1 : 0) +
                     (y.y > mine && f + 3 < n ? 1 : 0);
            }
            if (r < k) outk[r] = mine;
        }
        for (int r = n + lane; r < k; r += 64) outk[r] = 0;  // fewer than k rows here
    }
}

namespace {
template <int KU, bool PACKED, bool ONCE>
hipError_t launch_narrow_ku(const NarrowPlan& p, const void* h, int M, int d, const void* W, const int32_t* ids, int V_act,
                            int k, void* keys, void* stats, hipStream_t stream) {
    constexpr int R = KU <= 2 ? 4 : (KU <= 4 ? 2 : 1);                        // about 16 loads in flight per lane
    auto kern = lmhead_narrow_kernel<KU, R, PACKED, ONCE>;
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> attr_set[kMaxDevices] = {};      // concurrent first calls may both set the (idempotent) attribute
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices || !attr_set[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(p.n_slabs), dim3(kNW * 64), p.lds_bytes, stream, static_cast<const uint16_t*>(h), M, d,
                       static_cast<const uint16_t*>(W), ids, V_act, k, p.base_tiles, p.rem_tiles, p.z_stride,
                       static_cast<u64*>(keys), static_cast<float2*>(stats));
    return hipGetLastError();
}
}  // namespace

hipError_t launch_narrow_partials(const NarrowPlan& p, const void* h, int M, int d, const void* W, const int32_t* ids,
                                  int V_act, int k, void* keys, void* stats, hipStream_t stream, bool packed, bool once) {
    if (M < 1 || M > kNarrowRows || d > kNarrowMaxD) return hipErrorInvalidValue;
    switch ((packed_d(d) / 64 + kNW - 1) / kNW) {
#define EVOSPEC_ARGS p, h, M, d, W, ids, V_act, k, keys, stats, stream
#define EVOSPEC_KU(KU_)                                                                                     \
    case KU_:                                                                                               \
        return packed ? (once ? launch_narrow_ku<KU_, true, true>(EVOSPEC_ARGS) : launch_narrow_ku<KU_, true, false>(EVOSPEC_ARGS)) \
                      : (once ? launch_narrow_ku<KU_, false, true>(EVOSPEC_ARGS) : launch_narrow_ku<KU_, false, false>(EVOSPEC_ARGS));
        EVOSPEC_KU(1) EVOSPEC_KU(2) EVOSPEC_KU(3) EVOSPEC_KU(4) EVOSPEC_KU(5) EVOSPEC_KU(6) EVOSPEC_KU(7) EVOSPEC_KU(8)
        default: return hipErrorInvalidValue;
    }
#undef EVOSPEC_KU
#undef EVOSPEC_ARGS
}

}  // namespace evospec

// Medium-M variant of the restricted head (Eq. 1 of the EvoSpec paper on the active set of Eq. 3): a batch
// of a few sequences, where the 256 x 256 tiles of gemm.hip are too few to fill the chip.
//
// One workgroup of four wavefronts computes a 128 x 128 tile of z = W_act h^T (128 active rows x 128 draft
// rows) over the whole hidden dimension; each wavefront takes all 128 active rows for its own 32 draft rows,
// so that it can reduce them to one partial per draft row by itself.  Both operands travel HBM/L2 -> LDS
// with direct-to-LDS loads in pairs of 32-element chunks through a ring of S stages.  Four stages when there
// is one tile per compute unit (a tile this small is through with a stage long before a load comes back),
// two stages and two workgroups per compute unit when there are more tiles than that (300 x 20,000 x 2,048:
// 84 us against 91 with one).  Bound by LDS: per pair of chunks 32 KB go in and 80 KB come out, 875 cycles at
// 128 bytes per cycle against 512 of the matrix cores.  200 rows x 16,384 x 4,096: 43 us, 52 with the merge;
// the 64 tiles of 256 x 256 of this shape took 120 (130).
// Heads of 65 to 128 rows come here as well where use_tiles_early says so.  PARTS: the hidden dimension is summed in kTileParts parts,
// one after the other, whose total waits in registers of its own (use_tiles_early has the errors).  A turn of parts costs 900 cycles
// with one workgroup to a compute unit (20,000 x 4,096 at 80 rows 57.7 -> 60.1 us, 4,096 x 1,024 at 70 22.5 -> 25.0) and is hidden by
// the other one with two (36,864 x 4,096 85.7 -> 86.1).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "plan.hpp"
#include "slab_epilogue.hpp"

namespace evospec {

namespace {

constexpr int kTV = kGemmSlab;                                 // active rows per tile = one slab
constexpr int kTM = kTileRows;                                 // draft rows per tile
constexpr int kTOperand = 128 * 128;                           // bytes of one operand in a pair-stage: 128 rows x 64 elements
constexpr int kTStage = 2 * kTOperand;
constexpr size_t tile_lds(int stages) {
    const size_t ring = (size_t)stages * kTStage, epi = 4ull * epi_bytes(2);
    return (ring > epi ? ring : epi) + kTM * 4;                // and the draft rows' bounds
}
static_assert(kTV == 128 && kTM == 128, "the load and operand offsets below assume it");
static_assert(kTilePartsMinD >= kTileParts * 64, "a pair of chunks to every part");
static_assert(tile_lds(4) <= (size_t)kLdsLimit && 2 * tile_lds(2) <= (size_t)kLdsLimit, "one deep or two shallow rings per compute unit");

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// (the same with the accumulators in ordinary registers)
__device__ __forceinline__ void mfma_vec(f32x4& c, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// Where piece p (16 bytes of a 64-byte chunk row) of a row sits in the row's four slots: see gemm.hip.
__device__ __forceinline__ int swz(int row) { return (((row & 15) >> 1) + ((row & 15) >> 3)) & 3; }

}  // namespace

template <bool PACKED, int S, bool PARTS>
__global__ void __launch_bounds__(256, S > 2 ? 1 : 2)
lmhead_tile_kernel(const uint16_t* __restrict__ h, int M, int d, const uint16_t* __restrict__ W,
                   const int32_t* __restrict__ ids, int V_act, int k, int list_len, int m_tiles,
                   u64* __restrict__ part_keys, float2* __restrict__ part_stats, RowBound bound) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;

    // the m_tiles tiles of the same active rows run on one XCD (see gemm.hip)
    const int nb = gridDim.x, b = blockIdx.x;
    const int xcd = b & 7, full = nb >> 3, rem = nb & 7;
    const int logical = xcd * full + (xcd < rem ? xcd : rem) + (b >> 3);
    const int tile_v = logical / m_tiles, tile_m = logical - tile_v * m_tiles;
    const int v0 = tile_v * kTV, m0 = tile_m * kTM;

    // A wave-level load fills one 1 KB block of a pair-stage: 8 rows x 128 bytes of h or of a row-major W, stored
    // as [chunk parity][row][slot]; or one k-step of 16 rows of a packed W.  Each wavefront: 4 blocks of W, 4 of h.
    const uint16_t* asrc[4];
    const uint16_t* bsrc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int B = 4 * w + i, r = B * 8 + ((lane >> 2) & 7), piece = (lane & 3) ^ swz(r), half = lane >> 5;
        if constexpr (PACKED) {
            const int tile = min((v0 >> 4) + (B >> 1), (V_act - 1) >> 4);          // tiles past the end repeat the last
            asrc[i] = W + (size_t)tile * kPackRows * packed_d(d) + (B & 1) * 512 + lane * 8;
        } else {
            asrc[i] = W + (size_t)min(v0 + r, V_act - 1) * d + half * 32 + piece * 8;   // rows past the end repeat the
        }
        bsrc[i] = h + (size_t)min(m0 + r, M - 1) * d + half * 32 + piece * 8;      // last one, masked later
    }
    const int npairs = d / 64;
    // load j (0..7) of pair p; pairs past the end repeat the last into a stage that nobody reads again
    auto issue = [&](int p, int j) {
        const size_t koff = (size_t)min(p, npairs - 1) * 64;
        unsigned char* dst = smem + (p & (S - 1)) * kTStage + (j & 1) * kTOperand + (4 * w + (j >> 1)) * 1024;
        const uint16_t* src = (j & 1) ? bsrc[j >> 1] + koff : asrc[j >> 1] + (PACKED ? koff * 16 : koff);
        __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)dst, 16, 0, 0);
    };

    // the sum of a part is read out again and again: in ordinary registers, where there are enough of them
    constexpr bool VEC = PARTS && S > 2;
    auto pin = [](f32x4& c) {
        if constexpr (VEC) asm volatile("" : "+v"(c));
        else asm volatile("" : "+a"(c));
    };
    f32x4 acc[8][2];
#pragma unroll
    for (int rg = 0; rg < 8; ++rg)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) acc[rg][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // operand reads: lane (n16, g) takes piece g of row n16 of each 16-row block
    auto row_off = [&](int R) { return (R >> 3) * 1024 + (R & 7) * 64; };
    const int a_rd = PACKED ? lane * 16 : row_off(n16) + ((g ^ swz(n16)) * 16);
    constexpr int kAParity = PACKED ? 1024 : 512;
    const int b_rd = kTOperand + row_off(w * 32 + n16) + ((g ^ swz(n16)) * 16);
    bf16x8 opa[2][8], opb[2][2];
    auto read_a = [&](auto SET, int c, int i) {
        opa[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + ((c >> 1) & (S - 1)) * kTStage + (c & 1) * kAParity + a_rd + i * 2048);
    };
    auto read_b = [&](auto SET, int c, int i) {
        opb[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + ((c >> 1) & (S - 1)) * kTStage + (c & 1) * 512 + b_rd + i * 2048);
    };
    // One chunk: 16 MFMAs on the operands in set CUR, the 10 operand reads of chunk c + 1 into the other set and,
    // in odd chunks, the 8 loads of a pair dealt out between them.  (Instructions issue in order: with the reads
    // first, the matrix cores stood still until LDS had taken the reads of all four wavefronts.)
    auto step = [&](auto CUR, int c, bool load, int p) {
        constexpr int P = decltype(CUR)::value;
        using NXT = std::integral_constant<int, 1 - P>;
#pragma unroll
        for (int rg = 0; rg < 8; ++rg) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                if constexpr (VEC) mfma_vec(acc[rg][mb], opa[P][rg], opb[P][mb]);
                else mfma_acc(acc[rg][mb], opa[P][rg], opb[P][mb]);
            }
            if (rg < 2) read_b(NXT{}, c + 1, rg);
            read_a(NXT{}, c + 1, rg);
            if (load) issue(p, rg);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;

#pragma unroll
    for (int p = 0; p < S; ++p)
#pragma unroll
        for (int j = 0; j < 8; ++j) issue(p, j);
    // the draft rows' bounds, if there are any, while these loads are under way
    float* bnd = reinterpret_cast<float*>(smem + tile_lds(S) - kTM * 4);
    if (bound.n_chunks && tid < kTM) bnd[tid] = row_bound(bound, m0 + tid, M);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(8 * (S - 1)) : "memory");      // pair 0 has landed, for every wavefront
#pragma unroll
    for (int i = 0; i < 2; ++i) read_b(S0{}, 0, i);
#pragma unroll
    for (int i = 0; i < 8; ++i) read_a(S0{}, 0, i);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 7" ::: "memory");
    f32x4 total[8][2];                                           // (PARTS) the sum of the parts so far
    if constexpr (PARTS) {
#pragma unroll
        for (int rg = 0; rg < 8; ++rg)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) total[rg][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int turn = npairs / kTileParts;                              // (PARTS: at least 1)
    for (int p = 0; p < npairs; ++p) {
        if (PARTS && p == turn) {                                // (uniform)
            turn += npairs / kTileParts;
            // (the compiler does not see that these are results of matrix instructions: wait them out, and the zeros in)
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
            for (int rg = 0; rg < 8; ++rg)
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    pin(acc[rg][mb]);
                    total[rg][mb] += acc[rg][mb];
                    acc[rg][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
                    pin(acc[rg][mb]);
                }
            asm volatile("s_nop 7" ::: "memory");
        }
        step(S0{}, 2 * p, false, 0);
        // odd chunk: pair p + 1 must have landed (the S - 2 pairs after it may be under way), and every
        // wavefront must be through with its reads of pair p, whose stage is filled again
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(8 * (S - 2)) : "memory");
        step(S1{}, 2 * p + 1, true, p + S);               // (past the end: stale operands, never used)
    }
    // the last MFMAs drain before the accumulators are read; the ring is dead once the trailing loads have landed and every wavefront is here
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (PARTS) {
#pragma unroll
        for (int rg = 0; rg < 8; ++rg)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                pin(acc[rg][mb]);
                acc[rg][mb] += total[rg][mb];
            }
    }
    slab_epilogue<2>(acc, smem + (size_t)w * epi_bytes(2), v0, m0 + w * 32, M, V_act, ids, k, list_len, tile_v,
                     (V_act + kGemmSlab - 1) / kGemmSlab, bound.n_chunks ? bnd + w * 32 : nullptr, part_keys, part_stats);
}

hipError_t launch_tile_partials(const void* h, int M, int d, const void* W, const int32_t* ids, int V_act, int k, void* keys,
                                void* stats, hipStream_t stream, bool packed, int num_cu, bool parts, const RowBound& bound) {
    if (d % 64 != 0 || d < (parts ? kTilePartsMinD : 64)) return hipErrorInvalidValue;              // callers route such d elsewhere
    const int v_tiles = (V_act + kTV - 1) / kTV, m_tiles = (M + kTM - 1) / kTM;
    // more tiles than compute units: two workgroups with shallow rings share one, so that one computes while
    // the other starts or ends
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool two = v_tiles * m_tiles > num_cu;
    auto kern = packed ? (two ? lmhead_tile_kernel<true, 2, false> : lmhead_tile_kernel<true, 4, false>)
                       : (two ? lmhead_tile_kernel<false, 2, false> : lmhead_tile_kernel<false, 4, false>);
    if (parts)
        kern = packed ? (two ? lmhead_tile_kernel<true, 2, true> : lmhead_tile_kernel<true, 4, true>)
                      : (two ? lmhead_tile_kernel<false, 2, true> : lmhead_tile_kernel<false, 4, true>);
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> attr_set[kMaxDevices] = {};      // concurrent first calls may both set the (idempotent) attribute
    if (dev < 0 || dev >= kMaxDevices || !attr_set[dev].load(std::memory_order_acquire)) {
        for (auto kf : {lmhead_tile_kernel<true, 2, false>, lmhead_tile_kernel<true, 4, false>, lmhead_tile_kernel<false, 2, false>, lmhead_tile_kernel<false, 4, false>,
                        lmhead_tile_kernel<true, 2, true>, lmhead_tile_kernel<true, 4, true>, lmhead_tile_kernel<false, 2, true>, lmhead_tile_kernel<false, 4, true>}) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kf), hipFuncAttributeMaxDynamicSharedMemorySize, (int)tile_lds(4));
            if (e != hipSuccess) return e;
        }
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(v_tiles * m_tiles), dim3(256), tile_lds(two ? 2 : 4), stream, static_cast<const uint16_t*>(h), M, d,
                       static_cast<const uint16_t*>(W), ids, V_act, k, gemm_list_len(k), m_tiles, static_cast<u64*>(keys),
                       static_cast<float2*>(stats), bound);
    return hipGetLastError();
}

}  // namespace evospec

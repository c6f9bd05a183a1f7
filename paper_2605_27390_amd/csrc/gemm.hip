// Large-M variant of the restricted head (Eq. 1 of the EvoSpec paper on the active set of Eq. 3):
// with hundreds of draft rows in flight (batched serving, one shared core for all sequences) the
// projection is a dense contraction and bound by the matrix cores, not by the stream of W_act.
//
// One workgroup of four wavefronts (one per SIMD) computes a 256 x 256 tile of z = W_act h^T
// (256 active rows x 256 draft rows) over the whole hidden dimension.  Both operands travel
// HBM/L2 -> LDS with direct-to-LDS loads (no staging registers, whole 128-byte lines per request)
// in chunks of 32 hidden elements through a ring of four stages, filled two at a time.  Every
// wavefront owns a 128 x 128 quadrant = 8 x 8 accumulators of v_mfma_f32_16x16x32_bf16, which
// fill the 256 accumulation registers of a lane, and reads the operands of the next chunk from
// LDS while the matrix cores work on the current one.  The logits never leave the registers:
// each wavefront reduces its quadrant, per draft row, to a partial for a "slab" of its 128 rows:
// (max, sum-exp) and the logits that can still be among the row's k best, unranked, as
// (logit, id) pairs; the merge kernel ranks them.
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

constexpr int kGK = kGemmKChunk;              // hidden elements per chunk (one MFMA k-step)
constexpr int kGStages = 4;                   // ring of LDS stages
constexpr int kGOperandBytes = kGemmTile * kGK * 2;           // 16 KB: 256 rows x 64 B, no padding
constexpr int kGStageBytes = 2 * kGOperandBytes;              // W_act rows, then h rows
constexpr size_t kGLds = (size_t)kGStages * kGStageBytes;     // 128 KB
constexpr size_t kGLdsTotal = kGLds > 4ull * epi_bytes(8) ? kGLds : 4ull * epi_bytes(8);

constexpr size_t kGLdsAll = kGLdsTotal + kGemmTile * 4;       // and the draft rows' bounds

static_assert(kGLds <= (size_t)kLdsLimit, "operand ring exceeds the LDS of a compute unit");
static_assert(kGLdsAll <= (size_t)kLdsLimit, "epilogue lists exceed the LDS of a compute unit");

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// A row of a chunk holds 32 hidden elements = four 16-byte pieces, rows are stored in blocks of 8
// (see the kernel).  Piece p of row r sits in slot p ^ swz(r), which gives the same piece of 16 consecutive rows 16 different 16-byte
// columns of 256 bytes.  (A 128-bit read takes 16 lanes at a time from two pieces, {0-3, 12-15, 20-27} the first, and meets 12 columns with
// them, four twice.  An order that meets 16 gained nothing here, where the matrix cores are the bound.)  Consecutive rows are 64 bytes
// apart inside a block, blocks 1 KB.  The direct-to-LDS load writes lane L of a wavefront to byte 16 L of a 1 KB block, so
// the swizzle is applied on the source side: the lane that fills (row, slot) fetches piece
// slot ^ swz(row).
__device__ __forceinline__ int swz(int row) { return (((row & 15) >> 1) + ((row & 15) >> 3)) & 3; }

}  // namespace

// PACKED: W is in operand-tile layout (plan.hpp): a wave-level load then takes one whole 1 KB
// operand block (16 rows x 32 hidden elements), which lands in LDS in the order the lanes read it.
template <bool PACKED>
__global__ void __launch_bounds__(256, 1)
lmhead_gemm_kernel(const uint16_t* __restrict__ h, int M, int d,
                   const uint16_t* __restrict__ W, const int32_t* __restrict__ ids, int V_act, int k, int list_len,
                   int m_tiles, u64* __restrict__ part_keys, float2* __restrict__ part_stats, RowBound bound) {
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);       // wave-uniform: keeps LDS destinations scalar
    const int n16 = lane & 15, g = lane >> 4;
    const int wv = w >> 1, wm = w & 1;                             // quadrant: active-row half, draft-row half

    // Workgroups are handed to the 8 XCDs round robin; renumber them so that the m_tiles tiles
    // that read the same 256 rows of W_act run on one XCD (one L2) at about the same time.
    const int nb = gridDim.x, b = blockIdx.x;
    const int xcd = b & 7, full = nb >> 3, rem = nb & 7;
    const int logical = xcd * full + (xcd < rem ? xcd : rem) + (b >> 3);
    const int tile_v = logical / m_tiles, tile_m = logical - tile_v * m_tiles;
    const int v0 = tile_v * kGemmTile, m0 = tile_m * kGemmTile;

    // Direct-to-LDS loads fetch whole 128-byte lines: one wave-level load takes, for 8 rows, the
    // 64 bytes of an even chunk (lanes 0-31) and of the following odd chunk (lanes 32-63).  The
    // ring therefore consists of 2 pair-stages of 64 KB; in a pair-stage, operand o, block b of 8
    // rows: bytes [o * 32 KB + b * 1 KB, +1 KB) = [chunk parity][row][slot].
    constexpr int kPairBytes = 2 * kGStageBytes;                   // 64 KB
    constexpr int kPLoads = kGemmTile / 8 / 4;                     // 8 blocks of 8 rows per wavefront and operand
    const uint16_t* asrc[kPLoads];
    const uint16_t* bsrc[kPLoads];
#pragma unroll
    for (int i = 0; i < kPLoads; ++i) {
        const int r = (kPLoads * w + i) * 8 + ((lane >> 2) & 7);
        const int piece = (lane & 3) ^ swz(r);
        const int half = lane >> 5;
        if constexpr (PACKED) {
            // block B = 8 w + i of the pair-stage: k-step parity B & 1 of the 16-row tile B >> 1
            const int B = kPLoads * w + i;
            const int tile = min((v0 >> 4) + (B >> 1), (V_act - 1) >> 4);            // tiles past the end repeat the last
            asrc[i] = W + (size_t)tile * kPackRows * packed_d(d) + (B & 1) * (16 * kGK) + lane * 8;
        } else {
            asrc[i] = W + (size_t)min(v0 + r, V_act - 1) * d + half * kGK + piece * 8;   // rows past the end repeat
        }
        bsrc[i] = h + (size_t)min(m0 + r, M - 1) * d + half * kGK + piece * 8;       // the last one, masked later
    }
    const int nchunks = d / kGK;                                   // even: d is a multiple of 64 here
    const int npairs = nchunks / 2;
    // Load number j (0..15) of pair p: block j/2 of this wavefront's W_act rows (j even) or h rows (j odd).
    // Pairs past the end repeat the last one into a stage nobody reads again.
    auto issue_one = [&](int p, int j) {
        const size_t koff = (size_t)min(p, npairs - 1) * (2 * kGK);
        unsigned char* dst = smem + (p & 1) * kPairBytes + (j & 1) * (2 * kGOperandBytes) + (kPLoads * w + (j >> 1)) * 1024;
        // (a k-step of a packed tile is 16 rows x 32 elements long)
        const uint16_t* src = (j & 1) ? bsrc[j >> 1] + koff : asrc[j >> 1] + (PACKED ? koff * 16 : koff);
        __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)dst, 16, 0, 0);
    };

    f32x4 acc[8][8];
#pragma unroll
    for (int rg = 0; rg < 8; ++rg)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) acc[rg][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // operand reads: lane (n16, g) takes piece g of row n16 of each 16-row block of its quadrant;
    // row R of an operand sits in block R / 8 at row R % 8
    auto row_off = [&](int R) { return (R >> 3) * 1024 + (R & 7) * 64; };
    const int a_rd = PACKED ? wv * 128 * 128 + lane * 16 : row_off(wv * 128 + n16) + ((g ^ swz(n16)) * 16);
    constexpr int kAParity = PACKED ? 1024 : 512;                  // second chunk of a pair, W side
    const int b_rd = 2 * kGOperandBytes + row_off(wm * 128 + n16) + ((g ^ swz(n16)) * 16);
    bf16x8 opa[2][8], opb[2][8];
    auto stage_of = [&](int c) { return ((c >> 1) & 1) * kPairBytes + (c & 1) * 512; };
    auto read_a = [&](auto SET, int c, int i) {
        opa[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + ((c >> 1) & 1) * kPairBytes + (c & 1) * kAParity + a_rd + i * 2048);
    };
    auto read_b = [&](auto SET, int c, int i) {
        opb[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + stage_of(c) + b_rd + i * 2048);
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;

    // One chunk: 64 MFMAs on the operands in registers (set CUR); in the gaps, the 16 operand
    // reads of chunk c+1 (into set 1 - CUR) and, in odd chunks, the 16 loads of the pair (c+3, c+4)
    // into the pair-stage of chunks (c-1, c), which every wavefront finished reading before the
    // barrier.  An odd chunk needs the pair (c+1, c+2), requested two chunks ago and the youngest
    // request: wait for everything.  An even chunk needs its own pair, which its predecessor needed too.
    auto step = [&](auto CUR, int c) {
        constexpr int P = decltype(CUR)::value;
        using NXT = std::integral_constant<int, 1 - P>;
        if (P == 1) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int rg = 0; rg < 8; ++rg) {
#pragma unroll
            for (int mb = 0; mb < 8; ++mb) mfma_acc(acc[rg][mb], opa[P][rg], opb[P][mb]);
#pragma unroll
            for (int q = 3 * rg; q < 3 * rg + 3 && q < 16; ++q) {
                // (a stage past the last chunk holds stale data that is never used)
                if (q & 1) read_a(NXT{}, c + 1, q >> 1);
                else read_b(NXT{}, c + 1, q >> 1);
            }
            if (P == 1) { issue_one((c + 3) >> 1, 2 * rg); issue_one((c + 3) >> 1, 2 * rg + 1); }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };

#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int j = 0; j < 16; ++j) issue_one(p, j);
    // the draft rows' bounds, if there are any, while these loads are under way
    float* bnd = reinterpret_cast<float*>(smem + kGLdsTotal);
    if (bound.n_chunks) bnd[tid] = row_bound(bound, m0 + tid, M);
    // pair 0 must have landed before its operands are read
    asm volatile("s_waitcnt vmcnt(16)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i) { read_b(S0{}, 0, i); read_a(S0{}, 0, i); }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 7" ::: "memory");

    for (int c = 0; c < nchunks; c += 2) {
        step(S0{}, c);
        step(S1{}, c + 1);
    }
    // the last MFMAs drain before the accumulators are read; the ring is dead once the trailing
    // loads have landed and every wavefront is here
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- epilogue: wave-local from here on; the operand buffers are dead (all waves are past the
    // last barrier), each wavefront takes its own piece of them
    const int vrow0 = v0 + wv * kGemmSlab;
    if (vrow0 >= V_act) return;                                    // quadrant wholly past the active set
    slab_epilogue<8>(acc, smem + (size_t)w * epi_bytes(8), vrow0, m0 + wm * 128, M, V_act, ids, k, list_len,
                     tile_v * (kGemmTile / kGemmSlab) + wv, (V_act + kGemmSlab - 1) / kGemmSlab,
                     bound.n_chunks ? bnd + wm * 128 : nullptr, part_keys, part_stats);
}

hipError_t launch_gemm_partials(const void* h, int M, int d, const void* W, const int32_t* ids, int V_act,
                                int k, void* keys, void* stats, hipStream_t stream, bool packed, const RowBound& bound) {
    const int v_tiles = (V_act + kGemmTile - 1) / kGemmTile;
    const int m_tiles = (M + kGemmTile - 1) / kGemmTile;
    if (d % (2 * kGK) != 0 || d < 2 * kGK) return hipErrorInvalidValue;      // callers route such d elsewhere
    auto kern = packed ? lmhead_gemm_kernel<true> : lmhead_gemm_kernel<false>;
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> attr_set[kMaxDevices] = {};      // concurrent first calls may both set the (idempotent) attribute
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices || !attr_set[dev].load(std::memory_order_acquire)) {
        for (auto kf : {lmhead_gemm_kernel<true>, lmhead_gemm_kernel<false>}) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kf),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGLdsAll);
            if (e != hipSuccess) return e;
        }
        if (dev >= 0 && dev < kMaxDevices) attr_set[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(v_tiles * m_tiles), dim3(256), kGLdsAll, stream,
                       static_cast<const uint16_t*>(h), M, d, static_cast<const uint16_t*>(W), ids, V_act, k, gemm_list_len(k),
                       m_tiles, static_cast<u64*>(keys), static_cast<float2*>(stats), bound);
    return hipGetLastError();
}

}  // namespace evospec

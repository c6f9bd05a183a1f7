// Medium-M variant of the restricted head (Eq. 1 of the EvoSpec paper on the active set of Eq. 3): a batch
// of a few sequences, where the 256 x 256 tiles of gemm.hip are too few to fill the chip.
//
// One workgroup of four wavefronts computes a 128 x 128 tile of z = W_act h^T (128 active rows x 128 draft
// rows) over the whole hidden dimension; each wavefront reduces all 128 active rows for its own 32 draft rows to one partial per
// draft row.  lmhead_tile_kernel: both operands travel HBM/L2 -> LDS
// with direct-to-LDS loads in pairs of 32-element chunks through a ring of S stages: four stages when there
// is one workgroup per compute unit (a tile this small is through with a stage long before a load comes back),
// two stages and two workgroups per compute unit otherwise.  lmhead_packed_tile_kernel, for packed matrices with two workgroups per compute
// unit where w_in_registers says so: only h goes through LDS, W straight into registers (30,000 x 2,048 at 256 rows 63 -> 60 us; with one workgroup per compute unit
// 14,848 x 4,096 at 200 51 -> 54).
// Bound by what a compute unit is sent: 32 KB per pair of chunks, 0.3 us with few of them at work and 0.6 with all (54 GB/s each).
// Neither LDS, free of bank conflicts or not, nor a ring twice as deep, nor draft rows of zeros make a difference;
// W from two pairs that stay in the caches does (14,848 x 4,096 at 200 rows 53 -> 40 us).
//
// The extensions of a batched head are slabs of 64 rows (slab.hpp) in the same launch where joint_tiles says so: by themselves they are a
// chain of 11 us and 0.4 us per chunk (row-major 1.0) on a few workgroups.
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
#include "slab.hpp"
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

constexpr size_t kPackedTileLds = 4ull * epi_bytes(2) > (size_t)kPRing * kTOperand ? 4ull * epi_bytes(2) : (size_t)kPRing * kTOperand;
static_assert(kPackedTileLds >= 64 * 1024 && 2 * kPackedTileLds <= (size_t)kLdsLimit, "the logits of a tile; two workgroups per compute unit");
// operand of s_waitcnt: so many loads, and LDS (or scalar) accesses, may be under way
constexpr int wait_imm(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | (vm >> 4 << 14); }

constexpr int kRsrcFlags = 0x00020000;                         // raw buffer of 32-bit offsets
// Bytes of the rows of a tile (below 4 GB: the offsets are 32 bits).
__device__ __forceinline__ int tile_bytes(int rows, int d) { return (int)((unsigned)rows * (unsigned)d * 2u); }

// (the same with the accumulators in ordinary registers)
__device__ __forceinline__ void mfma_vec(f32x4& c, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

}  // namespace

// What the tiles of the batched head bring along: the extensions' slabs, as further workgroups of the launch.
struct TileExtensions {
    const uint16_t* W = nullptr;
    const int32_t* ids = nullptr;
    int seq_rows = 0;                    // rows of an extension
    int n_slabs = 0;                     // slabs of an extension
    int gl = 0;                          // selection group level (Plan::gl)
    size_t chunk_keys = 0;               // u64 (and float2) between two chunks' partials
    u64* keys = nullptr;
    float2* stats = nullptr;
};

// What a launch brings beside the tiles' own arguments, and nothing that it does not: 1.7 KB of them cost a launch some 0.3 us.
struct ExtensionArgs {
    ChunkBatch cb;
    TileExtensions ext;
};
template <int XMB>
using BesideArgs = std::conditional_t<(XMB > 0), ExtensionArgs, std::conditional_t<(XMB < 0), RowBound, int>>;

// XMB: 16-row blocks of an extension's draft rows (0: no extensions in this launch, -1: but a bound from their lists); XFULL: d is a multiple of kKC.
template <bool PACKED, int S, bool PARTS, int XMB, bool XFULL>
__global__ void __launch_bounds__(256, S > 2 ? 1 : 2)
lmhead_tile_kernel(const uint16_t* __restrict__ h, int M, int d, const uint16_t* __restrict__ W,
                   const int32_t* __restrict__ ids, int V_act, int k, int list_len, int m_tiles, int n_tiles,
                   u64* __restrict__ part_keys, float2* __restrict__ part_stats, BesideArgs<XMB> beside) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;

    if constexpr (XMB > 0) {
        if ((int)blockIdx.x >= n_tiles) {
            const ChunkBatch& cb = beside.cb;
            const TileExtensions& ext = beside.ext;
            int slab = (int)blockIdx.x - n_tiles;
            const int ci = slab / ext.n_slabs;
            slab -= ci * ext.n_slabs;
            const size_t seq_row0 = (size_t)cb.seq[ci] * ext.seq_rows;
            SlabProblem pr;
            pr.rows = cb.rows[ci];
            pr.h = h + (size_t)cb.m0[ci] * d;
            pr.W = ext.W + seq_row0 * d;
            pr.ids = ext.ids + seq_row0;
            pr.V_act = ext.seq_rows;
            pr.keys = ext.keys + (size_t)ci * ext.chunk_keys;
            pr.stats = ext.stats + (size_t)ci * ext.chunk_keys;
            slab_partials<4, 1, 2, XMB, XFULL, false, false, 1>(pr, slab, d, k, ext.gl, smem);
            return;
        }
    }

    // the m_tiles tiles of the same active rows run on one XCD (see gemm.hip)
    const int nb = n_tiles, b = blockIdx.x;
    const int xcd = b & 7, full = nb >> 3, rem = nb & 7;
    const int logical = xcd * full + (xcd < rem ? xcd : rem) + (b >> 3);
    const int tile_v = logical / m_tiles, tile_m = logical - tile_v * m_tiles;
    const int v0 = tile_v * kTV, m0 = tile_m * kTM;

    // A wave-level load fills one 1 KB block of a pair-stage: 8 rows x 128 bytes of h or of a row-major W, piece p of row r in
    // place p ^ (r / 2 mod 8) of its eight; or one k-step of 16 rows of a packed W.  Each wavefront: 4 blocks of W, 4 of h.
    // (A 128-bit read takes its 16 rows' pieces in four turns of 16 lanes, {0-3, 12-15, 20-27} the first: each turn meets 16 different
    // 16-byte columns of 256 bytes, so no bank twice.  Global loads: buffer loads cost row-major tiles of five rounds 5 to 7 % (512 rows, 40,000 x 2,560 169.3 us, so 181.8;
    // x 1,536 112.1 and 117.0), one round up to 1.5 % (5,000 x 2,048 at 400 28.9 and 29.3).)
    const char* wbase = reinterpret_cast<const char*>(W + (size_t)v0 * (PACKED ? packed_d(d) : d));
    const char* hbase = reinterpret_cast<const char*>(h + (size_t)m0 * d);
    unsigned aoff[4], boff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int B = 4 * w + i, r = B * 8 + (lane >> 3), piece = (lane & 7) ^ ((r & 15) >> 1);
        if constexpr (PACKED) {
            const int tile = min(B >> 1, (V_act - 1 - v0) >> 4);                   // tiles past the end repeat the last
            aoff[i] = (unsigned)tile * kPackRows * packed_d(d) * 2u + (B & 1) * 1024 + lane * 16;
        } else {
            aoff[i] = ((unsigned)min(r, V_act - 1 - v0) * d + piece * 8) * 2u;      // rows past the end repeat the
        }
        boff[i] = ((unsigned)min(r, M - 1 - m0) * d + piece * 8) * 2u;             // last one, masked later
    }
    const int npairs = d / 64;
    // load j (0..7) of pair p; pairs past the end repeat the last into a stage that nobody reads again
    auto issue = [&](int p, int j) {
        const size_t at = (size_t)min(p, npairs - 1) * 128;
        const auto dst = (lptr_t)(smem + (p & (S - 1)) * kTStage + (j & 1) * kTOperand + (4 * w + (j >> 1)) * 1024);
        const char* src = j & 1 ? hbase + boff[j >> 1] + at : wbase + aoff[j >> 1] + (PACKED ? at * 16 : at);
        __builtin_amdgcn_global_load_lds((gptr_t)src, dst, 16, 0, 0);
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
    const int rd = n16 * 128 + ((g ^ (n16 >> 1)) * 16);           // (even k-step of a pair; the odd one: 64 bytes away)
    const int a_rd[2] = {PACKED ? lane * 16 : rd, PACKED ? lane * 16 + 1024 : rd ^ 64};
    const int b_rd[2] = {kTOperand + w * 4096 + rd, kTOperand + w * 4096 + (rd ^ 64)};
    bf16x8 opa[2][8], opb[2][2];
    auto read_a = [&](auto SET, int c, int i) {                  // (c: a chunk of the set's parity)
        opa[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + ((c >> 1) & (S - 1)) * kTStage + a_rd[decltype(SET)::value] + i * 2048);
    };
    auto read_b = [&](auto SET, int c, int i) {
        opb[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + ((c >> 1) & (S - 1)) * kTStage + b_rd[decltype(SET)::value] + i * 2048);
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
    if constexpr (XMB < 0) {
        if (tid < kTM) bnd[tid] = row_bound(beside, m0 + tid, M);
    }
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
    slab_epilogue<2, true, XMB < 0>(acc, smem + (size_t)w * epi_bytes(2), v0, m0 + w * 32, M, V_act, ids, k, list_len, tile_v,
                     (V_act + kGemmSlab - 1) / kGemmSlab, XMB < 0 ? bnd + w * 32 : nullptr, part_keys, part_stats);
}

// The same for a packed W: a wavefront has the operand blocks of its own 32 active rows in registers, kPRing pairs ahead, and contracts them with all
// 128 draft rows, whose stages of 16 KB leave room for two workgroups on a compute unit with as long a lead.  At the end the logits change
// hands through LDS.
template <int XMB, bool XFULL>
__global__ void __launch_bounds__(256, 2)
lmhead_packed_tile_kernel(const uint16_t* __restrict__ h, int M, int d, const uint16_t* W,
                   const int32_t* __restrict__ ids, int V_act, int k, int list_len, int m_tiles, int n_tiles,
                   u64* __restrict__ part_keys, float2* __restrict__ part_stats, BesideArgs<XMB> beside) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int S = kPRing;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;

    if constexpr (XMB > 0) {
        if ((int)blockIdx.x >= n_tiles) {
            const ChunkBatch& cb = beside.cb;
            const TileExtensions& ext = beside.ext;
            int slab = (int)blockIdx.x - n_tiles;
            const int ci = slab / ext.n_slabs;
            slab -= ci * ext.n_slabs;
            const size_t seq_row0 = (size_t)cb.seq[ci] * ext.seq_rows;
            SlabProblem pr;
            pr.rows = cb.rows[ci];
            pr.h = h + (size_t)cb.m0[ci] * d;
            pr.W = ext.W + (size_t)cb.seq[ci] * packed_rows(ext.seq_rows) * packed_d(d);
            pr.ids = ext.ids + seq_row0;
            pr.V_act = ext.seq_rows;
            pr.keys = ext.keys + (size_t)ci * ext.chunk_keys;
            pr.stats = ext.stats + (size_t)ci * ext.chunk_keys;
            slab_partials<4, 1, 2, XMB, XFULL, true, false, 1>(pr, slab, d, k, ext.gl, smem);
            return;
        }
    }

    // the m_tiles tiles of the same active rows run on one XCD (see gemm.hip)
    const int nb = n_tiles, b = blockIdx.x;
    const int xcd = b & 7, full = nb >> 3, rem = nb & 7;
    const int logical = xcd * full + (xcd < rem ? xcd : rem) + (b >> 3);
    const int tile_v = logical / m_tiles, tile_m = logical - tile_v * m_tiles;
    const int v0 = tile_v * kTV, m0 = tile_m * kTM;

    // W: this wavefront's 32 rows, two operand blocks of 1 KB to a k-step, straight into registers through a ring of kPRing pairs (the loads
    // under way at each barrier: plan.hpp)
    const uint16_t* wsrc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)                                  // (tiles past the end repeat the last)
        wsrc[t] = W + (size_t)min((v0 >> 4) + 2 * w + t, (V_act - 1) >> 4) * kPackRows * packed_d(d) + lane * 8;
    // h: a wave-level load fills one 1 KB block of a pair-stage: 8 rows x 128 bytes, as in the kernel above
    const auto hrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(h + (size_t)m0 * d), 0, tile_bytes(min(M - m0, kTM), d), kRsrcFlags);
    unsigned hoff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = (4 * w + i) * 8 + (lane >> 3), piece = (lane & 7) ^ ((r & 15) >> 1);
        hoff[i] = ((unsigned)min(r, M - 1 - m0) * d + piece * 8) * 2u;               // rows past the end repeat the last one, masked later
    }
    const int npairs = d / 64;
    // (pairs past the end repeat the last, into a stage or registers that nobody reads again)
    auto issue_h = [&](int p, int i) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(hrsrc, (lptr_t)(smem + (p & (S - 1)) * kTOperand + (4 * w + i) * 1024), 16, (int)hoff[i],
                                                 min(p, npairs - 1) * 128, 0, 0);
    };
    u32x4 wr[2 * S][2];                                     // [k-step of the ring][tile]
    auto load_w = [&](auto SLOT, int p, int s) {                 // k-step s of pair p
#pragma unroll
        for (int t = 0; t < 2; ++t) wr[decltype(SLOT)::value][t] = *(gvec_ptr)(wsrc[t] + (size_t)min(p, npairs - 1) * 1024 + s * 512);
    };
    f32x4 acc[2][8];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) acc[t][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int b_rd = n16 * 128 + ((g ^ (n16 >> 1)) * 16), b_rd1 = b_rd ^ 64;       // even and odd k-step of a pair
    bf16x8 opb[2][8];
    auto read_b = [&](auto SET, int p, int s, int i) {
        opb[decltype(SET)::value][i] = *reinterpret_cast<const bf16x8*>(smem + (p & (S - 1)) * kTOperand + (s ? b_rd1 : b_rd) + i * 2048);
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // One k-step: 16 MFMAs on ring slot SLOT and operand set S, the operand reads of the next k-step between them; with LOAD, the pair p + S is
    // requested.
    auto step = [&](auto SLOT, auto PAR, int p, auto LOAD) {
        constexpr int s = decltype(PAR)::value, slot = decltype(SLOT)::value;
        constexpr bool load = decltype(LOAD)::value;
        using NXT = std::integral_constant<int, 1 - s>;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[slot][t]), opb[s][i], acc[t][i], 0, 0, 0);
            read_b(NXT{}, s ? p + 1 : p, 1 - s, i);              // (past the end: stale operands, never used)
            if (load && s == 1 && i < 4) issue_h(p + S, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (load) load_w(SLOT, p + S, s);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto pair = [&](auto R, int p) {
        constexpr int r = decltype(R)::value;
        step(std::integral_constant<int, 2 * r>{}, S0{}, p, std::true_type{});
        // pair p + 1 of h must have landed for every wavefront, and every wavefront must be through with its reads of pair p, whose
        // stage is filled again
        __builtin_amdgcn_s_waitcnt(wait_imm(ring_wait(S), 0));
        asm volatile("s_barrier" ::: "memory");
        step(std::integral_constant<int, 2 * r + 1>{}, S1{}, p, std::true_type{});
    };
    // (a pair whose successors have landed, all of them)
    auto last_pair = [&](auto R, int p) {
        constexpr int r = decltype(R)::value;
        step(std::integral_constant<int, 2 * r>{}, S0{}, p, std::false_type{});
        step(std::integral_constant<int, 2 * r + 1>{}, S1{}, p, std::false_type{});
    };

    auto prologue = [&](auto R) {
        constexpr int r = decltype(R)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) issue_h(r, i);
        __builtin_amdgcn_sched_barrier(0);
        load_w(std::integral_constant<int, 2 * r>{}, r, 0);
        load_w(std::integral_constant<int, 2 * r + 1>{}, r, 1);
        __builtin_amdgcn_sched_barrier(0);
    };
#define EVOSPEC_RING(X) X(0) X(1) X(2) X(3)
#define EVOSPEC_X(I) prologue(std::integral_constant<int, I>{});
    EVOSPEC_RING(EVOSPEC_X)
#undef EVOSPEC_X
    // pair 0 has landed, for every wavefront.  (Fewer pairs than stages: nothing reads the last ones' W, whose loads need not be there to be counted.)
    if (npairs >= S) __builtin_amdgcn_s_waitcnt(wait_imm(ring_first_wait(S), 15));
    else __builtin_amdgcn_s_waitcnt(wait_imm(0, 15));
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i) read_b(S0{}, 0, 0, i);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 7" ::: "memory");
    int p = 0;
    for (; p + S <= npairs; p += S) {
#define EVOSPEC_X(I) pair(std::integral_constant<int, I>{}, p + I);
        EVOSPEC_RING(EVOSPEC_X)
#undef EVOSPEC_X
    }
    // The last pairs, fewer than the ring has: all of them are on their way, nothing more is requested, and they are waited for together.  (Every
    // register of the ring is read here, so that the loads that the waits above count are there in the last turn of the loop too.)
#pragma unroll
    for (int i = 0; i < 2 * S; ++i) asm volatile("" : "+v"(wr[i][0]), "+v"(wr[i][1]));
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#define EVOSPEC_X(I) if constexpr (I + 1 < S) { if (p + I < npairs) last_pair(std::integral_constant<int, I>{}, p + I); }
    EVOSPEC_RING(EVOSPEC_X)
#undef EVOSPEC_X
#undef EVOSPEC_RING
    // the ring is dead once every wavefront is here
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // The logits change hands through LDS: from here on a wavefront has all 128 active rows for 32 draft rows.  (Blocks of 16 x 16, which keep
    // their lanes.)
    unsigned char* z = smem + lane * 16;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) *reinterpret_cast<f32x4*>(z + ((2 * w + t) * 8 + mb) * 1024) = acc[t][mb];
    __syncthreads();
    f32x4 mine[8][2];
#pragma unroll
    for (int rg = 0; rg < 8; ++rg)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) mine[rg][mb] = *reinterpret_cast<const f32x4*>(z + (rg * 8 + 2 * w + mb) * 1024);
    __syncthreads();
    slab_epilogue<2, false, false>(mine, smem + (size_t)w * epi_bytes(2), v0, m0 + w * 32, M, V_act, ids, k, list_len, tile_v,
                     (V_act + kGemmSlab - 1) / kGemmSlab, nullptr, part_keys, part_stats);
}

namespace {
// Lets a kernel have all the LDS of a compute unit, once per device (concurrent first calls may both set the idempotent attribute).
template <auto KERN>
hipError_t allow_lds() {
    static std::atomic<uint64_t> set{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (bit && (set.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERN), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLimit);
    if (e == hipSuccess) set.fetch_or(bit, std::memory_order_release);
    return e;
}
}  // namespace

hipError_t launch_tile_partials(const void* h, int M, int d, const void* W, const int32_t* ids, int V_act, int k, void* keys,
                                void* stats, hipStream_t stream, bool packed, int num_cu, bool parts, const RowBound& bound, const TileBatch* tb) {
    if (d % 64 != 0 || d < (parts ? kTilePartsMinD : 64) || d > kTileMaxD) return hipErrorInvalidValue;              // callers route such d elsewhere
    const int v_tiles = (V_act + kTV - 1) / kTV, m_tiles = (M + kTM - 1) / kTM, n_tiles = v_tiles * m_tiles;
    ExtensionArgs x;
    ChunkBatch& cb = x.cb;
    TileExtensions& ext = x.ext;
    int blocks = n_tiles, xmb = 0;
    size_t xlds = 0;
    if (tb) {
        const Plan& p = *tb->plan;
        if (parts || p.nw != 4 || p.ks != 1 || p.segs != 1 || tb->cb->n < 1 || tb->cb->n > kMaxChunks || tb->chunk_bytes % 8 != 0) return hipErrorInvalidValue;
        cb = *tb->cb;
        ext.W = static_cast<const uint16_t*>(tb->W); ext.ids = tb->ids; ext.seq_rows = tb->seq_rows;
        ext.n_slabs = p.n_slabs; ext.gl = p.gl; ext.chunk_keys = tb->chunk_bytes / 8;
        ext.keys = static_cast<u64*>(tb->keys); ext.stats = static_cast<float2*>(tb->stats);
        xlds = p.lds_bytes; xmb = p.mb;
        blocks += p.n_slabs * cb.n;
    }
    // more workgroups than compute units: two with shallow rings share one, so that one computes while the other starts or ends
    const bool two = blocks > num_cu;
    const bool bounded = bound.n_chunks > 0, own = packed && !parts && (tb || (two && w_in_registers(M, V_act, d, num_cu)));
    const size_t need = own ? kPackedTileLds : tile_lds(two ? 2 : 4), lds = need > xlds ? need : xlds;
    hipError_t e = hipSuccess;
    auto go = [&](hipError_t allowed, auto kern, const auto& beside) {
        e = allowed;
        if (e != hipSuccess) return;
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), lds, stream, static_cast<const uint16_t*>(h), M, d, static_cast<const uint16_t*>(W), ids,
                           V_act, k, gemm_list_len(k), m_tiles, n_tiles, static_cast<u64*>(keys), static_cast<float2*>(stats), beside);
        e = hipGetLastError();
    };
    auto args_of = [&](auto XMB) -> const auto& {
        if constexpr (decltype(XMB)::value > 0) return x;
        else if constexpr (decltype(XMB)::value < 0) return bound;
        else return blocks;                                        // (nothing)
    };
#define EVOSPEC_GO(X, ...) go(allow_lds<__VA_ARGS__>(), __VA_ARGS__, args_of(std::integral_constant<int, X>{}))
    auto go_packed = [&](auto XMB) {
        if (d % kKC == 0) EVOSPEC_GO(decltype(XMB)::value, lmhead_packed_tile_kernel<decltype(XMB)::value, true>);
        else EVOSPEC_GO(decltype(XMB)::value, lmhead_packed_tile_kernel<decltype(XMB)::value, false>);
    };
    auto go_rows = [&](auto ST, auto XMB) {
        if (d % kKC == 0) EVOSPEC_GO(decltype(XMB)::value, lmhead_tile_kernel<false, decltype(ST)::value, false, decltype(XMB)::value, true>);
        else EVOSPEC_GO(decltype(XMB)::value, lmhead_tile_kernel<false, decltype(ST)::value, false, decltype(XMB)::value, false>);
    };
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    using C4 = std::integral_constant<int, 4>;
    if (parts && packed) two ? EVOSPEC_GO(0, lmhead_tile_kernel<true, 2, true, 0, true>) : EVOSPEC_GO(0, lmhead_tile_kernel<true, 4, true, 0, true>);
    else if (parts) two ? EVOSPEC_GO(0, lmhead_tile_kernel<false, 2, true, 0, true>) : EVOSPEC_GO(0, lmhead_tile_kernel<false, 4, true, 0, true>);
    else if (bounded && !packed) two ? EVOSPEC_GO(-1, lmhead_tile_kernel<false, 2, false, -1, true>) : EVOSPEC_GO(-1, lmhead_tile_kernel<false, 4, false, -1, true>);
    else if (packed && !own && two && bounded) EVOSPEC_GO(-1, lmhead_tile_kernel<true, 2, false, -1, true>);
    else if (packed && !own) two ? EVOSPEC_GO(0, lmhead_tile_kernel<true, 2, false, 0, true>) : EVOSPEC_GO(0, lmhead_tile_kernel<true, 4, false, 0, true>);
    else if (packed) xmb == 0 ? EVOSPEC_GO(0, lmhead_packed_tile_kernel<0, true>) : xmb == 1 ? go_packed(C1{}) : xmb == 2 ? go_packed(C2{}) : go_packed(C4{});
    else if (xmb == 0) two ? EVOSPEC_GO(0, lmhead_tile_kernel<false, 2, false, 0, true>) : EVOSPEC_GO(0, lmhead_tile_kernel<false, 4, false, 0, true>);
    else if (two) xmb == 1 ? go_rows(C2{}, C1{}) : xmb == 2 ? go_rows(C2{}, C2{}) : go_rows(C2{}, C4{});
    else xmb == 1 ? go_rows(C4{}, C1{}) : xmb == 2 ? go_rows(C4{}, C2{}) : go_rows(C4{}, C4{});
#undef EVOSPEC_GO
    return e;
}

}  // namespace evospec

// Types and device helpers shared by the HIP kernels of the active-vocabulary LM head.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace evospec {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const u32x4 __attribute__((address_space(1))) * gvec_ptr;   // 16-byte loads from HBM

// A 16-byte load of data that this launch reads once: marked non-temporal, so that a stream larger than
// the caches does not drag its lines through them.  (Measured on MI355X with the streaming kernels of this
// library: 6.7 against 6.0 TB/s on 1.2 GB, 5.9 against 5.4 on 302 MB.)
__device__ __forceinline__ u32x4 load_once(gvec_ptr p) { return __builtin_nontemporal_load(p); }

// ---------------------------------------------------------------------------------------
// (logit, id) -> one 64-bit key whose unsigned order is "larger logit first, then smaller
// full-vocabulary id".  Key 0 is reserved for "no candidate".
__device__ __forceinline__ uint32_t f32_to_ordered(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);       // -0 -> +0 so that the two tie
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);   // negative: flip all bits, else the sign
}
__device__ __forceinline__ float ordered_to_f32(uint32_t o) {
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}
__device__ __forceinline__ u64 make_key(float z, int32_t id) {
    return ((u64)f32_to_ordered(z) << 32) | (uint32_t)(~(uint32_t)id);
}
__device__ __forceinline__ float key_value(u64 key) { return ordered_to_f32((uint32_t)(key >> 32)); }
__device__ __forceinline__ int32_t key_id(u64 key) { return (int32_t)(~(uint32_t)key); }

// Workgroup barrier that waits for this wave's LDS traffic only: global loads issued for
// the next chunk stay in flight across it (a plain __syncthreads() would drain them).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One set of per-slab partial results as the merge kernel reads it: the list of (slab L, row
// slot r) starts at keys + L * key_slab + r * key_row, its statistics are stats[L * stat_slab + r * stat_row].
struct PartialSet {
    const u64* keys;
    const float2* stats;
    int n_slabs;
    int row_base;           // slot of this launch's block 0 inside the set's row dimension
    size_t key_slab, key_row;       // strides in u64
    size_t stat_slab, stat_row;     // strides in float2
    int list_len;           // key slots per list (>= k); empty slots hold 0
    int sorted;             // lists hold keys, descending (slot 0 is the maximum); else (logit, id)
                            // pairs in any order, all ones = empty
};

// x of lane (lane ^ STRIDE), STRIDE a power of two below 64, without a trip through LDS (a
// ds_bpermute costs its full latency at every step of a dependent chain: 42 of them made a 64-lane sort
// 3,500 cycles long).  Strides 1 and 2 are quad permutes; 4 is a mirror of each group of 8
// lanes (lane ^ 7) followed by a reversal within quads (lane ^ 3); 8 is a rotation by 8 within the
// 16-lane row; 16 and 32 are the row / half swaps of gfx950: v_permlane16_swap(x, x) returns the even
// rows' values in all rows and the odd rows' values in all rows, v_permlane32_swap(x, x) the lower and
// the upper half.
template <int STRIDE>
__device__ __forceinline__ uint32_t xor_lane(uint32_t x, int lane) {
    static_assert(STRIDE == 1 || STRIDE == 2 || STRIDE == 4 || STRIDE == 8 || STRIDE == 16 || STRIDE == 32, "stride");
    if constexpr (STRIDE == 1) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0xB1, 0xF, 0xF, false);      // quad_perm [1,0,3,2]
    } else if constexpr (STRIDE == 2) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x4E, 0xF, 0xF, false);      // quad_perm [2,3,0,1]
    } else if constexpr (STRIDE == 4) {
        const int m = __builtin_amdgcn_update_dpp((int)x, (int)x, 0x141, 0xF, 0xF, false);        // row_half_mirror
        return (uint32_t)__builtin_amdgcn_update_dpp(m, m, 0x1B, 0xF, 0xF, false);                // quad_perm [3,2,1,0]
    } else if constexpr (STRIDE == 8) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, 0x128, 0xF, 0xF, false);     // row_ror:8
    } else if constexpr (STRIDE == 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane & 16) ? a[0] : a[1];
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (lane & 32) ? a[0] : a[1];
    }
}
// For narrow.hip: two MFMA operands (k-steps 2p and 2p + 1 of 16 row-major rows) from whole 128-byte lines: lane (n, g)
// loads piece g (n < 8) or g + 4 of line p of row n % 8 into `a`, and piece g + 4 (n < 8) or g of row
// 8 + n % 8 into `b`.  The first operand is then the lane's own a or b, the second that of lane l ^ 8.
// lanes l with (l & 8) set take `b`, the others `a`
__device__ __forceinline__ uint32_t pick_bank(uint32_t a, uint32_t b) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, 0xE4, 0xF, 0xC, false);       // quad_perm [0,1,2,3], banks 2 and 3
}
// the value of lane l ^ 8: from `a` for lanes without bit 3, from `b` for the others
__device__ __forceinline__ uint32_t pick_bank_ror8(uint32_t a, uint32_t b) {
    const int t = __builtin_amdgcn_update_dpp((int)a, (int)a, 0x128, 0xF, 0x3, false);         // row_ror:8 into banks 0 and 1
    return (uint32_t)__builtin_amdgcn_update_dpp(t, (int)b, 0x128, 0xF, 0xC, false);           // and into banks 2 and 3
}
__device__ __forceinline__ float wave_max(float x, int lane) {
    x = fmaxf(x, __uint_as_float(xor_lane<1>(__float_as_uint(x), lane)));
    x = fmaxf(x, __uint_as_float(xor_lane<2>(__float_as_uint(x), lane)));
    x = fmaxf(x, __uint_as_float(xor_lane<4>(__float_as_uint(x), lane)));
    x = fmaxf(x, __uint_as_float(xor_lane<8>(__float_as_uint(x), lane)));
    x = fmaxf(x, __uint_as_float(xor_lane<16>(__float_as_uint(x), lane)));
    x = fmaxf(x, __uint_as_float(xor_lane<32>(__float_as_uint(x), lane)));
    return x;
}
// Sum over the wavefront in a fixed butterfly order (the same bits in every lane and every launch).
__device__ __forceinline__ float wave_sum(float x, int lane) {
    x += __uint_as_float(xor_lane<1>(__float_as_uint(x), lane));
    x += __uint_as_float(xor_lane<2>(__float_as_uint(x), lane));
    x += __uint_as_float(xor_lane<4>(__float_as_uint(x), lane));
    x += __uint_as_float(xor_lane<8>(__float_as_uint(x), lane));
    x += __uint_as_float(xor_lane<16>(__float_as_uint(x), lane));
    x += __uint_as_float(xor_lane<32>(__float_as_uint(x), lane));
    return x;
}

// The q-th largest (counting repeats, 1 <= q <= 64) of the 64 values of a wavefront: the largest t
// that at least q values reach, found bit by bit.  One vector compare per bit, the rest is scalar:
// with 8 wavefronts per SIMD this costs a fifth of sorting the 64 values.
__device__ __forceinline__ uint32_t wave_kth_largest(uint32_t v, int q) {
    uint32_t t = 0;
#pragma unroll
    for (int bit = 31; bit >= 0; --bit) {
        const uint32_t c = t | (1u << bit);
        if (__popcll(__ballot(v >= c)) >= q) t = c;              // (uniform)
    }
    return t;
}

}  // namespace evospec

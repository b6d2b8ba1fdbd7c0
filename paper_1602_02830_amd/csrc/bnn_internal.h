// Internal helpers shared by the HIP translation units of libbnn_hip.
// Written for gfx950 (CDNA4, 64-wide wavefronts) only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bnn.h"

// v_writelane_b32 through its LLVM intrinsic (this compiler exposes no __builtin for it):
// returns `old` with lane `lane` replaced by the wavefront-uniform `value`.
extern "C" __device__ int bnn_llvm_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace bnn {

constexpr int kWave = 64;
constexpr int64_t kMaxDim = (int64_t(1) << 31) - 1;
// Largest K of a product: the kernels hold K and ceil(K / 32) = (K + 31) >> 5 in 32-bit integers.
constexpr int64_t kMaxK = (int64_t(1) << 31) - 32;

inline bool aligned_to(const void* p, size_t a) {
    return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0;
}

inline int check_launch() {
    return hipGetLastError() == hipSuccess ? BNN_OK : BNN_ERR_LAUNCH;
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Most workgroups of one launch: it holds fewer than 2^32 work items in a dimension.
inline constexpr int64_t max_blocks(int threads) { return ((int64_t(1) << 32) - 1) / threads; }

// Store of an int32 result with agent scope (global_store_dword ... sc1: written through the die's L2).
// Measured against plain and non-temporal stores on whole int32 products, it is the fastest policy while the
// output is not much larger than the last-level cache, and by far the fastest where rows of the output are
// not whole 128-byte lines (3000 x 3000 x 784: 13.6 vs 20.0 us).
__device__ inline void store_result(int32_t* p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Four consecutive results, 4-byte aligned, with the same policy.  The compiler keeps vector writes to the data registers
// of a store of more than 64 bits two wait states behind it, but does not see a store in assembly: the wait is part of it.
__device__ inline void store_result4(int32_t* p, int4 v) {
    typedef int quad_t __attribute__((ext_vector_type(4)));
    const quad_t q = {v.x, v.y, v.z, v.w};
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(q) : "memory");
}

// Mask of the valid bits of the last word of a K-bit row (all ones if K % 32 == 0).
__host__ __device__ inline uint32_t tail_mask(int64_t K) {
    const int r = int(K & 31);
    return r ? ((1u << r) - 1u) : 0xFFFFFFFFu;
}

// OR over each aligned group of 8 lanes, result in every lane of the group.
// Data-parallel-primitive (DPP) lane permutes: xor-1 and xor-2 inside a quad,
// then a mirror of the 8-lane half row, which swaps the two quads.
// Every lane of the wavefront must be active.
__device__ inline uint32_t or_reduce8(uint32_t v) {
    v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    v |= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x141, 0xF, 0xF, true));  // row_half_mirror
    return v;
}

// Work split of the streaming kernels' fast path (rows that are whole numbers of 128-element units, 16-byte
// aligned): a unit is 4 consecutive output words = 128 consecutive elements of one row, taken by an aligned group
// of 8 lanes; a 256-thread workgroup takes 32 consecutive units, counted row by row, `rows` rows (1 or 2) at a
// time - for one row at a time 16 KB of contiguous input when rows are dense.
constexpr int kUnitsPerBlock = 32;

struct UnitAt {
    int64_t row;   // first row of the group
    int unit;      // unit within the row
};

// Group `gi` of workgroup `block`.
__device__ inline UnitAt unit_at(uint32_t block, uint32_t gi, int units_per_row, int rows) {
    const uint32_t u = block * kUnitsPerBlock + gi, r = u / uint32_t(units_per_row);
    return UnitAt{int64_t(r) * rows, int(u - r * uint32_t(units_per_row))};
}

// Workgroups of the fast path for `rows_total` rows taken `rows` at a time; 0 if the shape does not fit it.
inline int64_t unit_blocks(int64_t rows_total, int64_t cols, int rows) {
    if (cols <= 0 || cols % 128 != 0) return 0;
    const int64_t blocks = ceil_div(ceil_div(rows_total, rows) * (cols / 128), kUnitsPerBlock);
    return blocks <= max_blocks(8 * kUnitsPerBlock) ? blocks : 0;
}

}  // namespace bnn

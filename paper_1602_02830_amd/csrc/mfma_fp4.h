// Pieces shared by the matrix-engine (fp4 MFMA) kernels: bit widening, row sums, and the
// epilogue that turns the MFMA sums into +-1 dot products or packed output bits.
#pragma once

#include <type_traits>

#include "bnn_internal.h"
#include "gemm_staging.h"

namespace bnn {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kMfmaKT = 16;              // words of A per row and staged tile
constexpr int kMfmaKQ = kMfmaKT / 4;     // 16-byte quads per row per tile
constexpr int64_t kMfmaMaxAcc = int64_t(1) << 24;   // exact fp32 accumulation of non-negative integers

__device__ inline v8i widen_fp4_a(uint32_t w) {
    v8i f = {int(w & 0x11111111u), int(w & 0x22222222u), int(w & 0x44444444u), int((w >> 2) & 0x22222222u),
             0, 0, 0, 0};
    return f;
}

__device__ inline v8i widen_fp4_b(uint32_t w) {
    const uint32_t r = w >> 2;
    v8i f = {int((w << 2) & 0x44444444u), int(w & 0x22222222u), int(r & 0x11111111u), int(r & 0x22222222u),
             0, 0, 0, 0};
    return f;
}

// The four fp4 operand registers of a word alone; the MFMA's operand type has eight, of which the fp4 format reads four.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ inline v4i widen4_a(uint32_t w) {
    return v4i{int(w & 0x11111111u), int(w & 0x22222222u), int(w & 0x44444444u), int((w >> 2) & 0x22222222u)};
}
__device__ inline v4i widen4_b(uint32_t w) {
    const uint32_t r = w >> 2;
    return v4i{int((w << 2) & 0x44444444u), int(w & 0x22222222u), int(r & 0x11111111u), int(r & 0x22222222u)};
}
__device__ inline v8i operand8(v4i f) { return v8i{f[0], f[1], f[2], f[3], 0, 0, 0, 0}; }

__device__ inline int popc4(uint4 v) { return __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w); }

__device__ inline uint32_t quad_word(const uint4& q, int s) { return s == 0 ? q.x : s == 1 ? q.y : s == 2 ? q.z : q.w; }

// int32 epilogue of a wavefront that owns WM x WN blocks of 32 x 32 fp32 accumulators at block
// position (wm, wn) of a (64*WM) x (64*WN) workgroup tile whose first row / column is row0 / col0.
// pop_a[tile row] / pop_b[tile column] hold 2*popcount.  fr = lane % 32, fh = lane / 32.
template <int WM, int WN>
__device__ inline void mfma_epilogue(const v16f (&acc)[WM][WN], const int* pop_a, const int* pop_b,
                                     int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, int row0, int col0,
                                     int wm, int wn, int fr, int fh) {
    // Result from the matrix-engine sum S: K - 2pa - 2pb + 4S.
    // Accumulator register v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32 of its 32x32 block.
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        const int nl = wn * 32 * WN + j * 32 + fr;
        const int n = col0 + nl;
        const int base_n = K - pop_b[nl];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const int ml = wm * 32 * WM + i * 32 + 8 * vq + 4 * fh;
                const int4 pa2 = *reinterpret_cast<const int4*>(&pop_a[ml]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = row0 + ml + e;
                    const int pa = e == 0 ? pa2.x : e == 1 ? pa2.y : e == 2 ? pa2.z : pa2.w;
                    const int dot = base_n - pa + (int(acc[i][j][4 * vq + e]) << 2);
                    if (m < M && n < N) store_result(&C[int64_t(m) * ldc + n], dot);
                }
            }
    }
}

// int32 epilogue of a wavefront whose accumulators hold the TRANSPOSED blocks (operands swapped, as for
// mfma_epilogue_bits below): a lane holds 16 columns of one output row in groups of 4.  16 rows x 64 columns at a time
// go through a wavefront's own piece of LDS (kStoreScratch floats, any memory that the K loop has left; rows padded to
// 68 floats, so that the 16-byte writes of 8 rows fall into different banks) and leave as 16-byte stores of 256
// consecutive bytes per row: a quarter of the store instructions of mfma_epilogue, and half of the lines that two of
// them share where rows are not whole 128-byte lines.
constexpr int kStoreRows = 16, kStorePitch = 68, kStoreScratch = kStoreRows * kStorePitch;

// Which int32 outputs take it: rows that are not whole, aligned 128-byte lines (6000 x 3000 x 2100 35.0 -> 29.8 us,
// 13000 x 2001 x 1300 35.4 -> 31.7, 9000 x 3000 x 3000 50.5 -> 45.1, 9000 x 2500 x 400 24.7 -> 22.4, 3000 x 3000 x 784
// 12.8 -> 12.1).  Where mfma_epilogue's stores are whole lines it is level or better (8192 x 4096 x 1200 35.9 vs 34.7, but
// 6144 x 2048 x 1500 15.3 vs 16.8; the whole-tile kernel, 8192 x 8192 x 2048, 67.6 vs 75.8).
inline bool wants_row_stores(const int32_t* C, int64_t ldc) { return ldc % 32 != 0 || !aligned_to(C, 128); }

template <int WM, int WN>
__device__ inline void mfma_epilogue_rows(const v16f (&acc)[WM][WN], float* scratch, const int* pop_a, const int* pop_b,
                                          int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, int row0, int col0,
                                          int wm, int wn, int lane) {
    static_assert(WN == 2, "a wavefront's rows are 64 columns");
    const int fr = lane & 31, fh = lane >> 5;
    const int cg = lane & 15, rr = lane >> 4;              // on the way out: column group and row of four
    const int n = col0 + wn * 64 + 4 * cg;
    const int4 pb2 = *reinterpret_cast<const int4*>(&pop_b[wn * 64 + 4 * cg]);
    int32_t* to = C + int64_t(row0 + wm * 32 * WM + rr) * ldc + n;              // the lane's rows are 4 apart
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if ((fr >> 4) == p) {
                float* at = scratch + (fr & 15) * kStorePitch + 4 * fh;
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        *reinterpret_cast<float4*>(at + j * 32 + 8 * g) =
                            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            }
            asm volatile("" : : : "memory");               // LDS is in order within a wavefront; so is the code
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < kStoreRows / 4; ++t) {
                const int lr = 4 * t + rr, ml = wm * 32 * WM + i * 32 + 16 * p + lr, m = row0 + ml;
                const float4 s = *reinterpret_cast<const float4*>(scratch + lr * kStorePitch + 4 * cg);
                const int base = K - pop_a[ml];
                const int4 dot = make_int4(base - pb2.x + (int(s.x) << 2), base - pb2.y + (int(s.y) << 2),
                                           base - pb2.z + (int(s.z) << 2), base - pb2.w + (int(s.w) << 2));
                if (m < M) {
                    if (n + 4 <= N) {
                        store_result4(to, dot);
                    } else {
                        if (n < N) store_result(to, dot.x);
                        if (n + 1 < N) store_result(to + 1, dot.y);
                        if (n + 2 < N) store_result(to + 2, dot.z);
                    }
                }
                to += 4 * ldc;
            }
            asm volatile("" : : : "memory");
            __builtin_amdgcn_wave_barrier();
        }
}

// Largest K for which the fused binary epilogue below may fold its threshold into the accumulators:
// every term is a multiple of 1/8 and the largest magnitude is about 2K, exact in fp32 below 2^21.
constexpr int kMfmaFoldMaxK = 1 << 19;

// Column term of the folded threshold (see mfma_epilogue_bits): 1/8 - (thr - K + 2*popcount(B_n)) / 4,
// pop_b2 = 2*popcount(B_n), thr clamped to [-K-1, K+1].  Exact in fp32 for K <= kMfmaFoldMaxK.
__device__ inline float fold_column_term(int thr, int K, int pop_b2) {
    return 0.125f - 0.25f * float(thr - K + pop_b2);
}

// Fused epilogue (binary product) of a wavefront whose accumulators hold the TRANSPOSED blocks:
// the kernel issued its MFMAs with the operands swapped, so accumulator register v of lane l is
// column 8*(v/4) + 4*(l/32) + v%4 and row l%32 of its 32 x 32 block - a lane holds 16 columns of
// ONE output row, and the output bits of a row can be packed inside the lane, without ballots.
//
//   bit(m, n) = (K - 2pa - 2pb + 4S >= thr) XOR flip  =  (S - pa/2 - (thr - K + 2pb)/4 + 1/8 > 0) XOR flip
//
// (all terms multiples of 1/4, so adding 1/8 turns >= 0 into > 0 and the sum is never zero).
// For K <= kMfmaFoldMaxK the row term -pa/2 and the column term colfix_s[n] (fold_column_term)
// are added to all 1024 accumulators of a block by one v_mfma_f32_32x32x2_f32 (a rank-2 update:
// column term x 1 + 1 x row term, exact in fp32), after which the output bit is the complement of
// the accumulator's sign bit: one v_alignbit per accumulator shifts it into the lane's word.
// Larger K compare in integers.  The two lane halves hold alternate groups of 4 columns; one
// v_permlane32_swap brings the halves of column block 0 to lanes 0-31 and those of block 1 to
// lanes 32-63, so that lane l stores the word of column block l / 32.
// pop_a / pop_b as in mfma_epilogue; pop_af[tile row] = pop_a / 4 as float; thr_s[tile column] / flip_s[tile
// column / 32]: the tile's thresholds and flip words (zero for columns beyond N).
// mfma_output_words leaves, in words[i], the finished output word (flip and column validity
// applied) of tile row wm*32*WM + i*32 + fr and column block fh of this wavefront's column pair;
// mfma_epilogue_bits stores them.
template <int WM, int WN>
__device__ inline void mfma_output_words(v16f (&acc)[WM][WN], const int* pop_a, const float* pop_af,
                                         const int* pop_b, const int* thr_s, const uint32_t* flip_s,
                                         const float* colfix_s, int N, int K, int col0, int wm, int wn, int fr,
                                         int fh, uint32_t (&words)[WM]) {
    static_assert(WN == 2, "the two column blocks are paired with the two lane halves");
    const uint32_t flip_word = flip_s[wn * WN + fh];                    // col0 is a multiple of 32
    const int cols_left = N - (col0 + wn * 32 * WN + fh * 32);
    const uint32_t live_word = cols_left >= 32 ? ~0u : cols_left <= 0 ? 0u : ((1u << cols_left) - 1u);
    const bool fold = K <= kMfmaFoldMaxK;
    // Operands of the rank-2 update: lane (r, h) holds element [r][k = h] of the 32 x 2 left factor
    // (column term, 1) and element [k = h][r] of the 2 x 32 right factor (1, row term).
    float left[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) left[j] = fh == 0 ? colfix_s[wn * 32 * WN + j * 32 + fr] : 1.0f;
    if (fold) {
        // All rank-2 updates first: the vector-ALU work on a block then never waits for its own MFMA.
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const float right = fh == 0 ? 1.0f : -pop_af[wm * 32 * WM + i * 32 + fr];
#pragma unroll
            for (int j = 0; j < WN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(left[j], right, acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int ml = wm * 32 * WM + i * 32 + fr;                       // this lane's row of the tile
        uint32_t part[WN];                                               // this lane's 16 columns: nibble g at bit 8g + 4*fh
        if (fold) {
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                // Sign bits of the block's 16 registers, nibble g (columns 8g + 4*fh ...) moved to bit 8g on the way.
                uint32_t neg = 0u;
#pragma unroll
                for (int g = 3; g >= 0; --g) {
#pragma unroll
                    for (int e = 3; e >= 0; --e)
                        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[i][j][4 * g + e]), 31);
                    if (g > 0) neg <<= 4;
                }
                part[j] = (~neg & 0x0F0F0F0Fu) << (4 * fh);
            }
        } else {
            const int base_m = K - pop_a[ml];
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                uint32_t bits = 0u;
#pragma unroll
                for (int g = 3; g >= 0; --g) {
                    const int nl = wn * 32 * WN + j * 32 + 8 * g + 4 * fh;
                    const int4 pb2 = *reinterpret_cast<const int4*>(&pop_b[nl]);
                    const int4 th = *reinterpret_cast<const int4*>(&thr_s[nl]);
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        const int pb = e == 0 ? pb2.x : e == 1 ? pb2.y : e == 2 ? pb2.z : pb2.w;
                        const int t = e == 0 ? th.x : e == 1 ? th.y : e == 2 ? th.z : th.w;
                        const int dot = base_m - pb + (int(acc[i][j][4 * g + e]) << 2);
                        bits = (bits << 1) | (dot >= t ? 1u : 0u);
                    }
                }
                // Bit 4g + e of bits is column 8g + 4*fh + e of block j: move nibble g to bit 8g + 4*fh.
                uint32_t x = bits;
                x = (x | (x << 8)) & 0x00FF00FFu;
                x = (x | (x << 4)) & 0x0F0F0F0Fu;
                part[j] = x << (4 * fh);
            }
        }
        // Lanes 32-63 of part[0] <-> lanes 0-31 of part[1]: afterwards lane l holds, in the two
        // registers, the two halves of the word of column block l / 32.
        const auto sw = __builtin_amdgcn_permlane32_swap(part[0], part[1], false, false);
        words[i] = ((sw[0] | sw[1]) ^ flip_word) & live_word;
    }
}

template <int WM, int WN>
__device__ inline void mfma_epilogue_bits(v16f (&acc)[WM][WN], const int* pop_a, const float* pop_af,
                                          const int* pop_b, const int* thr_s, const uint32_t* flip_s,
                                          const float* colfix_s, const BnSignArgs& bn, int M, int N, int K,
                                          int row0, int col0, int wm, int wn, int fr, int fh) {
    uint32_t words[WM];
    mfma_output_words<WM, WN>(acc, pop_a, pop_af, pop_b, thr_s, flip_s, colfix_s, N, K, col0, wm, wn, fr, fh, words);
    const int64_t nw = (int64_t(N) + 31) >> 5;
    const int64_t w = ((int64_t(col0) + wn * 32 * WN) >> 5) + fh;       // word column of this lane
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int m = row0 + wm * 32 * WM + i * 32 + fr;
        if (m < M && w < nw) bn.out[int64_t(m) * bn.ld_out + w] = words[i];
    }
}

// 2 x 2 pooling of output words whose windows are four neighbouring lanes (every lane active): OR where the channel's flip
// bit is 0, AND where it is 1, in all four lanes.
__device__ inline uint32_t pool_words(uint32_t word, uint32_t flip_word) {
    uint32_t any = word, all = word;
    any |= uint32_t(__builtin_amdgcn_update_dpp(0, int(any), 0xB1, 0xF, 0xF, true));      // lane ^ 1
    all &= uint32_t(__builtin_amdgcn_update_dpp(0, int(all), 0xB1, 0xF, 0xF, true));
    any |= uint32_t(__builtin_amdgcn_update_dpp(0, int(any), 0x4E, 0xF, 0xF, true));      // lane ^ 2
    all &= uint32_t(__builtin_amdgcn_update_dpp(0, int(all), 0x4E, 0xF, 0xF, true));
    return (any & ~flip_word) | (all & flip_word);
}

// Integers n / 8 of at most 16 bits as two bf16 numbers: the upper eight bits and the rest, both exact.  The largest that start an
// accumulator, in eighths: 4K + 3, the column term of a threshold -K - 1 or K + 1 (fold_column_term); -pa / 2 has 4K.
constexpr bool starts_in_bf16_pairs(int K) { return 4 * K + 3 < 1 << 16; }
typedef short v4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void split_bf16(float v, short& hi, short& lo) {
    const uint32_t top = __float_as_uint(v) & 0xFFFF0000u;
    hi = short(top >> 16);
    lo = short(__float_as_uint(v - __uint_as_float(top)) >> 16);
}

// The K loops of the strip kernels.  After every product: VALU vector operations and, with READ, one LDS read.
#define BNN_STRIP_SCHEDULE(MFMAS, READ, VALU)                               \
    do {                                                                    \
        _Pragma("unroll") for (int g_ = 0; g_ < (MFMAS); ++g_) {            \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);              \
            __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);           \
            if (READ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    \
        }                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                  \
    } while (0)

}  // namespace bnn

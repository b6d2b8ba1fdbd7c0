// bnn_pack_sign: Eq. (1) binarisation fused with the 32-per-word packing of Sec. 4.
//
// HBM-bound streaming kernel: 4 B read and 1/8 B written per element.
// Work unit: one output word = 32 consecutive elements of a row, handled by an
// aligned group of 8 lanes; each lane reads 4 consecutive floats (one 16-byte
// load, whatever the row's alignment), forms a 4-bit nibble and the group ORs the shifted
// nibbles together with three DPP permutes.  A wavefront therefore reads eight
// 128-byte segments and writes eight words per step, and groups never straddle
// a row, so rows whose length is not a multiple of 32 cost nothing extra apart
// from their own partial last word.  Rows that are whole numbers of 128 elements
// take pack_sign_units_kernel (4 words per group, one 16-byte store), long rows of other lengths pack_sign_pieces_kernel.
#include "bit_transpose.h"
#include "bnn_internal.h"
#include "row_pieces.h"

namespace bnn {

constexpr int kPackThreads = 256;
constexpr int kPackUnroll = 4;   // words per group of 8 lanes per pass (loads in flight)

__device__ inline uint32_t ge_zero(float v) { return v >= 0.0f ? 1u : 0u; }

// 16-byte load of the input.  ONCE: non-temporal, for inputs larger than the last-level cache, where nothing
// read now is found again later and the default policy only displaces what else is cached (1 GiB input:
// 6.02 -> 6.45 TB/s).  Inputs that fit the cache keep the default policy: they are often still there from
// their producer or from the previous step, and a non-temporal read does not find them (31 MB MLP input,
// re-read every step: 5.8 -> 5.5 TB/s non-temporally).
constexpr int64_t kOnceMinBytes = int64_t(256) << 20;
// The address need only be 4-byte aligned: rows of odd length take the same loads as all others (28754 x 3005:
// 111 us with four 4-byte loads per lane, 55 with one of 16 bytes).
template <bool ONCE>
__device__ inline float4 load_input(const float* p) {
    typedef float quad_t __attribute__((ext_vector_type(4), aligned(4)));
    const quad_t* q = reinterpret_cast<const quad_t*>(p);
    const quad_t t = ONCE ? __builtin_nontemporal_load(q) : *q;
    return make_float4(t[0], t[1], t[2], t[3]);
}

// Word groups are numbered row-major (g = row * kw + word).  (row, word) coordinates are stepped by a
// constant number of groups with a carry instead of being divided out for every group; both fit 32 bits.
struct WordStep {
    int d_row;   // groups / kw
    int d_word;  // groups % kw
};

inline WordStep word_step(int64_t groups, int64_t kw) { return WordStep{int(groups / kw), int(groups % kw)}; }

__device__ inline void advance(uint32_t& row, int& w, const WordStep& st, int kw) {
    row += st.d_row;
    w += st.d_word;
    if (w >= kw) {
        w -= kw;
        ++row;
    }
}

// A workgroup takes kPackUnroll consecutive slices of 32 word groups per pass (16 KB of contiguous
// input when rows are dense), thread t group t/8 of each slice; passes are a whole grid apart.
template <bool ONCE>
__global__ __launch_bounds__(kPackThreads) void pack_sign_kernel(
    const float* __restrict__ x, int cols, int64_t ld_x,
    uint32_t* __restrict__ out, int64_t ld_out, int kw, int64_t n_words, WordStep slice, WordStep pass) {
    constexpr int kSlice = kPackThreads / 8;             // word groups per slice
    const int q = threadIdx.x & 7;                       // lane within its group
    const int64_t pass_groups = int64_t(gridDim.x) * kSlice * kPackUnroll;
    int64_t g0 = int64_t(blockIdx.x) * kSlice * kPackUnroll + (threadIdx.x >> 3);
    uint32_t row0 = uint32_t(g0 / kw);                   // the only division of the thread
    int w0 = int(g0 - int64_t(row0) * kw);

    for (; g0 < n_words; g0 += pass_groups) {
        uint32_t nib[kPackUnroll];
        uint32_t row_of[kPackUnroll];                    // ~0: no such group
        int word_of[kPackUnroll];
        uint32_t row = row0;
        int w = w0;
        if (cols >= 4) {
            // Four unconditional 16-byte loads, all in flight together: a lane whose four elements do not all
            // exist (a slice past the last group, the tail of a row) loads the row's last four elements instead
            // and shifts away the bits that belong to the lanes before it.
            float4 f[kPackUnroll];
            int past[kPackUnroll];
#pragma unroll
            for (int u = 0; u < kPackUnroll; ++u) {
                const bool live = g0 + u * kSlice < n_words;
                row_of[u] = live ? row : ~0u;
                word_of[u] = w;
                const int c = live ? w * 32 + q * 4 : 0, c_at = min(c, cols - 4);
                past[u] = c - c_at;
                f[u] = load_input<ONCE>(x + int64_t(live ? row : 0u) * ld_x + c_at);
                advance(row, w, slice, kw);
            }
#pragma unroll
            for (int u = 0; u < kPackUnroll; ++u)
                nib[u] = (ge_zero(f[u].x) | (ge_zero(f[u].y) << 1) | (ge_zero(f[u].z) << 2) | (ge_zero(f[u].w) << 3)) >> past[u];
        } else {
#pragma unroll
            for (int u = 0; u < kPackUnroll; ++u) {
                const bool live = g0 + u * kSlice < n_words;
                row_of[u] = live ? row : ~0u;
                word_of[u] = w;
                const float* p = x + int64_t(live ? row : 0u) * ld_x;          // unconditional loads here too
                nib[u] = 0u;
#pragma unroll
                for (int e = 0; e < 3; ++e) nib[u] |= ge_zero(p[min(e, cols - 1)]) << e;
                nib[u] = q == 0 ? nib[u] & ((1u << cols) - 1u) : 0u;
                advance(row, w, slice, kw);
            }
        }
#pragma unroll
        for (int u = 0; u < kPackUnroll; ++u) {
            const uint32_t word = or_reduce8(nib[u] << (4 * q));
            if (q == 0 && row_of[u] != ~0u) out[int64_t(row_of[u]) * ld_out + word_of[u]] = word;
        }
        advance(row0, w0, pass, kw);
    }
}

// Fast path for rows that are whole numbers of 128-element units (see unit_at): a group of 8 lanes
// takes 4 consecutive output words, each of its four 16-byte loads per lane covers 128 contiguous bytes
// of the group, and lane 0 writes the four words with one 16-byte store, so a wavefront's store is one
// full 128-byte line instead of four partial ones.
template <bool ONCE>
__global__ __launch_bounds__(kPackThreads) void pack_sign_units_kernel(
    const float* __restrict__ x, int64_t rows, int64_t ld_x, uint32_t* __restrict__ out, int64_t ld_out,
    int units_per_row) {
    const int q = threadIdx.x & 7;
    const UnitAt at = unit_at(blockIdx.x, threadIdx.x >> 3, units_per_row, 1);
    if (at.row >= rows) return;
    const float* p = x + at.row * ld_x + int64_t(at.unit) * 128 + q * 4;
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = load_input<ONCE>(p + 32 * u);
    uint32_t w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t nib = ge_zero(v[u].x) | (ge_zero(v[u].y) << 1) | (ge_zero(v[u].z) << 2) | (ge_zero(v[u].w) << 3);
        w[u] = or_reduce8(nib << (4 * q));
    }
    if (q == 0)
        *reinterpret_cast<uint4*>(out + at.row * ld_out + int64_t(at.unit) * 4) = make_uint4(w[0], w[1], w[2], w[3]);
}

// The same for rows of any length and alignment, in pieces of 128 elements of which a row's last may be partial: a load that would pass the
// row's end takes its last four elements instead, and the nibble is shifted to where it belongs.  Lane q < 4 of a group stores
// word q.  For inputs that the last-level cache holds, which are bound by the number of instructions: no carry from word to word, no address
// per word.  us, before and now: 10000 x 784 4.9 and 3.9, 1000 x 784 2.25 and 2.05, 700 x 6001 3.2 and 2.5, 100000 x 500 29.7 and 29.0.
// Larger inputs are read past the cache, which does not bear lines that two loads share: 28754 x 3005 54 and 75.
__global__ __launch_bounds__(kPackThreads) void pack_sign_pieces_kernel(
    const float* __restrict__ x, int64_t rows, PieceRow row, int64_t ld_x, uint32_t* __restrict__ out, int64_t ld_out) {
    const int q = threadIdx.x & 7;
    const UnitAt at = unit_at(blockIdx.x, threadIdx.x >> 3, row.pieces(), 1);
    if (at.row >= rows) return;
    const float* p = x + at.row * ld_x;
    PieceRow::Quad quad[4];
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        quad[u] = row.quad(at.unit, u, q);
        v[u] = load_input<false>(p + quad[u].at);
    }
    uint32_t w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t nib = ge_zero(v[u].x) | (ge_zero(v[u].y) << 1) | (ge_zero(v[u].z) << 2) | (ge_zero(v[u].w) << 3);
        w[u] = or_reduce8((nib >> quad[u].past) << (4 * q));
    }
    if (row.stores(at.unit, q)) out[at.row * ld_out + at.unit * 4 + q] = q == 0 ? w[0] : q == 1 ? w[1] : q == 2 ? w[2] : w[3];
}

// Workgroups for the rows that take it, 0 for others: those of pieces_of, while one launch holds them.
static int64_t piece_blocks(int64_t rows, int64_t kw) {
    const int64_t blocks = ceil_div(rows * pieces_of(kw), kUnitsPerBlock);
    return blocks <= max_blocks(8 * kUnitsPerBlock) ? blocks : 0;
}

// ----------------------------------------------------------------------------
// bnn_pack_bitplanes: 8-bit inputs of the first layer (Sec. 1.6, Alg. 4 step 1) as eight
// packed bit planes.  out[r][8*w + p] holds bit p of x[r][32*w .. 32*w + 31].
//
// One thread per 32 elements: two 16-byte loads, a 4 x 4 byte transposition (16 v_perm) and an 8 x 8 bit
// transposition (48 operations) turn 32 bytes into 8 plane words, which leave as two 16-byte stores.  The kernel
// streams 1 B in and 1 B out per element and is bound by memory: 10000 x 784 4.5 us per launch against 10 when 8 lanes
// shared a word and gathered every plane with a multiply and three lane permutes.
// A row's last, partial word reads the row's last 32 elements instead and shifts the planes down.
// ----------------------------------------------------------------------------
__device__ inline uint4 load_bytes16(const uint8_t* p) {
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(1)));
    const quad_t v = *reinterpret_cast<const quad_t*>(p);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// The bytes of a row of 1 .. 31 as eight words, zero past its end: two loads that overlap in its middle, the second one
// shifted to where its bytes belong.  All conditions are the same for every thread.  (Byte by byte, each load waited for:
// 4400 rows of 20 3.6 us, 2.5 this way; 1000000 of 27 25.6 and 11.4.)
__device__ inline void load_short_row(const uint8_t* p, int cols, uint32_t (&w)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = 0u;
    if (cols >= 16) {
        const uint4 lo = load_bytes16(p), hi = load_bytes16(p + cols - 16);
        const int past = 32 - cols;                       // bytes of hi that lo has, 1 .. 16
        const uint64_t h0 = uint64_t(hi.y) << 32 | hi.x, h1 = uint64_t(hi.w) << 32 | hi.z;
        const int bits = 8 * (past & 7);
        const uint64_t low = bits == 0 ? h0 : h0 >> bits | h1 << (64 - bits), high = h1 >> bits;      // past bytes within 8
        const uint64_t v0 = past < 8 ? low : past < 16 ? high : 0u, v1 = past < 8 ? high : 0u;
        w[0] = lo.x; w[1] = lo.y; w[2] = lo.z; w[3] = lo.w;
        w[4] = uint32_t(v0); w[5] = uint32_t(v0 >> 32); w[6] = uint32_t(v1); w[7] = uint32_t(v1 >> 32);
    } else if (cols >= 8) {
        typedef uint32_t pair_t __attribute__((ext_vector_type(2), aligned(1)));
        const pair_t lo = *reinterpret_cast<const pair_t*>(p), hi = *reinterpret_cast<const pair_t*>(p + cols - 8);
        const uint64_t v = cols == 8 ? 0u : (uint64_t(hi[1]) << 32 | hi[0]) >> (8 * (16 - cols));
        w[0] = lo[0]; w[1] = lo[1]; w[2] = uint32_t(v); w[3] = uint32_t(v >> 32);
    } else if (cols >= 4) {
        typedef uint32_t word_t __attribute__((aligned(1)));
        const uint32_t lo = *reinterpret_cast<const word_t*>(p), hi = *reinterpret_cast<const word_t*>(p + cols - 4);
        w[0] = lo;
        w[1] = cols == 4 ? 0u : hi >> (8 * (8 - cols));
    } else {
        const uint32_t a = p[0], b = p[cols > 1 ? 1 : 0], c = p[cols - 1];
        w[0] = a | (cols > 1 ? b << 8 : 0u) | (cols > 2 ? c << 16 : 0u);
    }
}

__device__ inline void store_words4(uint32_t* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));
    *reinterpret_cast<quad_t*>(p) = quad_t{a, b, c, d};
}

// Bytes of four words as a 4 x 4 matrix, transposed: out w[s] byte j = in w[j] byte s.
__device__ inline void transpose_bytes_4x4(uint32_t (&w)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    w[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    w[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    w[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// SHORT: rows of fewer than 32 elements, one group each.
template <bool SHORT>
__global__ __launch_bounds__(kPackThreads) void pack_bitplanes_kernel(
    const uint8_t* __restrict__ x, int64_t cols, int64_t ld_x, uint32_t* __restrict__ out, int64_t ld_out, int64_t kw,
    int64_t n_groups) {
    for (int64_t base = int64_t(blockIdx.x) * kPackThreads; base < n_groups; base += int64_t(gridDim.x) * kPackThreads) {
        if (base + threadIdx.x >= n_groups) break;
        // The 64-bit division is the workgroup's, the thread's own is a 32-bit one (kw < 2^26).
        const int64_t row_base = SHORT ? base : base / kw;
        const uint32_t t = uint32_t(base - row_base * kw) + threadIdx.x;
        const uint32_t d_row = SHORT ? threadIdx.x : t / uint32_t(kw);
        const int64_t row = row_base + d_row;
        const int64_t w = SHORT ? 0 : t - d_row * uint32_t(kw);
        const int64_t c0 = w * 32;
        const uint8_t* p = x + row * ld_x;
        uint32_t even[4], odd[4];                         // 4-byte groups 0, 2, 4, 6 and 1, 3, 5, 7 of the 32
        int past = 0;                                     // elements of the word that do not exist
        if (!SHORT) {
            past = c0 + 32 <= cols ? 0 : int(c0 + 32 - cols);
            const uint4 lo = load_bytes16(p + c0 - past), hi = load_bytes16(p + c0 - past + 16);
            even[0] = lo.x; odd[0] = lo.y; even[1] = lo.z; odd[1] = lo.w;
            even[2] = hi.x; odd[2] = hi.y; even[3] = hi.z; odd[3] = hi.w;
        } else {
            uint32_t v[8];
            load_short_row(p, int(cols), v);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                even[i] = v[2 * i];
                odd[i] = v[2 * i + 1];
            }
        }
        transpose_bytes_4x4(even);
        transpose_bytes_4x4(odd);
        uint32_t pl[8] = {even[0], even[1], even[2], even[3], odd[0], odd[1], odd[2], odd[3]};
        transpose_bits_8x8(pl);
        uint32_t* o = out + row * ld_out + 8 * w;
        store_words4(o, pl[0] >> past, pl[1] >> past, pl[2] >> past, pl[3] >> past);
        store_words4(o + 4, pl[4] >> past, pl[5] >> past, pl[6] >> past, pl[7] >> past);
    }
}

}  // namespace bnn

extern "C" int bnn_pack_bitplanes(const uint8_t* x, int64_t rows, int64_t cols, int64_t ld_x, uint32_t* out,
                                  int64_t ld_out, void* stream) {
    using namespace bnn;
    if (rows < 0 || cols < 0 || rows > kMaxDim || cols > kMaxDim) return BNN_ERR_INVALID_ARG;
    const int64_t kw = ceil_div(cols, 32);
    if (ld_x < cols || ld_out < 8 * kw) return BNN_ERR_INVALID_ARG;
    if (rows == 0 || cols == 0) return BNN_OK;
    if (!x || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(out, 4)) return BNN_ERR_ALIGNMENT;
    const int64_t n_groups = rows * kw;
    int64_t blocks = ceil_div(n_groups, kPackThreads);
    if (blocks > max_blocks(kPackThreads)) blocks = max_blocks(kPackThreads);      // the kernel loops over the rest
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(kPackThreads), 0, static_cast<hipStream_t>(stream), x, cols, ld_x,
                           out, ld_out, kw, n_groups);
    };
    if (cols < 32) launch(pack_bitplanes_kernel<true>);
    else launch(pack_bitplanes_kernel<false>);
    return check_launch();
}

extern "C" int bnn_pack_sign(const float* x, int64_t rows, int64_t cols, int64_t ld_x,
                             uint32_t* out, int64_t ld_out, void* stream) {
    using namespace bnn;
    if (rows < 0 || cols < 0 || rows > kMaxDim || cols > kMaxDim) return BNN_ERR_INVALID_ARG;
    const int64_t kw = ceil_div(cols, 32);
    if (ld_x < cols || ld_out < kw) return BNN_ERR_INVALID_ARG;
    if (rows == 0 || cols == 0) return BNN_OK;
    if (!x || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(x, 4) || !aligned_to(out, 4)) return BNN_ERR_ALIGNMENT;

    const int64_t n_words = rows * kw;
    const int64_t groups_per_block = kPackThreads / 8;
    int64_t blocks = ceil_div(n_words, groups_per_block * kPackUnroll);
    // One pass per workgroup up to 16 GiB of input: measured faster than a smaller grid that loops
    // (1 GiB: 5.98 TB/s in one pass of 65536 workgroups, 5.60 TB/s with 8192 looping 8 times).
    const int64_t max_blocks = int64_t(1) << 20;
    if (blocks > max_blocks) blocks = max_blocks;
    const bool once = rows * cols * int64_t(sizeof(float)) > kOnceMinBytes;     // see load_input
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t units = unit_blocks(rows, cols, 1);
    if (units > 0 && aligned_to(x, 16) && ld_x % 4 == 0 && aligned_to(out, 16) && ld_out % 4 == 0) {
        if (once)
            hipLaunchKernelGGL(pack_sign_units_kernel<true>, dim3(unsigned(units)), dim3(kPackThreads), 0, s, x, rows, ld_x,
                               out, ld_out, int(cols / 128));
        else
            hipLaunchKernelGGL(pack_sign_units_kernel<false>, dim3(unsigned(units)), dim3(kPackThreads), 0, s, x, rows, ld_x,
                               out, ld_out, int(cols / 128));
        return check_launch();
    }
    if (const int64_t pieces = once ? 0 : piece_blocks(rows, kw)) {
        hipLaunchKernelGGL(pack_sign_pieces_kernel, dim3(unsigned(pieces)), dim3(kPackThreads), 0, s, x, rows, piece_row(cols), ld_x, out,
                           ld_out);
        return check_launch();
    }
    const WordStep slice = word_step(groups_per_block, kw);
    const WordStep pass = word_step(blocks * groups_per_block * kPackUnroll, kw);
    if (once)
        hipLaunchKernelGGL(pack_sign_kernel<true>, dim3(unsigned(blocks)), dim3(kPackThreads), 0, s,
                           x, int(cols), ld_x, out, ld_out, int(kw), n_words, slice, pass);
    else
        hipLaunchKernelGGL(pack_sign_kernel<false>, dim3(unsigned(blocks)), dim3(kPackThreads), 0, s,
                           x, int(cols), ld_x, out, ld_out, int(kw), n_words, slice, pass);
    return check_launch();
}

// bnn_bn_sign_pack: a^b_k = Sign(BatchNorm(a_k, theta_k)) of Alg. 4 on folded
// per-channel integer thresholds, written as packed bits for the next layer.
//
//   out[m][n/32] bit (n%32) = (C[m][n] >= thr[n]) XOR flip[n]
//
// HBM-bound streaming kernel (4 B read, 1/8 B written per element; thresholds
// and flip words stay in cache).  Same work split as the Sign packer: an
// aligned group of 8 lanes produces one output word, each lane comparing 4
// consecutive int32 (one 16-byte load, whatever the row's alignment), nibbles combined by
// three DPP permutes.  Rows that are whole numbers of 128 channels take
// bn_sign_pack_units_kernel (4 words per group, thresholds in registers,
// 16-byte stores), most other rows of 97 channels or more
// bn_sign_pack_pieces_kernel; everything else bn_sign_pack_kernel.
#include "bnn_internal.h"
#include "row_pieces.h"

namespace bnn {

// 16-byte load of pre-activations.  ONCE: non-temporal, for matrices larger than the last-level cache (1 GiB:
// 5.94 -> 6.01 TB/s); smaller ones are usually still cached from the product that wrote them, where a
// non-temporal read does not find them (164 MB: 5.8 -> 5.0 TB/s).  The thresholds, read by every row, always
// keep the default policy.
constexpr int64_t kOnceMinBytes = int64_t(256) << 20;
// The address need only be 4-byte aligned: rows of odd length take the same loads as all others (5284 x 2557: 28 us with
// four 4-byte loads of each operand per lane, 12 with one of 16 bytes).
typedef int quad_int __attribute__((ext_vector_type(4), aligned(4)));
template <bool ONCE>
__device__ inline int4 load_preact(const int32_t* p) {
    const quad_int* q = reinterpret_cast<const quad_int*>(p);
    const quad_int t = ONCE ? __builtin_nontemporal_load(q) : *q;
    return make_int4(t[0], t[1], t[2], t[3]);
}

constexpr int kBnThreads = 256;
constexpr int kBnUnroll = 4;
// Rows a workgroup of the fast path walks down with its thresholds in registers.  Measured on a 1 GiB input:
// 1 row 5.83 TB/s, 2 rows 5.95, 4 rows 5.75, 8 rows 5.60 (with or without the next row's loads issued early):
// short-lived workgroups keep the addresses in flight close together, which matters more than the saved
// threshold loads.  Counting units row by row lets any number of units per row in (9068 x 1280: 11.2 us in the general
// kernel, 8.5 here; 40000 x 1152: 32.0 and 28.0).
constexpr int kBnUnitRows = 2;

template <bool ONCE>
__global__ __launch_bounds__(kBnThreads) void bn_sign_pack_kernel(
    const int32_t* __restrict__ C, int64_t ldc, int N,
    const int32_t* __restrict__ thr, const uint32_t* __restrict__ flip_bits,
    uint32_t* __restrict__ out, int64_t ld_out, int nw, int64_t n_words, int slice_row, int slice_word, int pass_row,
    int pass_word) {
    // Word groups are numbered row-major (g = row * nw + word).  A workgroup takes kBnUnroll consecutive
    // slices of 32 groups per pass (16 KB of contiguous input when rows are dense), thread t group t/8 of
    // each slice; passes are a whole grid apart.  (row, word) are stepped by (groups / nw, groups % nw)
    // with a carry: one division per thread, not per group; all of them fit 32 bits.
    constexpr int kSlice = kBnThreads / 8;
    const int q = threadIdx.x & 7;
    const int64_t pass_groups = int64_t(gridDim.x) * kSlice * kBnUnroll;
    int64_t g0 = int64_t(blockIdx.x) * kSlice * kBnUnroll + (threadIdx.x >> 3);
    uint32_t row0 = uint32_t(g0 / nw);
    int w0 = int(g0 - int64_t(row0) * nw);

    for (; g0 < n_words; g0 += pass_groups) {
        uint32_t nib[kBnUnroll];
        uint32_t row_of[kBnUnroll];                      // ~0: no such group
        int word_of[kBnUnroll];
        uint32_t row = row0;
        int w = w0;
        if (N >= 4) {
            // Unconditional 16-byte loads of the pre-activations and of their thresholds, all in flight
            // together: a lane whose four channels do not all exist (a slice past the last group, the tail
            // of a row) loads the row's last four channels instead and shifts away the bits that belong to
            // the lanes before it.
            int4 c[kBnUnroll], t[kBnUnroll];
            int past[kBnUnroll];
#pragma unroll
            for (int u = 0; u < kBnUnroll; ++u) {
                const bool live = g0 + u * kSlice < n_words;
                row_of[u] = live ? row : ~0u;
                word_of[u] = w;
                const int n0 = live ? w * 32 + q * 4 : 0, n_at = min(n0, N - 4);
                past[u] = n0 - n_at;
                c[u] = load_preact<ONCE>(C + int64_t(live ? row : 0u) * ldc + n_at);
                t[u] = load_preact<false>(thr + n_at);
                row += slice_row;
                w += slice_word;
                if (w >= nw) {
                    w -= nw;
                    ++row;
                }
            }
#pragma unroll
            for (int u = 0; u < kBnUnroll; ++u)
                nib[u] = (uint32_t(c[u].x >= t[u].x) | (uint32_t(c[u].y >= t[u].y) << 1) |
                          (uint32_t(c[u].z >= t[u].z) << 2) | (uint32_t(c[u].w >= t[u].w) << 3)) >> past[u];
        } else {
#pragma unroll
            for (int u = 0; u < kBnUnroll; ++u) {
                const bool live = g0 + u * kSlice < n_words;
                row_of[u] = live ? row : ~0u;
                word_of[u] = w;
                // unconditional as well; the mask below drops what does not exist
                const int32_t* p = C + int64_t(live ? row : 0u) * ldc;
                nib[u] = 0u;
#pragma unroll
                for (int e = 0; e < 3; ++e) nib[u] |= uint32_t(p[min(e, N - 1)] >= thr[min(e, N - 1)]) << e;
                row += slice_row;
                w += slice_word;
                if (w >= nw) {
                    w -= nw;
                    ++row;
                }
            }
        }
        row0 += pass_row;
        w0 += pass_word;
        if (w0 >= nw) {
            w0 -= nw;
            ++row0;
        }
#pragma unroll
        for (int u = 0; u < kBnUnroll; ++u) {
            const int n0 = word_of[u] * 32 + q * 4;
            // Bits of channels >= N: flip word has zero pad bits, and the mask below clears them.
            const uint32_t flip = (flip_bits[word_of[u]] >> (4 * q)) & 0xFu;
            const int valid = N - n0;                           // channels left from this lane's first
            const uint32_t vmask = valid >= 4 ? 0xFu : (valid <= 0 ? 0u : ((1u << valid) - 1u));
            const uint32_t word = or_reduce8(((nib[u] ^ flip) & vmask) << (4 * q));
            if (q == 0 && row_of[u] != ~0u) out[int64_t(row_of[u]) * ld_out + word_of[u]] = word;
        }
    }
}

// Fast path for rows that are whole numbers of 128-channel units (see unit_at).  A group of lanes takes the same
// unit of kBnUnitRows consecutive rows, so a lane's 16 thresholds and flip nibbles are loaded once and stay in
// registers: per 16 bytes of pre-activations there is no second (cached) 16-byte threshold load and no flip-word
// load.  Lane 0 of a group writes its 4 output words with one 16-byte store.
template <bool ONCE>
__global__ __launch_bounds__(kBnThreads) void bn_sign_pack_units_kernel(
    const int32_t* __restrict__ C, int64_t ldc, int64_t M, const int32_t* __restrict__ thr,
    const uint32_t* __restrict__ flip_bits, uint32_t* __restrict__ out, int64_t ld_out, int units_per_row) {
    const int q = threadIdx.x & 7;
    const UnitAt at = unit_at(blockIdx.x, threadIdx.x >> 3, units_per_row, kBnUnitRows);
    const int64_t n0 = int64_t(at.unit) * 128 + q * 4;
    int4 t[4];
    uint32_t flip[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        t[u] = *reinterpret_cast<const int4*>(thr + n0 + 32 * u);
        flip[u] = (flip_bits[int64_t(at.unit) * 4 + u] >> (4 * q)) & 0xFu;
    }
    for (int i = 0; i < kBnUnitRows; ++i) {
        const int64_t row = at.row + i;
        if (row >= M) break;
        const int32_t* p = C + row * ldc + n0;
        int4 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = load_preact<ONCE>(p + 32 * u);
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t nib = (uint32_t(c[u].x >= t[u].x) | (uint32_t(c[u].y >= t[u].y) << 1) |
                                  (uint32_t(c[u].z >= t[u].z) << 2) | (uint32_t(c[u].w >= t[u].w) << 3)) ^ flip[u];
            w[u] = or_reduce8(nib << (4 * q));
        }
        if (q == 0)
            *reinterpret_cast<uint4*>(out + row * ld_out + int64_t(at.unit) * 4) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// The same for rows of any length and alignment, in pieces of 128 channels of which a row's last may be partial: loads that would pass
// the row's end take its last four channels instead, and the nibble is shifted to where it belongs.  Lane q < 4 of a group stores
// word q.  In cached matrices the number of instructions bounds such rows: against bn_sign_pack_kernel no carry from word to word, half the
// loads of thresholds, no mask per row.  us, before and now: 10000 x 4095 26.9 and 24.2, 10000 x 1000 8.2 and 6.6, 1000 x 1000 2.9 and
// 2.4, 700 x 6001 3.9 and 3.0, 300000 x 100 22.9 and 18.6.
template <bool ONCE>
__global__ __launch_bounds__(kBnThreads) void bn_sign_pack_pieces_kernel(
    const int32_t* __restrict__ C, int64_t ldc, int64_t M, PieceRow row, const int32_t* __restrict__ thr,
    const uint32_t* __restrict__ flip_bits, uint32_t* __restrict__ out, int64_t ld_out) {
    const int q = threadIdx.x & 7;
    const UnitAt at = unit_at(blockIdx.x, threadIdx.x >> 3, row.pieces(), kBnUnitRows);
    PieceRow::Quad quad[4];
    quad_int t[4];
    uint32_t flip[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        quad[u] = row.quad(at.unit, u, q);
        t[u] = *reinterpret_cast<const quad_int*>(thr + quad[u].at);
        flip[u] = (flip_bits[row.word(at.unit, u)] >> (4 * q)) & (0xFu >> quad[u].past);
    }
#pragma unroll
    for (int i = 0; i < kBnUnitRows; ++i) {
        const int64_t m = at.row + i;
        if (m >= M) break;
        const int32_t* p = C + m * ldc;
        int4 c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = load_preact<ONCE>(p + quad[u].at);
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t nib = uint32_t(c[u].x >= t[u][0]) | (uint32_t(c[u].y >= t[u][1]) << 1) |
                                 (uint32_t(c[u].z >= t[u][2]) << 2) | (uint32_t(c[u].w >= t[u][3]) << 3);
            w[u] = or_reduce8(((nib >> quad[u].past) ^ flip[u]) << (4 * q));
        }
        if (row.stores(at.unit, q)) out[m * ld_out + at.unit * 4 + q] = q == 0 ? w[0] : q == 1 ? w[1] : q == 2 ? w[2] : w[3];
    }
}

// Workgroups for the rows that take it, 0 for others: those of pieces_of, while one launch holds them.
static int64_t piece_blocks(int64_t M, int64_t nw) {
    const int64_t blocks = ceil_div(ceil_div(M, kBnUnitRows) * pieces_of(nw), kUnitsPerBlock);
    return blocks <= max_blocks(8 * kUnitsPerBlock) ? blocks : 0;
}

}  // namespace bnn

extern "C" int bnn_bn_sign_pack(const int32_t* C, int64_t ldc, int64_t M, int64_t N,
                                const int32_t* thr, const uint32_t* flip_bits, uint32_t* out,
                                int64_t ld_out, void* stream) {
    using namespace bnn;
    if (M < 0 || N < 0 || M > kMaxDim || N > kMaxDim) return BNN_ERR_INVALID_ARG;
    const int64_t nw = ceil_div(N, 32);
    if (ldc < N || ld_out < nw) return BNN_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return BNN_OK;
    if (!C || !thr || !flip_bits || !out) return BNN_ERR_INVALID_ARG;
    if (!aligned_to(C, 4) || !aligned_to(thr, 4) || !aligned_to(flip_bits, 4) || !aligned_to(out, 4))
        return BNN_ERR_ALIGNMENT;

    const int64_t n_words = M * nw;
    int64_t blocks = ceil_div(n_words, int64_t(kBnThreads / 8) * kBnUnroll);
    const int64_t max_blocks = int64_t(1) << 20;   // one pass per workgroup up to 16 GiB of input
    if (blocks > max_blocks) blocks = max_blocks;
    const bool once = M * N * int64_t(sizeof(int32_t)) > kOnceMinBytes;          // see load_preact
    const int64_t slice = kBnThreads / 8, pass = blocks * slice * kBnUnroll;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t units = unit_blocks(M, N, kBnUnitRows);
    if (units > 0 && aligned_to(C, 16) && aligned_to(thr, 16) && ldc % 4 == 0 && aligned_to(out, 16) && ld_out % 4 == 0) {
        if (once)
            hipLaunchKernelGGL(bn_sign_pack_units_kernel<true>, dim3(unsigned(units)), dim3(kBnThreads), 0, s, C, ldc, M,
                               thr, flip_bits, out, ld_out, int(N / 128));
        else
            hipLaunchKernelGGL(bn_sign_pack_units_kernel<false>, dim3(unsigned(units)), dim3(kBnThreads), 0, s, C, ldc, M,
                               thr, flip_bits, out, ld_out, int(N / 128));
        return check_launch();
    }
    if (const int64_t pieces = piece_blocks(M, nw)) {
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(unsigned(pieces)), dim3(kBnThreads), 0, s, C, ldc, M, piece_row(N), thr, flip_bits, out,
                               ld_out);
            return check_launch();
        };
        // A non-temporal load fetches a line again for the neighbour that shares it, so only rows of whole lines are read past the
        // cache: 20000 x 4000, before, now and with the default policy 60.1, 58.7 and 62.7 us; 28754 x 3005, before, now and
        // non-temporal 67.8, 67.3 and 79.5, 32768 x 8191 227.7, 209.5 and 249.9.
        return once && ldc % 32 == 0 && aligned_to(C, 128) ? launch(bn_sign_pack_pieces_kernel<true>)
                                                           : launch(bn_sign_pack_pieces_kernel<false>);
    }
    if (once)
        hipLaunchKernelGGL(bn_sign_pack_kernel<true>, dim3(unsigned(blocks)), dim3(kBnThreads), 0, s, C, ldc,
                           int(N), thr, flip_bits, out, ld_out, int(nw), n_words, int(slice / nw), int(slice % nw),
                           int(pass / nw), int(pass % nw));
    else
        hipLaunchKernelGGL(bn_sign_pack_kernel<false>, dim3(unsigned(blocks)), dim3(kBnThreads), 0, s, C, ldc,
                           int(N), thr, flip_bits, out, ld_out, int(nw), n_words, int(slice / nw), int(slice % nw),
                           int(pass / nw), int(pass % nw));
    return check_launch();
}

// First layer on 8-bit inputs (Alg. 4 step 1, Sec. 1.6) on the int8 matrix engine:
//
//   a_1 = sum_{n=1..8} 2^(n-1) * <a_0^n, W^b_1>  =  sum_k x[m][k] * w[n][k],   x in [0, 255], w = 2b - 1 in {-1, +1}
//
// The inputs arrive as packed bit planes (word 8*w + p of a row: bit p of elements 32w .. 32w + 31).  Eight plane
// words of 32 elements are an 8 x 8 bit transposition away from 32 bytes: 48 vector operations in registers
// (transpose_bits_8x8), after which ONE pass of v_mfma_i32_32x32x32_i8 replaces the eight of a product taken plane by
// plane (64 instead of 256 matrix cycles per 64 elements of K and 32 x 32 outputs).  Element 8j + s of a word ends
// up in byte j of register s; B's bits are widened into the same order, byte j of register s = 2 * bit (8j + s), by a
// shift and a mask.  The engine's bytes are signed, so plane 7 is inverted first and the bytes are x - 128:
//
//   sum_k x (2b - 1) = S + 256 * popcount(B_n) - sum_k x[m][k],      S = sum_k (x - 128) * 2b   (int32 accumulation)
//
// The row sums come from the staged bytes (v_dot4), the popcounts from B's words.  Everything is 32-bit integer
// arithmetic, exact modulo 2^32 and therefore exact for every K with 255*K < 2^31: single terms pass 2^31 from K = 2^23 on, so
// sums of them are formed in unsigned integers.
//
// Three organisations:
//   strips  128 x 512 tiles, WI = 4 x 2 blocks of 32 x 32 for each of 8 wavefronts, walked by one workgroup per compute unit
//           with all of K of its 512 columns in LDS (large fused products up to K = 1536).
//   tiles   32*WI*WR x 64*WC outputs per workgroup, WI x 2 blocks of 32 x 32 per wavefront: 128 x 512 with 8 wavefronts
//           (large fused products of longer K), 64 x 256 with 4, or 64 x 128 with 2 x 2 (few columns).  A's rows are transposed
//           once per workgroup while they are staged into LDS; B stays bits in LDS and is widened by the wavefront that
//           multiplies it (as bytes it would double the LDS traffic, which is what holds the plain int8 product at a third of
//           the matrix rate).  The wide, flat tile keeps both cheap: 4.4 vector operations per MFMA in all on 128 x 512 (a 2 x 2
//           arrangement of wavefronts on 128 x 256 needs 8).
//   split   32 x 32 outputs per workgroup, K split over its four wavefronts, operands straight from memory into
//           registers: for small grids, where the tiles above leave most compute units without work.
//
// What bounds them.  Tiles: a K-tile of 128 bits (64 MFMAs per SIMD, 2048 cycles) took 3400 - 3700 cycles.  A lane per column
// loads 16 bytes of every line of B per K-tile, and 512 lines do not stay in the first-level cache until the next one: 64 KB
// per K-tile through a path of 64 bytes a cycle.  Strips read B once, in whole lines: 2630 cycles, 41 per MFMA.  A loop of these
// MFMAs alone on random bytes takes 32.6 cycles and 15.0 ns with the bytes as first operand, 17.7 ns as second: the clock
// falls with the engine's power, 1.85 against 2.2 GHz.  Strips have them first; their accumulators are then columns by lane,
// and the output words are turned by a 32 x 32 bit transposition over the lanes (16 operations per pair of blocks).
// 10000 x 4096 x 784 fused: 85 us plane by plane on the fp4 engine, 40 - 43 in tiles, 31 - 35 in strips (K = 1536: 64 and 52);
// 100 x 4096 x 784: 5.2 us (22 us).
#include <type_traits>

#include "bit_transpose.h"
#include "bnn_internal.h"
#include "gemm_staging.h"
#include "strip_cut.h"

namespace bnn {
namespace planes {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Bytes of registers 4u .. 4u + 3: byte j of register s = 2 * bit (8j + s) of w.
template <int U>
__device__ inline v4i widen_bits(uint32_t w) {
    v4i f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int s = 4 * U + e;
        f[e] = int((s == 0 ? w << 1 : w >> (s - 1)) & 0x02020202u);
    }
    return f;
}

__device__ inline int add_bytes(uint32_t w, int sum) { return __builtin_amdgcn_sdot4(int(w), 0x01010101, sum, false); }

constexpr int kOffsetPerWord = 128 * 32;      // what the x - 128 of one word's 32 elements lacks to their x

// No result exceeds 255 * K in magnitude, so clamping a threshold to one past it changes no output bit; below this
// K the difference of a result and a clamped threshold stays inside int32.
constexpr int kSignMaxK = (1 << 30) / 256;

// ----------------------------------------------------------------------------
// tiles
// ----------------------------------------------------------------------------
constexpr int kWordsPerTile = 4;              // K-words per staged tile = 2 pairs = 4 MFMA steps

// WI x 2 blocks of 32 x 32 per wavefront, WR rows of WC wavefronts side by side: a tile of 32*WI*WR rows x 64*WC columns.
// TINY: rows of fewer than 4 words (K <= 96), which have no whole quad to load and one K-tile, or none.
template <int WI, int WR, int WC, bool FUSED, bool TINY>
__global__ __launch_bounds__(64 * WR * WC, 2) void bitplane_gemm_kernel(
    const uint32_t* __restrict__ Xp, int64_t ldx, const uint32_t* __restrict__ B, int64_t ldb,
    int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, TileMap tiles, BnSignArgs bn) {
    constexpr int T = 64 * WR * WC, BM = 32 * WI * WR, BN = 64 * WC;      // the first BN threads stage a column of B each
    constexpr int PLANE_A = BM + 1;                        // 16-byte slots; odd, so that the 4 words x 2 rows that 8 lanes
                                                           // store fall into eight different bank groups
    static_assert(T == BM * kWordsPerTile, "a thread stages one word (32 elements, 8 plane words) of A per tile");
    __shared__ uint4 lds_a[TINY ? 1 : 2][2 * kWordsPerTile * PLANE_A];    // [word][half of its 32 bytes][row]
    __shared__ uint32_t lds_b[TINY ? 1 : 2][kWordsPerTile * BN];          // [word][column]
    __shared__ int rowsum_s[BM];
    __shared__ __attribute__((aligned(16))) int colterm_s[BN]; // 256 * popcount, less the threshold when the sign decides
    __shared__ __attribute__((aligned(16))) int thr_s[FUSED ? BN : 4];

    int tile_m, tile_n;
    tile_of_block(blockIdx.x, tiles, tile_m, tile_n);
    const int row0 = tile_m * BM, col0 = tile_n * BN;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, wr = WR > 1 ? wave / WC : 0, wc = WR > 1 ? wave % WC : wave;
    const int fr = lane & 31, fh = lane >> 5;
    const int kw = (K + 31) >> 5;
    const uint32_t tmask = tail_mask(K);
    const int n_ktiles = (kw + kWordsPerTile - 1) / kWordsPerTile;
    const int n_full = (K >> 5) / kWordsPerTile;           // tiles of complete, unmasked words
    const int n_pairs = (kw + 1) >> 1;

    const int st_w = tid & 3, st_r = tid >> 2;
    const uint32_t* pa = Xp + int64_t(min(row0 + st_r, M - 1)) * ldx;
    const bool st_b = WR == 1 || tid < BN;
    const int b_col = min(col0 + (WR == 1 ? tid : tid & (BN - 1)), N - 1);             // rows past the matrix repeat its last one
    const uint32_t* pb = B + int64_t(b_col) * ldb;

    uint4 ra[2], rb;
    int cnt_a = 0, cnt_b = 0;

    // Loads carry no control flow (a branch around them makes the compiler wait for them where the branches meet, which
    // exposes the whole memory latency in every iteration): word indices are clamped into the row, and the last tile's
    // words that do not exist are sorted out when they are staged.  A row has at least one whole quad (the launcher).
    auto fetch_a = [&](int kt) {
        const int w = 8 * min(kWordsPerTile * kt + st_w, kw - 1);
        ra[0] = load_quad_any(pa + w);
        ra[1] = load_quad_any(pa + w + 4);
    };
    auto fetch_b = [&](int kt) {
        if (TINY) rb = make_uint4(pb[0], pb[min(1, kw - 1)], pb[min(2, kw - 1)], 0u);
        else rb = load_quad_any(pb + min(kWordsPerTile * kt, kw - kWordsPerTile));
    };
    // The last, partial tile: words past the row's end become zero, the last word's pad bits are masked.
    auto mask_tail = [&](int kt) {
        const int w = kWordsPerTile * kt + st_w;
        const uint32_t mask = w < kw - 1 ? ~0u : w == kw - 1 ? tmask : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) ra[h] = make_uint4(ra[h].x & mask, ra[h].y & mask, ra[h].z & mask, ra[h].w & mask);
        const int left = kw - kWordsPerTile * kt;
        if (TINY) {
            rb = mask_row_quad(rb, left, tmask);
            return;
        }
        // rb holds the row's last four words: word 0 of the tile is its word 4 - left.
        const uint32_t last = rb.w & tmask;
        rb = left == 1 ? make_uint4(last, 0u, 0u, 0u) : left == 2 ? make_uint4(rb.z, last, 0u, 0u)
           : left == 3 ? make_uint4(rb.y, rb.z, last, 0u) : make_uint4(rb.x, rb.y, rb.z, last);
    };
    uint32_t bytes[8];
    auto transpose_a = [&] {
        bytes[0] = ra[0].x; bytes[1] = ra[0].y; bytes[2] = ra[0].z; bytes[3] = ra[0].w;
        bytes[4] = ra[1].x; bytes[5] = ra[1].y; bytes[6] = ra[1].z; bytes[7] = ~ra[1].w;
        transpose_bits_8x8(bytes);
    };
    auto store_a = [&](int buf) {
#pragma unroll
        for (int s = 0; s < 8; ++s) cnt_a = add_bytes(bytes[s], cnt_a);
#pragma unroll
        for (int u = 0; u < 2; ++u)
            lds_a[buf][(2 * st_w + u) * PLANE_A + st_r] =
                make_uint4(bytes[4 * u], bytes[4 * u + 1], bytes[4 * u + 2], bytes[4 * u + 3]);
    };
    auto store_b = [&](int buf) {
        if (!st_b) return;
        cnt_b += __popc(rb.x) + __popc(rb.y) + __popc(rb.z) + __popc(rb.w);
        lds_b[buf][0 * BN + tid] = rb.x;
        lds_b[buf][1 * BN + tid] = rb.y;
        lds_b[buf][2 * BN + tid] = rb.z;
        lds_b[buf][3 * BN + tid] = rb.w;
    };

    v16i acc[WI][2];
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    // Step (t, u) of a tile: lane half fh takes word 2t + fh, half u of its 32 bytes.
    auto step = [&](int buf, int t, int u) {
        v4i fa[WI], fb[2];
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            const uint4 q = lds_a[buf][(2 * (2 * t + fh) + u) * PLANE_A + (wr * WI + i) * 32 + fr];
            fa[i] = v4i{int(q.x), int(q.y), int(q.z), int(q.w)};
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t w = lds_b[buf][(2 * t + fh) * BN + (wc * 2 + j) * 32 + fr];
            fb[j] = u == 0 ? widen_bits<0>(w) : widen_bits<1>(w);
        }
#pragma unroll
        for (int i = 0; i < WI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                // fused: operands swapped, so that a lane holds 16 columns of one output row
                acc[i][j] = FUSED ? __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
    };

    int thr = 0;
    const int lim = 255 * K + 1;
    if (FUSED) thr = max(-lim, min(lim, bn.thr[b_col]));
    auto fetch = [&](int kt) {
        fetch_a(kt);
        fetch_b(kt);
    };
    auto stage = [&](int kt, int buf) {
        if (kt >= n_full) mask_tail(kt);
        transpose_a();
        store_a(buf);
        store_b(buf);
    };
    if (!TINY || n_ktiles > 0) {
        fetch(0);
        stage(0, 0);
    }
    if (!TINY) fetch(1);
    __syncthreads();

    // Tile kt is multiplied while tile kt + 1 (in registers since the iteration before) is transposed and stored to the
    // other LDS buffer, and the loads of tile kt + 2 are issued as soon as their registers are free.
    int kt = 0;
    for (; kt + 1 < n_full; ++kt) {
        const int buf = kt & 1;
        // Slots the scheduler may not cross: it would sink the loads to the end of the iteration and wait for them at
        // the top of the next.
        step(buf, 0, 0);
        transpose_a();
        fetch_a(kt + 2);
        __builtin_amdgcn_sched_barrier(0);
        step(buf, 0, 1);
        store_a(buf ^ 1);
        store_b(buf ^ 1);
        fetch_b(kt + 2);
        __builtin_amdgcn_sched_barrier(0);
        step(buf, 1, 0);
        step(buf, 1, 1);
        __syncthreads();
    }
    // The last full tile and the partial one.
    for (; kt < n_ktiles; ++kt) {
        const int buf = kt & 1;
#pragma unroll
        for (int t = 0; t < kWordsPerTile / 2; ++t) {
            if (2 * kt + t >= n_pairs) break;
            step(buf, t, 0);
            step(buf, t, 1);
        }
        if (kt + 1 < n_ktiles) {
            stage(kt + 1, buf ^ 1);
            fetch(kt + 2);
        }
        __syncthreads();
    }

    {
        int c = cnt_a + kOffsetPerWord * n_ktiles;                          // words past the row's end included
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        if (st_w == 0) rowsum_s[st_r] = c;
    }
    const bool sign = FUSED && K <= kSignMaxK;
    if (st_b) {
        colterm_s[tid] = int(256u * uint32_t(cnt_b) - uint32_t(sign ? thr : 0));
        if (FUSED) thr_s[tid] = thr;
    }
    __syncthreads();

    if constexpr (!FUSED) {
        // Accumulator register v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32 of its 32 x 32 block.
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int nl = (wc * 2 + j) * 32 + fr, n = col0 + nl;
            const int ct = colterm_s[nl];
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int ml = (wr * WI + i) * 32 + 8 * (v / 4) + 4 * fh + (v % 4), m = row0 + ml;
                    if (m < M && n < N) store_result(&C[int64_t(m) * ldc + n], int(uint32_t(acc[i][j][v]) + uint32_t(ct) - uint32_t(rowsum_s[ml])));
                }
        }
    } else {
        // Register v of lane l: column 8*(v/4) + 4*(l/32) + v%4, row l%32.  The output bit is the complement of the
        // sign of result - threshold: an add of three, and an alignbit that shifts the sign into the lane's word.
        // A wavefront's words (2 per row) meet the others' in LDS, from where rows leave in 16-byte pieces.
        uint32_t* words_s = reinterpret_cast<uint32_t*>(lds_a[0]);          // [BM][BN / 32], free since the last barrier
        static_assert(BM * BN / 32 * 4 <= sizeof(lds_a), "the tile's output words fit the operand buffers");
        auto collect = [&](auto sign_tag) {
            constexpr bool SIGN = decltype(sign_tag)::value;
            uint32_t part[WI][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                int4 ct[4], th[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    ct[g] = *reinterpret_cast<const int4*>(&colterm_s[(wc * 2 + j) * 32 + 8 * g + 4 * fh]);
                    if (!SIGN) th[g] = *reinterpret_cast<const int4*>(&thr_s[(wc * 2 + j) * 32 + 8 * g + 4 * fh]);
                }
#pragma unroll
                for (int i = 0; i < WI; ++i) {
                    const int r = rowsum_s[(wr * WI + i) * 32 + fr];
                    uint32_t neg = 0u;
#pragma unroll
                    for (int g = 3; g >= 0; --g) {
#pragma unroll
                        for (int e = 3; e >= 0; --e) {
                            const int c = e == 0 ? ct[g].x : e == 1 ? ct[g].y : e == 2 ? ct[g].z : ct[g].w;
                            int d = int(uint32_t(acc[i][j][4 * g + e]) + uint32_t(c) - uint32_t(r));
                            if (!SIGN) {
                                const int t = e == 0 ? th[g].x : e == 1 ? th[g].y : e == 2 ? th[g].z : th[g].w;
                                d = d >= t ? 0 : -1;
                            }
                            neg = __builtin_amdgcn_alignbit(neg, uint32_t(d), 31);
                        }
                        if (g > 0) neg <<= 4;
                    }
                    part[i][j] = (~neg & 0x0F0F0F0Fu) << (4 * fh);
                }
            }
            // One v_permlane32_swap brings the two lane halves' nibbles together: lane half h holds the word of block h.
#pragma unroll
            for (int i = 0; i < WI; ++i) {
                const auto sw = __builtin_amdgcn_permlane32_swap(part[i][0], part[i][1], false, false);
                words_s[((wr * WI + i) * 32 + fr) * (BN / 32) + wc * 2 + fh] = sw[0] | sw[1];
            }
        };
        if (sign) collect(std::true_type{});
        else collect(std::false_type{});
        __syncthreads();
        constexpr int QUADS = BN / 128;                    // 16-byte pieces of a tile row
        const int64_t nw = (int64_t(N) + 31) >> 5;
        const int quad = tid % QUADS;
        const int64_t w0 = (int64_t(col0) >> 5) + 4 * quad;
        uint32_t flip[4], live[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int64_t left = N - 32 * (w0 + p);
            live[p] = left >= 32 ? ~0u : left <= 0 ? 0u : ((1u << left) - 1u);
            flip[p] = bn.flip_bits[w0 + p < nw ? w0 + p : nw - 1];
        }
#pragma unroll
        for (int r = tid / QUADS; r < BM; r += T / QUADS) {
            if (row0 + r >= M) break;
            const uint4 v = *reinterpret_cast<const uint4*>(&words_s[r * (BN / 32) + 4 * quad]);
            const uint32_t w[4] = {(v.x ^ flip[0]) & live[0], (v.y ^ flip[1]) & live[1], (v.z ^ flip[2]) & live[2],
                                   (v.w ^ flip[3]) & live[3]};
            uint32_t* o = bn.out + int64_t(row0 + r) * bn.ld_out + w0;
            if (w0 + 4 <= nw) {
                store_quad_any(o, make_uint4(w[0], w[1], w[2], w[3]));
            } else {
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    if (w0 + p < nw) o[p] = w[p];
            }
        }
    }
}

// ----------------------------------------------------------------------------
// strips: 128 x 512 tiles of the large fused products, walked by one workgroup per compute unit
//
// The N / 512 column tiles times equal strips of rows are at most one workgroup per compute unit (10000 x 4096: 2.5 tiles
// each, where whole tiles need three rounds).  A K-tile is four steps of 8 MFMAs; the operands of a step are read and widened
// under the step before, the K-tile two further on is transposed under steps 0 and 1 and stored under step 2, into the third
// of three buffers, with one barrier in between; the stream of K-tiles runs on across the strip's tiles.  Nothing in a K-tile
// branches, so that the compiler can keep to the order given (BNN_PLANES_SCHEDULE): partial words are zero bytes of A, whatever
// B holds there.
// ----------------------------------------------------------------------------
constexpr int kStripT = 512, kStripBM = 128, kStripBN = 512, kStripBuffers = 3;
constexpr int kStripPitchB = kStripBN + 2;     // words per plane of B: 8 lanes' quads of 8 columns fall into 64 different banks
constexpr int kStripWords = 48;                // K-words of B beside three buffers of A: 96 of 160 KB

struct StripCut {
    FastDiv by_tiles_n;
    int tiles_n, per_die;      // column tiles; workgroups / 8
    int rows;                  // rows per strip, a multiple of 32
};

// After every product: one LDS read with READ, VALU vector operations, one LDS write with WRITE, one load with LOAD.
#define BNN_PLANES_SCHEDULE(MFMAS, READ, VALU, WRITE, LOAD)                           \
    do {                                                                              \
        _Pragma("unroll") for (int g_ = 0; g_ < (MFMAS); ++g_) {                      \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        \
            if (READ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);              \
            if (LOAD) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);              \
            __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);                     \
            if (WRITE) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);             \
        }                                                                             \
        __builtin_amdgcn_sched_barrier(0);                                            \
    } while (0)

__global__ __launch_bounds__(kStripT, 2) void bitplane_gemm_strip_kernel(
    const uint32_t* __restrict__ Xp, int64_t ldx, const uint32_t* __restrict__ B, int64_t ldb, int M, int N, int K,
    StripCut cut, BnSignArgs bn) {
    constexpr int T = kStripT, BM = kStripBM, BN = kStripBN, WI = 4;
    constexpr int PLANE_A = BM + 1;                        // 16-byte slots, odd (see above)
    constexpr int A_BUF = 2 * kWordsPerTile * PLANE_A;
    constexpr int PITCH_B = kStripPitchB;
    static_assert(T == BN && T == BM * kWordsPerTile, "a thread stages a column of B and a word of A per K-tile");
    __shared__ uint4 lds_a[kStripBuffers * A_BUF];         // [word][half of its 32 bytes][row]
    extern __shared__ uint32_t lds_b[];                    // [word][column]: all of K, for the workgroup's life
    __shared__ __attribute__((aligned(16))) int rowsum_s[2][BM];           // minus the sums of the rows' bytes
    __shared__ __attribute__((aligned(16))) int colterm_s[BN];
    static_assert(32 * kStripWords <= kSignMaxK, "the difference of a result and a clamped threshold fits int32");

    int logical = int(blockIdx.x);
    if (logical < kDies * cut.per_die) logical = (logical % kDies) * cut.per_die + logical / kDies;
    const int group = cut.by_tiles_n(logical), col0 = (logical - group * cut.tiles_n) * BN;
    const StripRows strip = strip_rows(group, cut.rows, M);
    const int row_begin = strip.begin, row_end = strip.end;

    const int tid = threadIdx.x, lane = tid & 63, wc = tid >> 6;
    const int fr = lane & 31, fh = lane >> 5;
    const int kw = (K + 31) >> 5;
    const uint32_t tmask = tail_mask(K);
    const int n_ktiles = (kw + kWordsPerTile - 1) / kWordsPerTile;         // at least 3 (the launcher)
    const bool short_end = kw - kWordsPerTile * (n_ktiles - 1) <= 2;       // the last K-tile has one pair of words

    const int st_w = tid & 3, st_r = tid >> 2;
    auto row_at = [&](int row0) __attribute__((always_inline)) { return Xp + int64_t(min(row0 + st_r, row_end - 1)) * ldx; };

    uint4 ra[2];
    uint32_t bytes[8];
    int cnt_a = 0;
    // K-tile kt of the row at p / of B.  Nothing here carries control flow (a branch around loads makes the compiler wait for
    // them where it ends, and the code between two branches is scheduled by itself): word indices are clamped into the row.
    auto fetch_a = [&](const uint32_t* p, int kt) __attribute__((always_inline)) {
        const int w = 8 * min(kWordsPerTile * kt + st_w, kw - 1);
        ra[0] = load_quad_any(p + w);
        ra[1] = load_quad_any(p + w + 4);
    };
    // Bytes of K-tile kt: x - 128, and 0 past the row's end, whatever B has there.
    auto take = [&](int kt) __attribute__((always_inline)) {
        const int w = kWordsPerTile * kt + st_w;
        const uint32_t mask = w < kw - 1 ? ~0u : w == kw - 1 ? tmask : 0u;
        const uint32_t p[8] = {ra[0].x, ra[0].y, ra[0].z, ra[0].w, ra[1].x, ra[1].y, ra[1].z, ~ra[1].w};
#pragma unroll
        for (int s = 0; s < 8; ++s) bytes[s] = p[s] & mask;
    };
    auto store_a = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            lds_a[buf * A_BUF + (2 * st_w + u) * PLANE_A + st_r] =
                make_uint4(bytes[4 * u], bytes[4 * u + 1], bytes[4 * u + 2], bytes[4 * u + 3]);
    };
    // Row sums so far of the K-tile's rows (complete with the last one, two K-tiles before they are read).
    auto sum_rows = [&](int kt, int parity) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 8; ++s) cnt_a = add_bytes(bytes[s], cnt_a);
        int c = cnt_a;
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        rowsum_s[parity][st_r] = -c;
        cnt_a = kt == n_ktiles - 1 ? 0 : cnt_a;
    };

    // Start: K-tiles 0 and 1 of the first row tile, and all of B, into LDS; K-tile 2 in flight.  8 lanes take a column's 128
    // bytes at a time (a lane per column fetched every line of B once per K-tile: 512 lines do not stay in the first-level
    // cache, and 64 KB per K-tile through it were what the loop waited for).
    const uint32_t* pa = row_at(row_begin);
    fetch_a(pa, 0);
    const uint4 first_a[2] = {ra[0], ra[1]};
    fetch_a(pa, 1);
    const int lim = 255 * K + 1;
    constexpr int COLS = T / 8;                            // columns per pass
    const int bq = tid & 7, bc = tid >> 3;
    const int last_quad = kw - kWordsPerTile;              // of a row: the quad at its end (K > 96)
    constexpr int PASSES = BN / COLS;
    int th[PASSES], pop[PASSES] = {};
#pragma unroll
    for (int p = 0; p < PASSES; ++p) th[p] = bn.thr[min(col0 + p * COLS + bc, N - 1)];
    for (int q = bq; q - bq < (kw + 3) >> 2; q += 8) {     // 32 words of every column at a time
        uint4 v[PASSES];
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            v[p] = load_quad_any(B + int64_t(min(col0 + p * COLS + bc, N - 1)) * ldb + min(4 * q, last_quad));
        if (4 * q < kw) {
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                const uint4 w = place_row_quad(v[p], q, kw, tmask);
                pop[p] += __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
                uint32_t* to = lds_b + 4 * q * PITCH_B + p * COLS + bc;
                to[0] = w.x;
                to[PITCH_B] = w.y;
                to[2 * PITCH_B] = w.z;
                to[3 * PITCH_B] = w.w;
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int c = p * COLS + bc;
        int sum = pop[p];
        sum += __builtin_amdgcn_update_dpp(0, sum, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        sum += __builtin_amdgcn_update_dpp(0, sum, 0x141, 0xF, 0xF, true);      // the other four of eight
        const int thr = max(-lim, min(lim, th[p]));
        if (bq == 0) {
            colterm_s[c] = int(256u * uint32_t(sum) - uint32_t(thr));
        }
    }
    {
        const uint4 second_a[2] = {ra[0], ra[1]};
        ra[0] = first_a[0]; ra[1] = first_a[1];
        take(0);
        transpose_bits_8x8(bytes);
        store_a(0);
        sum_rows(0, 0);
        ra[0] = second_a[0]; ra[1] = second_a[1];
        take(1);
        transpose_bits_8x8(bytes);
        store_a(1);
        sum_rows(1, 0);
    }
    fetch_a(pa, 2);
    __syncthreads();

    // This lane's output word: column block 2 * wc + fh.
    const int64_t nw = (int64_t(N) + 31) >> 5, word = (int64_t(col0) >> 5) + 2 * wc + fh;
    const int64_t cols_left = N - 32 * word;
    const uint32_t live = cols_left >= 32 ? ~0u : cols_left <= 0 ? 0u : ((1u << cols_left) - 1u);
    const uint32_t flip = bn.flip_bits[word < nw ? word : nw - 1] & live;

    v16i acc[WI][2];
    int buf = 0;                                           // LDS buffer of the K-tile that is multiplied
    // Step s = 2t + u of a K-tile: lane half fh takes word 2t + fh, half u of its 32 bytes.
    v4i fa[WI], ga[WI], fb[2], gb[2];
    uint32_t wb[2];
    const uint4* rd_a = lds_a + 2 * fh * PLANE_A + fr;
    const uint32_t* rd_b = lds_b + fh * PITCH_B + wc * 64 + fr;
    auto run = [&](auto nb_tag, int row0, int parity) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_tag)::value;
        auto read_a = [&](int b, int s, v4i (&f)[WI]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const uint4 q = rd_a[b * A_BUF + (4 * (s >> 1) + (s & 1)) * PLANE_A + i * 32];
                f[i] = v4i{int(q.x), int(q.y), int(q.z), int(q.w)};
            }
        };
        auto read_b = [&](int kt, int t) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) wb[j] = rd_b[(kWordsPerTile * kt + 2 * t) * PITCH_B + j * 32];
        };
        auto multiply = [&](const v4i (&a)[WI], const v4i (&b)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
        };
        const uint32_t* pa_next = row_at(min(row0 + BM, row_end - 1));     // past the strip: rows that nothing reads
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
        // The operands of a step are read and widened during the step before.
        read_a(buf, 0, fa);
        read_b(0, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j] = widen_bits<0>(wb[j]);
        constexpr int P = 2 * NB;                          // products per step
        auto k_tile = [&](int kt, auto pair_tag) __attribute__((always_inline)) {
            constexpr bool ONE_PAIR = decltype(pair_tag)::value;
            const int buf1 = buf == kStripBuffers - 1 ? 0 : buf + 1, buf2 = buf1 == kStripBuffers - 1 ? 0 : buf1 + 1;
            // K-tile that is staged (in registers; its row tile's parity), and the one that is loaded.
            const bool over = kt + 2 >= n_ktiles, over3 = kt + 3 >= n_ktiles;
            const int s_kt = over ? kt + 2 - n_ktiles : kt + 2, f_kt = over3 ? kt + 3 - n_ktiles : kt + 3;
            const uint32_t* f_row = over3 ? pa_next : pa;
            __builtin_amdgcn_sched_barrier(0);
            // step 0
            read_a(buf, 1, ga);
#pragma unroll
            for (int j = 0; j < 2; ++j) gb[j] = widen_bits<1>(wb[j]);
            take(s_kt);
            exchange_fields<4, 0x0F0F0F0Fu>(bytes);
#pragma unroll
            for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(bytes[s]));
            multiply(fa, fb);
            BNN_PLANES_SCHEDULE(P, 1, (16 + 30 + P - 1) / P, 0, 0);
            // step 1
            if constexpr (!ONE_PAIR) {
                read_a(buf, 2, fa);
                read_b(kt, 1);
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[j] = widen_bits<0>(wb[j]);
            }
            fetch_a(f_row, f_kt);
            exchange_fields<2, 0x33333333u>(bytes);
            exchange_fields<1, 0x55555555u>(bytes);
#pragma unroll
            for (int s = 0; s < 8; ++s) asm volatile("" : "+v"(bytes[s]));
            if constexpr (!ONE_PAIR) {
                multiply(ga, gb);
                BNN_PLANES_SCHEDULE(P, 1, (16 + 36 + P - 1) / P, 0, 1);
            }
            // Every wavefront has left the K-tile before, whose buffer is written now, and has written the next one's.
            __syncthreads();
            // step 2
            if constexpr (!ONE_PAIR) {
                read_a(buf, 3, ga);
#pragma unroll
                for (int j = 0; j < 2; ++j) gb[j] = widen_bits<1>(wb[j]);
            }
            store_a(buf2);
            sum_rows(s_kt, over ? parity ^ 1 : parity);
            if constexpr (!ONE_PAIR) {
                multiply(fa, fb);
                BNN_PLANES_SCHEDULE(P, 1, (16 + 14 + P - 1) / P, 1, 0);
            }
            // step 3, under which the next K-tile's (or row tile's) first operands are read
            read_a(buf1, 0, fa);
            read_b(kt + 1 == n_ktiles ? 0 : kt + 1, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) fb[j] = widen_bits<0>(wb[j]);
            multiply(ga, gb);
            BNN_PLANES_SCHEDULE(P, 1, (16 + 4 + P - 1) / P, 0, 0);
            buf = buf1;
        };
        const int whole = n_ktiles - (short_end ? 1 : 0);
        for (int kt = 0; kt < whole; ++kt) k_tile(kt, std::false_type{});
        if (short_end) k_tile(n_ktiles - 1, std::true_type{});
        pa = pa_next;

        // Register v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32.  The output bit is the complement of the sign of
        // result - threshold: an add of three, and an alignbit that shifts the sign into the lane's word of rows.
        int ct[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
            ct[j] = int(uint32_t(colterm_s[(wc * 2 + j) * 32 + fr]) - 128u * uint32_t(K));      // (sum x = the bytes' sum + 128 K)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            int4 rs[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) rs[g] = *reinterpret_cast<const int4*>(&rowsum_s[parity][i * 32 + 8 * g + 4 * fh]);
            uint32_t part[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                uint32_t neg = 0u;
#pragma unroll
                for (int g = 3; g >= 0; --g) {
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        const int r = e == 0 ? rs[g].x : e == 1 ? rs[g].y : e == 2 ? rs[g].z : rs[g].w;
                        const uint32_t d = uint32_t(acc[i][j][4 * g + e]) + uint32_t(ct[j]) + uint32_t(r);
                        neg = __builtin_amdgcn_alignbit(neg, d, 31);
                    }
                    if (g > 0) neg <<= 4;
                }
                part[j] = (~neg & 0x0F0F0F0Fu) << (4 * fh);
            }
            // One v_permlane32_swap brings the two lane halves' nibbles together: lane l holds the rows of column l % 32
            // of block l / 32, and after the transposition the columns of row l % 32.
            const auto sw = __builtin_amdgcn_permlane32_swap(part[0], part[1], false, false);
            const uint32_t bits = transpose_bits_32_lanes(sw[0] | sw[1]);
            const int m = row0 + i * 32 + fr;
            if (m < row_end && word < nw) bn.out[int64_t(m) * bn.ld_out + word] = (bits & live) ^ flip;
        }
    };

    int parity = 0;
    for (int row0 = row_begin; row0 < row_end; row0 += BM, parity ^= 1) {
        const int blocks = (min(BM, row_end - row0) + 31) / 32;
        if (blocks == 4) run(std::integral_constant<int, 4>{}, row0, parity);
        else if (blocks == 3) run(std::integral_constant<int, 3>{}, row0, parity);
        else if (blocks == 2) run(std::integral_constant<int, 2>{}, row0, parity);
        else run(std::integral_constant<int, 1>{}, row0, parity);
    }
}

// ----------------------------------------------------------------------------
// split: 32 x 32 outputs, K split over the wavefronts
// ----------------------------------------------------------------------------
constexpr int kSplitWaves = 4;
constexpr int kSplitBatch = 2;                // word pairs a wavefront loads at a time (two such batches in flight)

template <bool FUSED>
__global__ __launch_bounds__(256) void bitplane_gemm_split_kernel(
    const uint32_t* __restrict__ Xp, int64_t ldx, const uint32_t* __restrict__ B, int64_t ldb,
    int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, TileMap tiles, BnSignArgs bn) {
    __shared__ uint4 part[kSplitWaves][4][kWave];          // [wavefront][accumulator registers 4g .. 4g + 3][lane]
    __shared__ __attribute__((aligned(16))) uint32_t sum_part[kSplitWaves][kWave];   // [0, 32) row sums of A, [32, 64) 256 * popcounts of B
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fr = lane & 31, fh = lane >> 5;
    int tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const int row0 = tm * 32, col0 = tn * 32;
    const int kw = (K + 31) >> 5;
    const uint32_t tmask = tail_mask(K);
    const int n_pairs = (kw + 1) >> 1;
    const uint32_t* a_row = Xp + int64_t(min(row0 + fr, M - 1)) * ldx;
    const uint32_t* b_row = B + int64_t(min(col0 + fr, N - 1)) * ldb;
    const int col = col0 + fr;
    int thr = 0;
    uint32_t flip_word = 0u;
    if constexpr (FUSED) {
        thr = bn.thr[min(col, N - 1)];
        flip_word = bn.flip_bits[min(col, N - 1) >> 5];
    }

    v16i acc[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0;
    int ca = 0;
    uint32_t cb = 0u;

    // Of a group of 8 pairs wavefront w takes pairs w and w + 4, lane half fh word fh of each.  Word indices are clamped
    // into the row and what was loaded is masked away where the word does not exist.
    struct Batch {
        uint4 a[kSplitBatch][2];
        uint32_t b[kSplitBatch];
    };
    auto load = [&](int pair0, Batch& q) {
#pragma unroll
        for (int t = 0; t < kSplitBatch; ++t) {
            const int w = min(2 * (pair0 + kSplitWaves * t) + fh, kw - 1);
            q.a[t][0] = load_quad_any(a_row + 8 * w);
            q.a[t][1] = load_quad_any(a_row + 8 * w + 4);
            q.b[t] = b_row[w];
        }
    };
    Batch cur, next;
    if (n_pairs > 0) load(wave, cur);
    for (int p0 = wave; p0 < n_pairs; p0 += kSplitWaves * kSplitBatch) {
        const int p1 = p0 + kSplitWaves * kSplitBatch;
        if (p1 < n_pairs) load(p1, next);
#pragma unroll
        for (int t = 0; t < kSplitBatch; ++t) {
            const int w = 2 * (p0 + kSplitWaves * t) + fh;
            const uint32_t mask = w < kw - 1 ? ~0u : w == kw - 1 ? tmask : 0u;
            const uint32_t b = cur.b[t] & mask;
            uint32_t p[8] = {cur.a[t][0].x & mask, cur.a[t][0].y & mask, cur.a[t][0].z & mask, cur.a[t][0].w & mask,
                             cur.a[t][1].x & mask, cur.a[t][1].y & mask, cur.a[t][1].z & mask, ~(cur.a[t][1].w & mask)};
            transpose_bits_8x8(p);
#pragma unroll
            for (int s = 0; s < 8; ++s) ca = add_bytes(p[s], ca);
            ca += kOffsetPerWord;
            cb += 256u * uint32_t(__popc(b));
            acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(v4i{int(p[0]), int(p[1]), int(p[2]), int(p[3])}, widen_bits<0>(b),
                                                          acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(v4i{int(p[4]), int(p[5]), int(p[6]), int(p[7])}, widen_bits<1>(b),
                                                          acc[1], 0, 0, 0);
        }
        if (p1 < n_pairs) cur = next;
    }

    // Lanes 0-31 end up with the sum of A's row fr over both lane halves, lanes 32-63 with that of B's row fr.
    const auto sw = __builtin_amdgcn_permlane32_swap(uint32_t(ca), cb, false, false);
    sum_part[wave][lane] = sw[0] + sw[1];
#pragma unroll
    for (int g = 0; g < 4; ++g)
        part[wave][g][lane] = make_uint4(uint32_t(acc[0][4 * g]) + uint32_t(acc[1][4 * g]),
                                         uint32_t(acc[0][4 * g + 1]) + uint32_t(acc[1][4 * g + 1]),
                                         uint32_t(acc[0][4 * g + 2]) + uint32_t(acc[1][4 * g + 2]),
                                         uint32_t(acc[0][4 * g + 3]) + uint32_t(acc[1][4 * g + 3]));
    __syncthreads();

    // Accumulator register v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32.  This wavefront finishes registers
    // 4*wave .. 4*wave + 3.
    uint32_t sum[4] = {0u, 0u, 0u, 0u}, pb = 0u;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
        const uint4 s4 = part[w][wave][lane];
        const uint4 ra = *reinterpret_cast<const uint4*>(&sum_part[w][8 * wave + 4 * fh]);
        sum[0] += s4.x - ra.x;
        sum[1] += s4.y - ra.y;
        sum[2] += s4.z - ra.z;
        sum[3] += s4.w - ra.w;
        pb += sum_part[w][32 + fr];
    }
    int dot[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) dot[e] = int(sum[e] + pb);
    if constexpr (!FUSED) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = row0 + 8 * wave + 4 * fh + e;
            if (row < M && col < N) C[int64_t(row) * ldc + col] = dot[e];
        }
    } else {
        const bool valid = col < N;
        const bool flip = (flip_word >> (col & 31)) & 1u;
        // Ballot e: low half = the word of row 8*wave + e, high half = that of row 8*wave + 4 + e.
        uint32_t word = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint64_t mask = __ballot(valid && ((dot[e] >= thr) != flip));
            if ((lane & 3) == e) word = (lane & 4) ? uint32_t(mask >> 32) : uint32_t(mask);
        }
        const int row = row0 + 8 * wave + lane;
        if (lane < 8 && row < M) bn.out[int64_t(row) * bn.ld_out + tn] = word;
    }
}

}  // namespace planes

template <int WI, int WR, int WC, bool FUSED, bool TINY>
static int launch_tiles(const uint32_t* Xp, int64_t ldx, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                        int64_t M, int64_t N, int64_t K, BnSignArgs bn, hipStream_t s) {
    constexpr int BM = 32 * WI * WR, T = 64 * WR * WC;
    const int64_t tiles_n = ceil_div(N, 64 * WC);
    const int64_t rows = max_blocks(T) / tiles_n * BM;      // of one launch: all of them, short of 2^23 tiles
    for (int64_t m0 = 0; m0 < M; m0 += rows) {
        const int64_t m = M - m0 < rows ? M - m0 : rows, tiles_m = ceil_div(m, BM);
        hipLaunchKernelGGL((planes::bitplane_gemm_kernel<WI, WR, WC, FUSED, TINY>), dim3(unsigned(tiles_m * tiles_n)), dim3(T), 0, s,
                           Xp + m0 * ldx, ldx, B, ldb, C + m0 * ldc, ldc, int(m), int(N), int(K), tile_map(tiles_m, tiles_n), bn);
        const int st = check_launch();
        if (st != BNN_OK) return st;
        bn.out += rows * bn.ld_out;
    }
    return BNN_OK;
}

// The choice, from sweeps of 70 shapes with M = 7 .. 1000000, N = 10 .. 4096, K = 9 .. 3072 (fused, us; those of the first
// and third item with K >= 97 with the packing of the planes):
//  - split up to 1024 of its 32 x 32 tiles: 100 x 4096 x 784 7.8 vs 10.2 on 64 x 256 tiles, 233 x 4096 x 784 (1024 tiles)
//    10.1 vs 10.4, 300 x 512 x 3072 11.4 vs 21.5; but 363 x 4096 x 784 12.5 vs 10.5, 501 x 2954 x 3072 33.0 vs 22.8.  Few
//    words in K leave most of its wavefronts idle: 1000 x 4096 x 64 (4096 tiles) 10.1 vs 3.9, 10000 x 4096 x 64 70 vs 13.7.
//  - 64 x 128 up to 128 columns, which wider tiles would multiply as 256 or 512: 262144 x 128 x 27 12.6 vs 19.7 on 64 x 256
//    and 35.6 on 128 x 512, 262144 x 128 x 147 17.7 vs 24.5 and 49.3, 1000000 x 32 x 75 43.6 vs 75 and 151.  With 129 columns
//    and more the 64 x 256 tile is level or better (100000 x 300 x 200 20.8 vs 21.3, 40000 x 640 x 784 36.7 vs 33.5).
//  - strips with at most a quarter of columns that do not exist, strips of more than one tile, at least three K-tiles (the
//    stream runs three ahead) and K that fits LDS beside A: 10000 x 4096 x 784 43.0 on 128 x 512 tiles and 35.1, x 1536 65.6 and
//    53.8, 16384 x 4096 x 784 57.1 and 49.2, 6000 x 4096 x 784 26.3 and 23.9, 5000 x 4096 x 784 (160 rows) 23.3 and 21.9, 8192 x 4096
//    x 300 17.2 and 16.4; but of one tile, 4000 x 4096 x 784 (128 rows, one round of tiles) 15.4 and 16.3.  They also have to
//    keep the chip at work: a strip's last tile costs as much staging as a whole one, which short K-loops do not cover, and
//    256 / (N / 512) strips are rounded down.  Outputs there are against whole tiles on 256 units, least share taken: 70 % up to
//    K = 384 (12300 x 1226 x 440 11.6 and 14.5, 5190 x 3247 x 258 11.4 and 12.5, strips of 160 rows each; 16412 x 3697 x 309, 72 %,
//    37.8 and 29.9), 63 % up to K = 512 (2539 x 8192 x 496, 62 %, 14.7 and 15.3), 50 % above (9101 x 1701 x 743, 46 %, 16.9 and 18.8;
//    9633 x 1920 x 788, 55 %, 21.7 and 20.0; 1500 x 66048 x 784, 49 %, 93.6 and 122).
//  - 128 x 512 where its tiles fill whole rounds of the 256 compute units to 4/5 with at most a quarter of columns that do
//    not exist, and K > 256 or one round: 4000 x 4096 x 784 21.5 vs 24.3 on 64 x 256; but 262144 x 256 x 147 (half of the columns)
//    50.4 vs 25.2, 10000 x 4096 x 129 18.9 vs 15.9, 4096 x 4096 x 160 (one round) 7.1 vs 7.6.  Its int32 form does not fit the
//    registers.
//  - 64 x 256 (four workgroups per compute unit) otherwise: 2000 x 4096 x 784 15.4 vs 18.0, 3280 x 1152 x 2394 30 vs 39.
constexpr int64_t kSplitMaxTiles = 1024;
constexpr int64_t kComputeUnits = 256;

template <bool FUSED, bool TINY>
static int launch_planes(const uint32_t* Xp, int64_t ldx, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                         int64_t M, int64_t N, int64_t K, const BnSignArgs& bn, void* stream) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (ceil_div(M, 256) * ceil_div(N, 128) > kMaxDim) return BNN_ERR_UNSUPPORTED;
    const int64_t small_m = ceil_div(M, 32), small_n = ceil_div(N, 32);
    if (small_m * small_n <= kSplitMaxTiles) {
        hipLaunchKernelGGL(planes::bitplane_gemm_split_kernel<FUSED>, dim3(unsigned(small_m * small_n)), dim3(256), 0, s, Xp,
                           ldx, B, ldb, C, ldc, int(M), int(N), int(K), tile_map(small_m, small_n), bn);
        return check_launch();
    }
    if (N <= 128) return launch_tiles<1, 2, 2, FUSED, TINY>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, s);
    if constexpr (FUSED && !TINY) {
        const int64_t tiles_n = ceil_div(N, planes::kStripBN);
        const bool wide = 4 * N >= 3 * planes::kStripBN * tiles_n;           // at most a quarter of columns that do not exist
        if (wide && tiles_n <= kStripUnits && K > 256 && K <= 32 * planes::kStripWords) {
            const StripPlan plan = strip_plan(M, tiles_n);
            const int64_t rows = plan.rows, groups = plan.groups;
            // Whole tiles; the share of the chip that works on columns that exist.
            const int64_t cost = ceil_div(rows, planes::kStripBM) * planes::kStripBM * planes::kStripBN;
            if (rows > planes::kStripBM && strips_fill(M, N, cost, K <= 384 ? 70 : K <= 512 ? 63 : 50)) {
                const planes::StripCut cut{fast_div(tiles_n), int(tiles_n), int(groups * tiles_n / kDies), int(rows)};
                hipLaunchKernelGGL(planes::bitplane_gemm_strip_kernel, dim3(unsigned(groups * tiles_n)), dim3(planes::kStripT),
                                   size_t(4) * planes::kStripPitchB * (4 * ceil_div(K, 128)), s, Xp, ldx, B, ldb, int(M), int(N),
                                   int(K), cut, bn);
                return check_launch();
            }
        }
        const int64_t tiles = ceil_div(M, 128) * tiles_n, rounds = ceil_div(tiles, kComputeUnits);
        if ((K > 256 || rounds == 1) && 5 * tiles >= 4 * rounds * kComputeUnits && wide)
            return launch_tiles<4, 1, 8, true, false>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, s);
    }
    return launch_tiles<2, 1, 4, FUSED, TINY>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, s);
}

// The callers have validated the arguments.  fused: bn holds thresholds, flip words and the output.
int launch_bitplane_gemm(const uint32_t* Xp, int64_t ldx, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                         int64_t M, int64_t N, int64_t K, bool fused, const BnSignArgs& bn, void* stream) {
    if (K <= 96)
        return fused ? launch_planes<true, true>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, stream)
                     : launch_planes<false, true>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, stream);
    return fused ? launch_planes<true, false>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, stream)
                 : launch_planes<false, false>(Xp, ldx, B, ldb, C, ldc, M, N, K, bn, stream);
}

}  // namespace bnn

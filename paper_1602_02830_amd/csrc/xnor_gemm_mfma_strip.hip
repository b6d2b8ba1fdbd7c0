// Fused binary layer (XnorDotProduct -> Sign(BatchNorm), bits in, bits out) of short rows, 576 < K <= 1024, on grids that fill
// the chip: the first layer of an MLP over a whole test set.
//
// The organisation of conv_strip.hip for plain rows: one workgroup of eight wavefronts per compute unit, 128 columns of B resident
// in LDS, an equal strip of A's rows walked in tiles of 512 whose whole K sits in LDS (two buffers); the next tile is
// loaded and stored under the products of the current one, a row's 128 bytes by 8 lanes; accumulators start as the folded
// threshold; the operands of a step are widened between the products of the step before.
//
// What bounds it is the issue of vector operations, two wavefronts to a SIMD: a wavefront's 8 x 13 products (K = 784) bring 510 of them
// for widening, so the staging of the next tile's rows beside them is kept to 20 per 64 rows: addresses are 32-bit offsets that a pass
// steps, a row's last quad is masked where it was loaded instead of shifted into place, and planes for all eight quads are written
// whatever K is.  (With 64-bit addresses, shifts and stores under a mask, 65, a tile took 14000 cycles for 6700 of products.)  us, before
// that and now: 10000 x 4096 x 784 18.4 and 15.9, 16384 x 4096 x 784 26.4 and 22.9, 3000 x 3000 x 784 6.7 and 6.2, 16000 x 1000 x 800
// 8.3 and 7.7; on the 128 x 128 tiles 20.6, 28.4, 7.9 and 11.2.  Rows too far apart for 32 bits have a kernel with 64-bit offsets: 2000 x 8000 x
// 784 with rows 360000 words apart 8.0, on the tiles 10.6, with 340000 7.8.
#include <type_traits>

#include "bnn_internal.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"
#include "strip_cut.h"

namespace bnn {
namespace row_strip {

constexpr int T = 512, BN = 128, PLANE_B = BN + 2;     // 8-byte slots per plane of B
constexpr int WAVE_ROWS = 4, NB_MAX = 4, BM = 32 * WAVE_ROWS * NB_MAX;
constexpr int PLANE_A = BM + 4;                        // 8-byte slots per plane of A: the quads that 8 lanes store of 8 rows fall into different banks
constexpr int MAX_QUADS = 8;                           // K <= 1024: a row is one line
constexpr int PASS_ROWS = T / MAX_QUADS, PASSES = BM / PASS_ROWS;      // 64 rows per pass, 8 passes
constexpr int TILE_A = 2 * MAX_QUADS * PLANE_A;
constexpr int PARTS = 4;                               // of a tile's K loop, two passes of the next tile in flight under each

struct Cut {
    FastDiv by_tiles_n;
    int tiles_n, per_die;      // column tiles; workgroups / 8
    int rows;                  // rows per strip, a multiple of 32
};

// Offset: of bytes, from a strip's first row and from a column tile's.  32 bits but for rows so far apart that they do not hold it.
template <typename Offset>
__global__ __launch_bounds__(T, 2) void xnor_gemm_mfma_strip_kernel(const uint32_t* __restrict__ A, int64_t lda,
                                                                    const uint32_t* __restrict__ B, int64_t ldb, int M, int N,
                                                                    int K, BnSignArgs bn, Cut cut) {
    constexpr int WN = 2;
    extern __shared__ __attribute__((aligned(16))) uint2 dyn[];            // B [MAX_QUADS][2][PLANE_B], then one or two buffers of A [MAX_QUADS][2][PLANE_A]
    __shared__ float colfix_s[BN];
    __shared__ uint32_t flip_s[BN / 32];
    __shared__ float pop_s[2][BM];                     // minus popcount / 2 of a tile's rows
    const int kw = (K + 31) >> 5, kq = (kw + 3) >> 2;
    const uint32_t tmask = tail_mask(K);
    uint2* tiles_a = dyn + 2 * MAX_QUADS * PLANE_B;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fh = lane >> 5;

    int logical = int(blockIdx.x);
    if (logical < kDies * cut.per_die) logical = (logical % kDies) * cut.per_die + logical / kDies;
    const int group = cut.by_tiles_n(logical), col0 = (logical - group * cut.tiles_n) * BN;
    const StripRows strip = strip_rows(group, cut.rows, M);
    const int row_begin = strip.begin, row_end = strip.end;

    // Lane q of 8 takes quad q of a row.  The quad at a row's end that is not whole is the row's last four words with those that
    // belong to the quad before zeroed, not shifted: the same for A and B, whose K may run in any order.  Past it zeros.
    const int st_q = tid & 7, st_r = tid >> 3;
    const int words_left = kw - 4 * st_q;
    uint32_t mask[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) mask[p] = words_left <= 0 || p < 4 - words_left ? 0u : p == 3 && words_left <= 4 ? tmask : ~0u;
    const Offset quad_at = 4u * uint32_t(min(4 * st_q, kw - 4));
    // 16 bytes at `offset` from a uniform address.
    auto load_at = [&](const uint32_t* P, Offset offset) __attribute__((always_inline)) {
        asm volatile("" : "+v"(offset));               // or 32 bits become a 64-bit address per lane
        return load_quad_any(reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(P) + offset));
    };
    // Words to LDS, set bits of the row in every one of its 8 lanes.
    auto store_row = [&](uint4 v, uint2* to, int plane) __attribute__((always_inline)) {
        v = make_uint4(v.x & mask[0], v.y & mask[1], v.z & mask[2], v.w & mask[3]);
        to[0] = make_uint2(v.x, v.y);
        to[plane] = make_uint2(v.z, v.w);
        int c = popc4(v);
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        c += __builtin_amdgcn_update_dpp(0, c, 0x141, 0xF, 0xF, true);      // the other four of eight
        return c;
    };
    // Rows from the strip's first on, pass by pass, through all its tiles; past the strip's end its last row again.
    const uint32_t* strip_a = A + int64_t(row_begin) * lda;
    const Offset pass_bytes = Offset(PASS_ROWS) * Offset(lda) * 4u;
    const Offset last_row_at = Offset(row_end - 1 - row_begin) * Offset(lda) * 4u + quad_at;
    Offset row_at = Offset(st_r) * Offset(lda) * 4u + quad_at;
    auto load_a = [&]() __attribute__((always_inline)) {
        const uint4 v = load_at(strip_a, row_at < last_row_at ? row_at : last_row_at);
        row_at += pass_bytes;
        return v;
    };
    uint2* put_a = tiles_a + 2 * st_q * PLANE_A + st_r;
    auto store_a = [&](uint4 v, int pass, int buf) __attribute__((always_inline)) {
        const int c = store_row(v, put_a + buf * TILE_A + pass * PASS_ROWS, PLANE_A);
        if (st_q == 0) pop_s[buf][pass * PASS_ROWS + st_r] = -0.5f * float(c);
    };

    // Start: B, thresholds and the first tile, all in flight before the first of them is waited for.
    {
        uint4 vb[BN / PASS_ROWS], va[PASSES];
        int thr[BN / PASS_ROWS];
#pragma unroll
        for (int p = 0; p < BN / PASS_ROWS; ++p) {
            const int n = min(p * PASS_ROWS + st_r, N - 1 - col0);
            vb[p] = load_at(B + int64_t(col0) * ldb, Offset(n) * Offset(ldb) * 4u + quad_at);
            thr[p] = bn.thr[col0 + n];
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) va[p] = load_a();
        if (tid < BN / 32) flip_s[tid] = col0 + 32 * tid < N ? bn.flip_bits[(col0 >> 5) + tid] : 0u;
#pragma unroll
        for (int p = 0; p < BN / PASS_ROWS; ++p) {
            const int c = store_row(vb[p], dyn + 2 * st_q * PLANE_B + p * PASS_ROWS + st_r, PLANE_B);
            if (st_q == 0) colfix_s[p * PASS_ROWS + st_r] = fold_column_term(max(-K - 1, min(K + 1, thr[p])), K, 2 * c);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) store_a(va[p], p, 0);
    }
    __syncthreads();

    // Left factors of the accumulators' start (see conv_strip.hip).
    constexpr short kOne = 0x3F80;
    v4s left[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j) {
        short hi, lo;
        split_bf16(colfix_s[wn * 32 * WN + j * 32 + fr], hi, lo);
        left[j] = fh == 0 ? v4s{hi, lo, kOne, kOne} : v4s{0, 0, 0, 0};
    }
    const uint32_t flip_word = flip_s[wn * WN + fh];
    const int cols_left = N - (col0 + wn * 64 + fh * 32);
    const uint32_t live_word = cols_left >= 32 ? ~0u : cols_left <= 0 ? 0u : ((1u << cols_left) - 1u);
    const uint2* rd_b0 = dyn + fh * PLANE_B + wn * 64 + fr;
    const int half_end = kw - 4 * (kq - 1) == 1;       // the last quad's one word is its fourth: no products of its first step
    // Bytes from the strip's first output word of the wavefront's columns to this lane's.
    char* strip_out = reinterpret_cast<char*>(bn.out + (int64_t(row_begin) * bn.ld_out + ((col0 + wn * 64) >> 5)));
    const Offset out_row = Offset(bn.ld_out) * 4u;

    auto run = [&](auto nb_tag, int row0, int buf, bool more_tiles) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_tag)::value;
        constexpr int VALU = (5 * NB + 6 * WN + NB * WN - 1) / (NB * WN);      // widening of a step, per product
        const bool more = NB == NB_MAX && more_tiles;                          // a tile before the last one is whole
        const uint2* rd_a = tiles_a + buf * TILE_A + fh * PLANE_A + wr * 32 + fr;       // + i * 32 * WAVE_ROWS
        v16f acc[NB][WN];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            short hi, lo;
            split_bf16(pop_s[buf][(i * WAVE_ROWS + wr) * 32 + fr], hi, lo);
            const v4s right = {kOne, kOne, hi, lo};
            v16f zero;
#pragma unroll
            for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
#pragma unroll
            for (int j = 0; j < WN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(left[j], right, zero, 0, 0, 0);
        }
        uint4 next[2];
        if (more) {
            next[0] = load_a();
            next[1] = load_a();
        }
        const uint2* rd_b = rd_b0;
        uint2 aw[NB], bw[WN];
        auto read_words = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) aw[i] = rd_a[i * 32 * WAVE_ROWS];
#pragma unroll
            for (int j = 0; j < WN; ++j) bw[j] = rd_b[j * 32];
        };
        v4i fa[NB], fb[WN], ha[NB], hb[WN];
        read_words();
#pragma unroll
        for (int i = 0; i < NB; ++i) fa[i] = widen4_a(aw[i].x);
#pragma unroll
        for (int j = 0; j < WN; ++j) fb[j] = widen4_b(bw[j].x);
        auto multiply = [&](const v4i (&a)[NB], const v4i (&b)[WN]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand8(b[j]), operand8(a[i]), acc[i][j], 4, 4, 0, 0, 0, 0);
        };
        int q = 0;
        for (int part = more ? 0 : PARTS - 1; part < PARTS; ++part) {
            const int q_end = (part + 1) * (kq - half_end) / PARTS;
            for (; q < q_end; ++q) {
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < kq) {                      // past the end the last quad again, whose products are not taken
                    rd_a += 2 * PLANE_A;
                    rd_b += 2 * PLANE_B;
                }
#pragma unroll
                for (int i = 0; i < NB; ++i) ha[i] = widen4_a(aw[i].y);
#pragma unroll
                for (int j = 0; j < WN; ++j) hb[j] = widen4_b(bw[j].y);
                read_words();
                multiply(fa, fb);
                BNN_STRIP_SCHEDULE(NB * WN, true, VALU);
#pragma unroll
                for (int i = 0; i < NB; ++i) fa[i] = widen4_a(aw[i].x);
#pragma unroll
                for (int j = 0; j < WN; ++j) fb[j] = widen4_b(bw[j].x);
                multiply(ha, hb);
                BNN_STRIP_SCHEDULE(NB * WN, false, VALU);
            }
            if (more) {                                // the other buffer: left by every wavefront before this tile's barrier
                store_a(next[0], 2 * part, buf ^ 1);
                store_a(next[1], 2 * part + 1, buf ^ 1);
                if (part + 1 < PARTS) {
                    next[0] = load_a();
                    next[1] = load_a();
                }
            }
        }

        if (half_end) {
#pragma unroll
            for (int i = 0; i < NB; ++i) ha[i] = widen4_a(aw[i].y);
#pragma unroll
            for (int j = 0; j < WN; ++j) hb[j] = widen4_b(bw[j].y);
            multiply(ha, hb);
        }

        // The output bit is the complement of the accumulator's sign (mfma_output_words).
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            uint32_t part[WN];
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                uint32_t neg = 0u;
#pragma unroll
                for (int v = 3; v >= 0; --v) {
#pragma unroll
                    for (int e = 3; e >= 0; --e)
                        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[i][j][4 * v + e]), 31);
                    if (v > 0) neg <<= 4;
                }
                part[j] = (~neg & 0x0F0F0F0Fu) << (4 * fh);
            }
            const auto sw = __builtin_amdgcn_permlane32_swap(part[0], part[1], false, false);
            const int m = row0 - row_begin + (i * WAVE_ROWS + wr) * 32 + fr;
            if (m < row_end - row_begin && cols_left > 0)
                *reinterpret_cast<uint32_t*>(strip_out + (Offset(m) * out_row + 4u * fh)) = ((sw[0] | sw[1]) ^ flip_word) & live_word;
        }
    };

    int buf = 0;
    for (int row0 = row_begin;;) {
        const bool more = row_end - row0 > BM;
        const int blocks = (min(BM, row_end - row0) + 31) / 32, mine = (blocks - wr + WAVE_ROWS - 1) / WAVE_ROWS;
        if (__builtin_expect(mine == 4, 1)) run(std::integral_constant<int, 4>{}, row0, buf, more);
        else if (mine == 3) run(std::integral_constant<int, 3>{}, row0, buf, more);
        else if (mine == 2) run(std::integral_constant<int, 2>{}, row0, buf, more);
        else if (mine == 1) run(std::integral_constant<int, 1>{}, row0, buf, more);
        if (!more) break;
        row0 += BM;
        buf ^= 1;
        __syncthreads();
    }
}

}  // namespace row_strip

// Which of the products that fit are taken.  Measured on 481 products of 96 < K <= 1024, 44 to 21148 columns and 137 to 28168 rows (us,
// tiles and strips):
//  - strips of more than 128 rows, a block row for every wavefront along the rows and more: with 128 rows 726 x 5243 x 449 4.2 and 4.7, 10120
//    x 260 x 415 4.1 and 4.5; with 192 13618 x 278 x 784 6.2 and 5.4, 388 x 8704 x 674 6.3 and 5.4;
//  - enough of the chip at work: 60 % of it in strips of one or two tiles (9890 x 2048 x 784, 640 rows, 11.2 and 10.1, 2534 x 8485 x 784, 77 %,
//    13.9 and 11.5; 577 x 18637 x 784, 43 %, 8.1 and 9.8), 74 % up to four and 82 % beyond (10019 x 18758 x 784, 57 %, 82.3 and 97.8); a
//    last tile counts as half of one at least;
//  - where the 128 x 128 tiles are at most two to a compute unit, one round, not strips of more than 320 rows with K > 704: 343 x 21148 x 784
//    6.50 and 6.65, 384 x 21248 x 832 6.54 and 6.83, K = 704 6.51 and 6.47, 640 6.50 and 6.09, 310 x 20480 x 784 6.51 and 6.14.
// Three limits date from a kernel whose staging took three times as long, and strips are the faster form beyond them too: K <= 576 (11175 x
// 2225 x 539 13.5 and 10.0; only 384 < K <= 512 on at most 512 tiles of 128 x 128 is 0.92 to 0.98 times as fast in strips), K > 832 on at
// most 512 tiles (13015 x 640 x 838, 510 of them, 6.5 and 5.9), K > 896 in strips of several tiles (18769 x 3584 x 1015 34.3 and 28.7); and
// long strips gain from 65 % of the chip on in part (10397 x 12419 x 784, 77 %, 58.3 and 54.2).
constexpr int64_t kRowStripMinRows = 160;
static_assert(starts_in_bf16_pairs(128 * row_strip::MAX_QUADS));

// BNN_ERR_UNSUPPORTED, with nothing launched, for a product that this kernel does not take or that is faster elsewhere.
int launch_xnor_gemm_mfma_strip(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                const BnSignArgs& bn, void* stream) {
    using namespace row_strip;
    const int64_t tiles_n = ceil_div(N, BN);
    if (K <= 576 || K > 128 * MAX_QUADS || tiles_n > kStripUnits) return BNN_ERR_UNSUPPORTED;
    const StripPlan plan = strip_plan(M, tiles_n);
    const int64_t rows = plan.rows, groups = plan.groups;
    if (rows < kRowStripMinRows || (rows > BM && K > 128 * (MAX_QUADS - 1))) return BNN_ERR_UNSUPPORTED;
    if (ceil_div(M, 128) * tiles_n <= 512 && (K > 832 || (K > 704 && rows > 320))) return BNN_ERR_UNSUPPORTED;
    const int64_t last = rows % BM, cost = rows > BM && last > 0 && last < BM / 2 ? rows - last + BM / 2 : rows;
    if (!strips_fill(M, tiles_n, cost, rows <= 2 * BM ? 60 : rows <= 4 * BM ? 74 : 82)) return BNN_ERR_UNSUPPORTED;
    const Cut cut{fast_div(tiles_n), int(tiles_n), int(groups * tiles_n / kDies), int(rows)};
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(groups * tiles_n)), dim3(T),
                           size_t(2 * MAX_QUADS * (PLANE_B + (rows > BM ? 2 : 1) * PLANE_A)) * sizeof(uint2), static_cast<hipStream_t>(stream), A,
                           lda, B, ldb, int(M), int(N), int(K), bn, cut);
        return check_launch();
    };
    // Rows of A and of the output are counted from a strip's first, up to two tiles past its last; 128 rows of B.
    const int64_t ld = lda > bn.ld_out ? lda : bn.ld_out;
    const bool near = ldb < int64_t(1) << 22 && ld < (int64_t(1) << 29) / (rows + 2 * BM);
    return near ? launch(xnor_gemm_mfma_strip_kernel<uint32_t>) : launch(xnor_gemm_mfma_strip_kernel<uint64_t>);
}

}  // namespace bnn

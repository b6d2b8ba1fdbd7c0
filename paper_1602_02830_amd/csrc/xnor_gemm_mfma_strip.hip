// Fused binary layer (XnorDotProduct -> Sign(BatchNorm), bits in, bits out) of short rows, 576 < K <= 1024, on grids that fill
// the chip: the first layer of an MLP over a whole test set.
//
// The organisation of conv_strip.hip for plain rows: one workgroup of eight wavefronts per compute unit, 128 columns of B resident
// in LDS, an equal strip of A's rows walked in tiles of 512 whose whole K sits in LDS (two buffers); the next tile is
// loaded and stored under the products of the current one, a row's 128 bytes by 8 lanes; accumulators start as the folded
// threshold; the operands of a step are widened between the products of the step before.
//
// What bounds it: with 10 - 16 steps of K a wavefront has 8 x 13 products (K = 784, 3500 cycles at 34) beside a start of 2 - 3 us,
// so what counts is that everything is loaded once and by every compute unit alike.  us, the tiles taken before (128 x 128, whole
// rounds of workgroups) and strips: 16000 x 1000 x 800 11.2 and 9.1, 2000 x 8000 x 600 9.7 and 7.6, 3000 x 3000 x 784 7.9 and 6.8, 6000 x
// 2048 x 784 8.5 and 7.6, 10000 x 4096 x 784 20.6 and 19.9, 16384 x 4096 x 784 28.4 and 26.7.
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
constexpr int PARTS = 4;                               // of a tile's K loop, two passes of the next tile in flight under each

struct Cut {
    FastDiv by_tiles_n;
    int tiles_n, per_die;      // column tiles; workgroups / 8
    int rows;                  // rows per strip, a multiple of 32
};

__global__ __launch_bounds__(T, 2) void xnor_gemm_mfma_strip_kernel(const uint32_t* __restrict__ A, int64_t lda,
                                                                    const uint32_t* __restrict__ B, int64_t ldb, int M, int N,
                                                                    int K, BnSignArgs bn, Cut cut) {
    constexpr int WN = 2;
    extern __shared__ __attribute__((aligned(16))) uint2 dyn[];            // B [kq][2][PLANE_B], then two buffers of A [kq][2][PLANE_A]
    __shared__ float colfix_s[BN];
    __shared__ uint32_t flip_s[BN / 32];
    __shared__ float pop_s[2][BM];                     // minus popcount / 2 of a tile's rows
    const int kw = (K + 31) >> 5, kq = (kw + 3) >> 2;
    const uint32_t tmask = tail_mask(K);
    const int tile_size = 2 * kq * PLANE_A;
    uint2* tiles_a = dyn + 2 * kq * PLANE_B;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fh = lane >> 5;

    int logical = int(blockIdx.x);
    if (logical < kDies * cut.per_die) logical = (logical % kDies) * cut.per_die + logical / kDies;
    const int group = cut.by_tiles_n(logical), col0 = (logical - group * cut.tiles_n) * BN;
    const StripRows strip = strip_rows(group, cut.rows, M);
    const int row_begin = strip.begin, row_end = strip.end;

    // Lane q of 8 takes quad q of a row (lanes past the row's end the last one again, which they do not store).
    const int st_q = tid & 7, st_r = tid >> 3;
    const bool st_live = st_q < kq;
    auto load_row = [&](const uint32_t* P, int64_t ld, int row) __attribute__((always_inline)) {
        return load_row_quad(P + int64_t(row) * ld, min(st_q, kq - 1), kw);
    };
    // Words to LDS, set bits of the row in every one of its 8 lanes.
    auto store_row = [&](uint4 v, uint2* to, int plane) __attribute__((always_inline)) {
        v = place_row_quad(v, st_q, kw, tmask);
        if (st_live) {
            to[(2 * st_q) * plane] = make_uint2(v.x, v.y);
            to[(2 * st_q + 1) * plane] = make_uint2(v.z, v.w);
        }
        int c = popc4(v);
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        c += __builtin_amdgcn_update_dpp(0, c, 0x141, 0xF, 0xF, true);      // the other four of eight
        return c;
    };
    auto load_a = [&](int row0, int pass) __attribute__((always_inline)) { return load_row(A, lda, min(row0 + pass * PASS_ROWS + st_r, row_end - 1)); };
    auto store_a = [&](uint4 v, int pass, int buf) __attribute__((always_inline)) {
        const int r = pass * PASS_ROWS + st_r, c = store_row(v, tiles_a + buf * tile_size + r, PLANE_A);
        if (st_q == 0) pop_s[buf][r] = -0.5f * float(c);
    };

    // Start: B, thresholds and the first tile, all in flight before the first of them is waited for.
    {
        uint4 vb[BN / PASS_ROWS], va[PASSES];
        int thr[BN / PASS_ROWS];
#pragma unroll
        for (int p = 0; p < BN / PASS_ROWS; ++p) {
            const int n = min(col0 + p * PASS_ROWS + st_r, N - 1);
            vb[p] = load_row(B, ldb, n);
            thr[p] = bn.thr[n];
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) va[p] = load_a(row_begin, p);
        if (tid < BN / 32) flip_s[tid] = col0 + 32 * tid < N ? bn.flip_bits[(col0 >> 5) + tid] : 0u;
#pragma unroll
        for (int p = 0; p < BN / PASS_ROWS; ++p) {
            const int c = store_row(vb[p], dyn + p * PASS_ROWS + st_r, PLANE_B);
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
    uint32_t* out = bn.out + ((col0 + wn * 64) >> 5) + fh;                  // this lane's word column
    const uint2* rd_b0 = dyn + fh * PLANE_B + wn * 64 + fr;
    const bool half_end = kw - 4 * (kq - 1) < 2;       // the last quad's second step would multiply words that do not exist

    auto run = [&](auto nb_tag, int row0, int buf, bool more_tiles) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_tag)::value;
        constexpr int VALU = (5 * NB + 6 * WN + NB * WN - 1) / (NB * WN);      // widening of a step, per product
        const bool more = NB == NB_MAX && more_tiles;                          // a tile before the last one is whole
        const uint2* rd_a = tiles_a + buf * tile_size + fh * PLANE_A + wr * 32 + fr;       // + i * 32 * WAVE_ROWS
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
            next[0] = load_a(row0 + BM, 0);
            next[1] = load_a(row0 + BM, 1);
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
            const int q_end = (part + 1) * kq / PARTS;
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
                if (q + 1 == kq && half_end) continue;
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
                    next[0] = load_a(row0 + BM, 2 * part + 2);
                    next[1] = load_a(row0 + BM, 2 * part + 3);
                }
            }
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
            const int m = row0 + (i * WAVE_ROWS + wr) * 32 + fr;
            if (m < row_end && cols_left > 0) out[int64_t(m) * bn.ld_out] = ((sw[0] | sw[1]) ^ flip_word) & live_word;
        }
    };

    int buf = 0;
    for (int row0 = row_begin;;) {
        const bool more = row_end - row0 > BM;
        const int blocks = (min(BM, row_end - row0) + 31) / 32, mine = (blocks - wr + WAVE_ROWS - 1) / WAVE_ROWS;
        if (mine == 4) run(std::integral_constant<int, 4>{}, row0, buf, more);
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

// Strips of more than one block row per wavefront; K from 577 on (shorter rows have kernels 6 and 7, chosen by alignment); at most
// an eighth of columns that do not exist (16384 x 300 x 900 6.4 us before, 6.7 in strips); strips of one tile, or of two
// tiles and more whose two buffers are refilled under K loops of at most 7 quads: 5000 x 4096 x 784 (640 rows, the second tile of one
// block row) 10.9 and 11.4, 10000 x 4096 x 1024 20.1 and 20.8; and with K > 832 only where the 128 x 128 tiles are more than two to a
// compute unit: 15227 x 512 x 987 (476 tiles) 6.6 and 6.9, 1853 x 4224 x 1002 (495) 6.8 and 7.4, 609 x 12519 x 912 (490) 6.7 and 7.2,
// but 5105 x 1732 x 862 (560) 8.0 and 7.1, 36308 x 238 x 926 (568) 8.0 and 7.2; shorter K 2940 x 3000 x 671 (552) 7.9 and 6.4, 2924 x
// 2048 x 784 (368) 6.5 and 6.0.
// Strips that keep most of the chip at work, where the tiles taken otherwise fill it by themselves: 65 % of it with strips of one
// tile (2000 x 6656 x 784, 79 %, 10.1 and 8.3; 1164 x 19579 x 600, 59 %, 13.1 and 15.7), 74 % of two to four (4000 x 6656 x 784, 79 %,
// 15.6 and 14.3; 4000 x 12000 x 784, 73 %, 25.1 and 26.0), 82 % with longer ones (10000 x 6656 x 784, 80 %, 31.2 and 32.0, 10000 x 12000
// x 784, 72 %, 53.7 and 60.9, 10000 x 16512 x 784, 50 %, 82 and 116; 10000 x 5504 x 784, 83 %, level, 4000 x 32768 x 784, 98 %, 53.3
// and 49.4).  A last tile counts as half of one at least (4141 x 7168 x 810, 1056 rows, 15.9 and 17.6).
constexpr int64_t kRowStripMinRows = 160;
static_assert(starts_in_bf16_pairs(128 * row_strip::MAX_QUADS));

// BNN_ERR_UNSUPPORTED, with nothing launched, for a product that this kernel does not take or that is faster elsewhere.
int launch_xnor_gemm_mfma_strip(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                const BnSignArgs& bn, void* stream) {
    using namespace row_strip;
    const int64_t tiles_n = ceil_div(N, BN);
    if (K <= 576 || K > 128 * MAX_QUADS || tiles_n > kStripUnits || 8 * N < 7 * BN * tiles_n) return BNN_ERR_UNSUPPORTED;
    const StripPlan plan = strip_plan(M, tiles_n);
    const int64_t rows = plan.rows, groups = plan.groups;
    if (K > 832 && ceil_div(M, 128) * tiles_n <= 512) return BNN_ERR_UNSUPPORTED;
    if (rows < kRowStripMinRows || (rows > BM && (rows < 2 * BM || K > 128 * (MAX_QUADS - 1)))) return BNN_ERR_UNSUPPORTED;
    const int64_t last = rows % BM, cost = rows > BM && last > 0 && last < BM / 2 ? rows - last + BM / 2 : rows;
    if (!strips_fill(M, tiles_n, cost, rows <= BM ? 65 : rows <= 4 * BM ? 74 : 82)) return BNN_ERR_UNSUPPORTED;
    const Cut cut{fast_div(tiles_n), int(tiles_n), int(groups * tiles_n / kDies), int(rows)};
    const int64_t kq = ceil_div(K, 128);
    hipLaunchKernelGGL(xnor_gemm_mfma_strip_kernel, dim3(unsigned(groups * tiles_n)), dim3(T),
                       size_t(2 * kq * (PLANE_B + (rows > BM ? 2 : 1) * PLANE_A)) * sizeof(uint2), static_cast<hipStream_t>(stream), A, lda,
                       B, ldb, int(M), int(N), int(K), bn, cut);
    return check_launch();
}

}  // namespace bnn

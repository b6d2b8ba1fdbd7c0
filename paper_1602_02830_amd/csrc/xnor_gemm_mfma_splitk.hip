// Bits-in, matrix-engine-inside binary product (Sec. 4 Eq. (5), the XnorDotProduct of Alg. 4) for
// small outputs with a long K: the fully connected layers of a network at inference batch sizes
// (in the ConvNet architecture that Sec. 2.2 refers to, at batch 256: 256 x 1024 outputs over
// K = 8192), where 128 x 128 or 256 x 128 output tiles would leave most of the 256 compute units
// without a tile.
//
// A workgroup owns one 32 x 32 or 64 x 32 output tile and splits K over its four wavefronts; every
// wavefront multiplies its share of K into partial sums of the whole tile, which meet in LDS once.
// v_mfma_f32_32x32x64_f8f6f4 takes "lane (r = lane % 32, h = lane / 32) holds 32 consecutive K elements of row
// r" as its operand, and the order in which K is summed is free, so a quad (4 words = 128 bits of a row) feeds four
// MFMAs: its words are widened to fp4 codes (mfma_fp4.h) one after the other.  How the quads get there:
//
//   direct  of every aligned group of 8 quads wavefront w takes quads 2w and 2w + 1, one per lane half, loaded
//           from global memory straight into the operand registers.  Nothing is staged in LDS and no
//           barrier is met inside the K loop; a lane fetches the next 4 quads of each operand while it multiplies the
//           current 4, so the loop exposes one round trip to memory.
//   staged  of every 32 quads a wavefront takes 8 consecutive ones, 8 lanes a row's 128 bytes, and exchanges them
//           through a piece of LDS of its own (no barrier either); the next round's loads are in flight
//           meanwhile.  A direct load touches 32 rows with 32 bytes each, which costs the memory pipe 19
//           cycles where rows are 16-byte aligned and 62 where they are not, and four wavefronts fetch a line each
//           their quarter; staged, both are whole lines.  The way through LDS costs a few hundred cycles once.
//
// What bounds them (cycle stamps, 1000 x 1000, K = 4097 int32, 1024 tiles of 32 x 32, direct: 12500 cycles per
// workgroup, 4 on a compute unit): 4600 until the loads are issued (unaligned rows), 3500 of multiplying in their shadow,
// 1500 waiting for the slowest wavefront, 1400 in the epilogue; 8.6 us.  64 x 32 staged, rows leaving in 16-byte
// stores: 6.8 us.
//
// Requirements (checked by the launcher): 96 < K <= 2^24 (a row has at least one quad to load; exact fp32
// sums).  Rows may start at any 4-byte alignment.
#include <cstdint>

#include "bnn_internal.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"

namespace bnn {
namespace splitk {

constexpr int kWaves = 4;
constexpr int kQuadStride = 2 * kWaves;   // direct: quads between two consecutive quads of one lane
constexpr int kBatch = 4;                 // direct: quads of each operand a lane loads at a time (two such batches in flight)
constexpr int kChunk = 8;                 // staged: quads of a row that a wavefront takes at a time, one 128-byte line

// Sums and popcounts of a wavefront's share of K for RB blocks of 32 x 32 below each other (quads: RB of A, then one of B).
template <int RB, bool SWAPPED>
struct Partial {
    static constexpr int ROWS = RB + 1;
    // One block has two accumulators, so that consecutive MFMAs do not wait for each other's result.
    static constexpr int ACCS = RB == 1 ? 2 : 1;
    v16f acc[RB][ACCS];
    int cnt[ROWS];

    __device__ inline void clear() {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int x = 0; x < ACCS; ++x)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][x][v] = 0.0f;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) cnt[i] = 0;
    }

    __device__ inline void multiply(const uint4 (&q)[ROWS]) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) cnt[i] += popc4(q[i]);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const v8i fb = widen_fp4_b(quad_word(q[RB], s));
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const v8i fa = widen_fp4_a(quad_word(q[i], s));
                v16f& to = acc[i][s % ACCS];
                to = SWAPPED ? __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb, fa, to, 4, 4, 0, 0, 0, 0)
                             : __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa, fb, to, 4, 4, 0, 0, 0, 0);
            }
        }
    }

    // Accumulator registers 4g .. 4g + 3 of block i.
    __device__ inline float4 sums(int i, int g) const {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = ACCS == 1 ? acc[i][0][4 * g + e] : acc[i][0][4 * g + e] + acc[i][ACCS - 1][4 * g + e];
        return make_float4(v[0], v[1], v[2], v[3]);
    }
};

template <int RB, bool SWAPPED>
__device__ inline void multiply_direct(Partial<RB, SWAPPED>& part, const uint32_t* const (&row)[RB + 1], int K, int first) {
    constexpr int ROWS = RB + 1;
    const int kw = (K + 31) >> 5, nq = (kw + 3) >> 2, n_whole = K >> 7;
    const uint32_t tmask = tail_mask(K);
    auto load_step = [&](int step, uint4 (&q)[ROWS]) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) q[i] = load_quad_any(row[i] + 4 * (kQuadStride * step + first));
    };
    // K as whole batches of 32 quads and a rest of up to four steps.  The rest goes first: its loads sit behind
    // branches (steps none of whose quads exist are left out: their loads would cost as much as any), so whoever waits
    // for them waits for every load before them as well - here the first batch, which is in flight with them.  The
    // batches' own loads carry no control flow.  Every lane runs every MFMA of a step: a quad of the rest that is not
    // whole, or not there, is loaded from the row's last four words and put right afterwards.
    // (A K of at most one batch is all rest: one piece of straight code, 256 x 1024 x 1024 3.2 -> 3.1 us.)
    const int batches = nq <= kQuadStride * kBatch ? 0 : n_whole / (kQuadStride * kBatch);
    const int rest = batches * (kQuadStride * kBatch);
    uint4 q[kBatch][ROWS], n[kBatch][ROWS];
    if (batches > 0) {
#pragma unroll
        for (int t = 0; t < kBatch; ++t) load_step(t, q[t]);
    }
#pragma unroll
    for (int t = 0; t < kBatch; ++t)
        if (rest + kQuadStride * t < nq) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) n[t][i] = load_row_quad(row[i], rest + first + kQuadStride * t, kw);
        }
#pragma unroll
    for (int t = 0; t < kBatch; ++t) {
        const int qt = rest + kQuadStride * t;
        if (qt >= nq) break;
        if (qt + kQuadStride > n_whole) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) n[t][i] = place_row_quad(n[t][i], qt + first, kw, tmask);
        }
        part.multiply(n[t]);
    }
    // A step's registers are loaded again for the next batch as soon as it is multiplied: three steps of the batch (and
    // the other wavefronts) cover the load, and 64 registers fewer than with a second set keep 4 workgroups resident.
    for (int b = 1; b < batches; ++b) {
#pragma unroll
        for (int t = 0; t < kBatch; ++t) {
            part.multiply(q[t]);
            load_step(b * kBatch + t, q[t]);
            __builtin_amdgcn_sched_barrier(0);             // or the loads sink behind the MFMAs
        }
    }
    if (batches > 0) {
#pragma unroll
        for (int t = 0; t < kBatch; ++t) part.multiply(q[t]);
    }
}

// The fused product on 32 x 32 tiles, direct: Sign(BatchNorm(.)) of Alg. 4 on folded thresholds (bn_fold.cpp).  Wavefront w
// finishes accumulator registers 4w .. 4w + 3, i.e. rows 8w + 4h + e of the tile: pre-activation K - 2pa - 2pb + 4S, compared
// with the threshold and turned into output words by one ballot per register (the ballot's two halves are the words of
// two rows).
__global__ __launch_bounds__(256, 4) void xnor_gemm_mfma_splitk_kernel(
    const uint32_t* __restrict__ A, int64_t lda, const uint32_t* __restrict__ B, int64_t ldb, int M, int N, int K,
    TileMap tiles, BnSignArgs bn) {
    __shared__ float4 part_s[kWaves][4][kWave];   // [wavefront][accumulator registers 4g .. 4g+3][lane]
    __shared__ __attribute__((aligned(16))) int pop_part[kWaves][kWave];   // 2*popcount over the wavefront's share of K:
                                                                          // [0, 32) rows of A, [32, 64) rows of B
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fr = lane & 31, fh = lane >> 5;
    int tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const int row0 = tm * 32, col0 = tn * 32;

    // Rows beyond the matrix repeat its last row; their results are never stored.
    const uint32_t* const rows[2] = {A + int64_t(min(row0 + fr, M - 1)) * lda, B + int64_t(min(col0 + fr, N - 1)) * ldb};
    // The column's threshold and flip bit are fetched with the first operands, not after the K loop.
    const int col = col0 + fr;
    const int thr = bn.thr[min(col, N - 1)];
    const uint32_t flip_word = bn.flip_bits[min(col, N - 1) >> 5];

    Partial<1, false> part;
    part.clear();
    multiply_direct(part, rows, K, 2 * wave + fh);

    // Lanes 0-31 end up with the popcount of A's row fr over both lane halves, lanes 32-63 with
    // that of B's row fr (one v_permlane32_swap exchanges the upper half of one with the lower half of the other).
    const auto sw = __builtin_amdgcn_permlane32_swap(uint32_t(part.cnt[0]), uint32_t(part.cnt[1]), false, false);
    pop_part[wave][lane] = 2 * int(sw[0] + sw[1]);
#pragma unroll
    for (int g = 0; g < 4; ++g) part_s[wave][g][lane] = part.sums(0, g);
    __syncthreads();

    // Accumulator register v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32.
    float4 s4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int4 pa4 = make_int4(0, 0, 0, 0);
    int pb = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const float4 p = part_s[w][wave][lane];
        s4.x += p.x; s4.y += p.y; s4.z += p.z; s4.w += p.w;
        const int4 pa = *reinterpret_cast<const int4*>(&pop_part[w][8 * wave + 4 * fh]);
        pa4.x += pa.x; pa4.y += pa.y; pa4.z += pa.z; pa4.w += pa.w;
        pb += pop_part[w][32 + fr];
    }
    const int base = K - pb;
    const int dot[4] = {base - pa4.x + (int(s4.x) << 2), base - pa4.y + (int(s4.y) << 2),
                        base - pa4.z + (int(s4.z) << 2), base - pa4.w + (int(s4.w) << 2)};
    const bool valid = col < N;
    const bool flip = (flip_word >> (col & 31)) & 1u;
    // Ballot e: low half = the word of row 8*wave + e, high half = that of row 8*wave + 4 + e.
    // Lane i < 8 stores row 8*wave + i.
    uint32_t word = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint64_t mask = __ballot(valid & ((dot[e] >= thr) != flip));     // not &&: a branch here takes the LDS reads apart
        if ((lane & 3) == e) word = (lane & 4) ? uint32_t(mask >> 32) : uint32_t(mask);
    }
    const int row = row0 + 8 * wave + lane;
    if (lane < 8 && row < M) bn.out[int64_t(row) * bn.ld_out + tn] = word;
}

// The other forms: 32*RB x 32 tiles, direct or staged, int32 or fused.  The MFMAs have their operands swapped, so that a lane
// holds 16 columns of one output row in groups of 4, and 8 neighbouring threads finish the 32 columns of one row: an
// int32 row leaves in 16-byte stores (with one column per lane, four-byte stores of two rows each, the epilogue took
// 1400 cycles instead of 800: 100 x 4096 x 784 3.7 -> 3.2 us), a fused one is OR-ed together to one word.
// REST (staged): up to kRestMost quads past whole rounds of 32 make no round, whose trip to memory nothing would cover: every wavefront
// has a pair of them at most, loaded with its first round's by the lanes that multiply it.  1000 x 1000 x 4097 6.7 -> 5.9 us (4096 5.7),
// x 8193 9.3 -> 8.4, fused 1000 x 1000 x 4097 6.4 -> 5.9.  A kernel of its own: as a branch it made products without such a rest up to 4 % slower.
constexpr int kRound = kWaves * kChunk, kRestMost = 2 * kWaves;
template <int RB, bool FUSED, bool STAGED, bool REST = false>
__global__ __launch_bounds__(256, RB == 1 ? 4 : 2) void xnor_gemm_mfma_splitk_rows_kernel(
    const uint32_t* __restrict__ A, int64_t lda, const uint32_t* __restrict__ B, int64_t ldb,
    int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, TileMap tiles, BnSignArgs bn) {
    constexpr int ROWS = RB + 1;                               // operand rows of a lane: RB of A, one of B
    // A wavefront's piece of LDS: first its chunk (STAGED), [row][quad, exchanged within the row by the row's last three
    // bits], then its partial sums, [block][register group][lane half][row].  Odd strides (in 16-byte slots) keep both the
    // writes, consecutive rows, and the reads, 8 column quads of a row, spread over the banks.
    constexpr int HALF = 33, GROUP = 2 * HALF, CHUNK = STAGED ? 32 * ROWS * kChunk : 0, SUMS = 4 * RB * GROUP;
    __shared__ uint4 lds[kWaves][CHUNK > SUMS ? CHUNK : SUMS];
    __shared__ __attribute__((aligned(16))) int pop_part[kWaves][(ROWS + 1) / 2 * kWave];   // popcounts over the
                                                               // wavefront's share of K: rows of A, then rows of B
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    int tm, tn;
    tile_of_block(blockIdx.x, tiles, tm, tn);
    const int row0 = tm * 32 * RB, col0 = tn * 32;

    // This thread finishes columns n0 .. n0 + 3 of every 32nd row.  Thresholds and flip word are fetched with the first
    // operands, not after the K loop.
    const int cq = tid & 7, n0 = col0 + 4 * cq;
    int thr[4];
    uint32_t flip = 0u;
    auto load_thresholds = [&] {
        if constexpr (FUSED) {
#pragma unroll
            for (int e = 0; e < 4; ++e) thr[e] = bn.thr[min(n0 + e, N - 1)];
            flip = bn.flip_bits[min(n0, N - 1) >> 5];
        }
    };

    Partial<RB, true> part;
    part.clear();
    uint4* mine = lds[wave];
    // Rows beyond the matrix repeat its last row; their results are never stored.
    if constexpr (STAGED) {
        const int kw = (K + 31) >> 5, nq = (kw + 3) >> 2, n_whole = K >> 7;
        const uint32_t tmask = tail_mask(K);
        constexpr int LOADS = 4 * ROWS;                        // of a chunk: 8 rows of 8 quads each
        const int st_q = lane & 7, st_r = lane >> 3;
        const int st_slot = st_r * kChunk + (st_q ^ st_r);     // + 64 * load
        const uint32_t* from[LOADS];
#pragma unroll
        for (int l = 0; l < 4 * RB; ++l) from[l] = A + int64_t(min(row0 + 8 * l + st_r, M - 1)) * lda;
#pragma unroll
        for (int l = 0; l < 4; ++l) from[4 * RB + l] = B + int64_t(min(col0 + 8 * l + st_r, N - 1)) * ldb;
        uint4 r[LOADS];
        // Rounds of 32 quads, 8 per wavefront; the last round's are shared out evenly, in pairs (the lane halves).
        const int n_staged = REST ? nq - nq % kRound : nq, rounds = (n_staged + kRound - 1) / kRound;
        const int share = REST ? kChunk : ((n_staged - (rounds - 1) * kRound + 7) >> 3) * 2;       // 2, 4, 6 or 8
        auto first_quad = [&](int round) { return round * kWaves * kChunk + wave * (REST || round + 1 < rounds ? kChunk : share); };
        auto fetch = [&](int round) {
            const int q = first_quad(round) + (REST ? st_q : min(st_q, round + 1 < rounds ? kChunk : share - 1));
            const int w = REST ? 4 * q : min(4 * q, kw - 4);                           // see load_row_quad
#pragma unroll
            for (int l = 0; l < LOADS; ++l) r[l] = load_quad_any(from[l] + w);
        };
        fetch(0);
        const int rest_q = n_staged + 2 * wave;
        const bool my_rest = REST && rest_q < nq;
        uint4 rest_words[ROWS];
        if (my_rest) {
#pragma unroll
            for (int i = 0; i < RB; ++i)
                rest_words[i] = load_row_quad(A + int64_t(min(row0 + 32 * i + fr, M - 1)) * lda, rest_q + fh, kw);
            rest_words[RB] = load_row_quad(B + int64_t(min(col0 + fr, N - 1)) * ldb, rest_q + fh, kw);
        }
        load_thresholds();
        for (int round = 0; round < rounds; ++round) {
            const int q0 = first_quad(round), q_end = min(n_staged, round + 1 < rounds ? q0 + kChunk : q0 + share);
#pragma unroll
            for (int l = 0; l < LOADS; ++l) mine[64 * l + st_slot] = r[l];
            if (round + 1 < rounds) fetch(round + 1);
            asm volatile("" : : : "memory");                   // LDS is in order within a wavefront; so is the code
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < kChunk / 2; ++t) {
                if (!REST && q0 + 2 * t >= q_end) break;
                uint4 q[ROWS];
#pragma unroll
                for (int i = 0; i < ROWS; ++i) q[i] = mine[(32 * i + fr) * kChunk + ((2 * t + fh) ^ (fr & 7))];
                // A quad that is not whole, or not there, was loaded from the row's last four words.
                if (!REST && q0 + 2 * t + 2 > n_whole) {
#pragma unroll
                    for (int i = 0; i < ROWS; ++i) q[i] = place_row_quad(q[i], q0 + 2 * t + fh, kw, tmask);
                }
                part.multiply(q);
            }
            asm volatile("" : : : "memory");
            __builtin_amdgcn_wave_barrier();
        }
        if (my_rest) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) rest_words[i] = place_row_quad(rest_words[i], rest_q + fh, kw, tmask);
            part.multiply(rest_words);
        }
    } else {
        const uint32_t* row[ROWS];
#pragma unroll
        for (int i = 0; i < RB; ++i) row[i] = A + int64_t(min(row0 + 32 * i + fr, M - 1)) * lda;
        row[RB] = B + int64_t(min(col0 + fr, N - 1)) * ldb;
        load_thresholds();
        multiply_direct(part, row, K, 2 * wave + fh);
    }

    // Lanes 0-31 end up with the popcount of one row over both lane halves, lanes 32-63 with that of the next (one
    // v_permlane32_swap exchanges the upper half of the first with the lower half of the second).
#pragma unroll
    for (int i = 0; i < ROWS; i += 2) {
        const auto sw = __builtin_amdgcn_permlane32_swap(uint32_t(part.cnt[i]), uint32_t(part.cnt[i + 1 < ROWS ? i + 1 : i]), false, false);
        pop_part[wave][32 * i + lane] = int(sw[0] + sw[1]);
    }
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(&mine[(4 * i + g) * GROUP + fh * HALF + fr]) = part.sums(i, g);
    __syncthreads();

    // Register 4g + e of lane (r, h): row r, column 8g + 4h + e of its block.  All LDS reads first: left to itself the
    // compiler moves those of a row behind the check that the row exists, and each row waits for its own.
    float4 p[RB][kWaves];
    int pa[RB][kWaves];
    int4 pb[kWaves];
    const int ml = tid >> 3;
    const int slot = (cq >> 1) * GROUP + (cq & 1) * HALF + ml;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        pb[w] = *reinterpret_cast<const int4*>(&pop_part[w][32 * RB + 4 * cq]);
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            p[i][w] = *reinterpret_cast<const float4*>(&lds[w][slot + 4 * i * GROUP]);
            pa[i][w] = pop_part[w][32 * i + ml];
        }
    }
    int base[4] = {K, K, K, K};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        base[0] -= 2 * pb[w].x; base[1] -= 2 * pb[w].y; base[2] -= 2 * pb[w].z; base[3] -= 2 * pb[w].w;
    }
    int dot[RB][4];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        int a = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            s[0] += p[i][w].x; s[1] += p[i][w].y; s[2] += p[i][w].z; s[3] += p[i][w].w;
            a += pa[i][w];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dot[i][e] = base[e] - 2 * a + (int(s[e]) << 2);
            asm volatile("" : "+v"(dot[i][e]));
        }
    }
    if constexpr (!FUSED) {
        int32_t* to = C + int64_t(row0 + ml) * ldc + n0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (row0 + ml + 32 * i < M) {
                if (n0 + 4 <= N) {
                    store_quad_any(reinterpret_cast<uint32_t*>(to), make_uint4(uint32_t(dot[i][0]), uint32_t(dot[i][1]),
                                                                               uint32_t(dot[i][2]), uint32_t(dot[i][3])));
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (n0 + e < N) to[e] = dot[i][e];
                }
            }
            to += 32 * ldc;
        }
    } else {
        const int left = N - col0;
        const uint32_t live = left >= 32 ? ~0u : (1u << left) - 1u;
        uint32_t word[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            uint32_t bits = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) bits |= (dot[i][e] >= thr[e] ? 1u : 0u) << e;
            word[i] = (or_reduce8(bits << (4 * cq)) ^ flip) & live;
        }
        if (cq == 0) {
            uint32_t* to = bn.out + int64_t(row0 + ml) * bn.ld_out + tn;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                if (row0 + ml + 32 * i < M) *to = word[i];
                to += 32 * bn.ld_out;
            }
        }
    }
}

}  // namespace splitk

bool mfma_splitk_supports(int64_t M, int64_t N, int64_t K) {
    return K > 96 && K <= kMfmaMaxAcc && M >= 1 && N >= 1 && ceil_div(M, 32) * ceil_div(N, 32) <= kMaxDim;
}

template <int RB, bool STAGED, bool REST = false>
static int launch_splitk_rows(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                              int64_t M, int64_t N, int64_t K, bool fused, const BnSignArgs& bn, hipStream_t s) {
    if constexpr (STAGED && !REST) {
        // Fused 32 x 32 tiles have no such kernel, though they would gain as others do (100 x 4096 x 4097 8 %).
        const int64_t nq = ceil_div(K, 128), past = nq % splitk::kRound;
        if (nq > splitk::kRound && past > 0 && past <= splitk::kRestMost && (RB > 1 || !fused))
            return launch_splitk_rows<RB, true, true>(A, lda, B, ldb, C, ldc, M, N, K, fused, bn, s);
    }
    const int64_t tiles_m = ceil_div(M, 32 * RB), tiles_n = ceil_div(N, 32);
    const dim3 grid(unsigned(tiles_m * tiles_n));
    if (!fused) {
        hipLaunchKernelGGL((splitk::xnor_gemm_mfma_splitk_rows_kernel<RB, false, STAGED, REST>), grid, dim3(256), 0, s, A, lda, B, ldb,
                           C, ldc, int(M), int(N), int(K), tile_map(tiles_m, tiles_n), bn);
    } else if constexpr (RB == 1 && !STAGED) {
        hipLaunchKernelGGL(splitk::xnor_gemm_mfma_splitk_kernel, grid, dim3(256), 0, s, A, lda, B, ldb, int(M), int(N), int(K),
                           tile_map(tiles_m, tiles_n), bn);
    } else if constexpr (RB > 1 || !REST) {
        hipLaunchKernelGGL((splitk::xnor_gemm_mfma_splitk_rows_kernel<RB, true, STAGED, REST>), grid, dim3(256), 0, s, A, lda, B, ldb,
                           static_cast<int32_t*>(nullptr), int64_t(0), int(M), int(N), int(K), tile_map(tiles_m, tiles_n), bn);
    }
    return check_launch();
}

// Which products with t tiles of 32 x 32 the automatic choice sends here (fused and int32 alike), and in which form.
// Launches replayed from a graph, us; "tiles": the 64 x 128 tiles with K in one piece that take what is not sent here.  1750
// products were measured in both forms.
//  - 64 x 32 tiles above 896 tiles of 32 x 32 (t = 704 fused K = 4096 5.5 vs 5.4 on 32 x 32, t = 1024 5.5 vs 6.1) where that
//    multiplies no more than an eighth of rows that do not exist, and only in as many as two of them fill a compute unit, three
//    above t = 1024: one more leaves most units waiting for a few (416 x 2368 x 4580, t = 962 in 518, 7.8 vs 6.4 on 32 x 32, 672 x
//    2235 x 4480, t = 1470 in 770, 9.6 vs 8.4 on tiles);
//  - so up to t = 1536 with K >= 1000 instead of t = 1024 with K >= 512: t = 1250 fused K = 1000 4.4 vs 4.6 on tiles,
//    K = 3000 6.2 vs 7.0, K = 8192 9.7 vs 12.6, t = 1504 int32 K = 4096 7.0 vs 8.1; but K = 512 4.2 vs 3.8 and t = 1824
//    K = 4096 8.3 vs 8.0;
//  - staged above t = 256, not where many rows repeat the last one, which are loaded once directly (1 x 32000, K = 4097 6.6 vs 7.3
//    staged, 33 x 8000, K = 4097 5.1 vs 5.6):
//      rows that are whole 128-byte lines apart but for a word, from 32 quads on: what 32 rows of a direct load want then lies at
//      the same place of their lines, and staged is 1.04 to 1.3 times faster at every t and form (t = 512 fused K = 4096 4.3
//      vs 5.0, t = 1024 int32 K = 4097 6.8 vs 8.0, t = 485 K = 10212 6.4 vs 7.9);
//      other rows only where the last round of 32 quads is well filled: 49 to 64 quads (t = 776 int32 K = 7680 1.08 times faster; fused
//      up to t = 896 from 57 on; 64 x 32 fused from 41 on, and above t = 1024 from 34 on without end), 89 to 96, 121 to 128 and so
//      on above t = 512 (1.03), and 24 to 30, one round, int32 up to t = 896 (1.02).  With 33 to 40 quads staged takes 1.05 to 1.15 times as long (t = 750 fused K = 4160 5.9 vs 5.4),
//      with 65 to 88 as well (1003 tiles, int32 K = 8704 11.5 vs 10.2).  Those figures are of rounds alone: where a short rest makes no
//      round (REST), 33 to 40 and 65 to 72 quads of such rows were not measured again and are read directly.
static bool splitk_two_rows(int64_t M, int64_t N) {
    const int64_t t = ceil_div(M, 32) * ceil_div(N, 32), t64 = ceil_div(M, 64) * ceil_div(N, 32);
    return t > 896 && t64 <= (t <= 1024 ? 512 : 768) && 16 * ceil_div(M, 64) <= 9 * ceil_div(M, 32);
}

bool mfma_splitk_prefers(int64_t M, int64_t N, int64_t K, bool fused) {
    const int64_t t = ceil_div(M, 32) * ceil_div(N, 32);
    if (t <= 512 || (t <= 1024 && K >= 512)) return true;
    const bool skinny = !fused && (N <= 16 || M <= 4);          // the lane-group kernel's
    return t <= 1536 && K >= 1000 && !skinny && splitk_two_rows(M, N);
}

// `bn.out == nullptr` selects the int32 form.  The caller has validated the arguments and
// checked mfma_splitk_supports.
int launch_xnor_gemm_mfma_splitk(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C,
                                 int64_t ldc, int64_t M, int64_t N, int64_t K, bool fused, const BnSignArgs& bn,
                                 void* stream) {
    if (!mfma_splitk_supports(M, N, K)) return BNN_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t t = ceil_div(M, 32) * ceil_div(N, 32);
    const int64_t quads = ceil_div(K, 128), last = (quads - 1) % 32;        // quads of the last round, less one
    const bool two_rows = splitk_two_rows(M, N);
    const bool few_repeated = 4 * M >= 96 * ceil_div(M, 32) && 4 * N >= 96 * ceil_div(N, 32);
    auto whole_lines = [](int64_t ld) { return (ld + 1) % 32 <= 2; };        // but for a word
    const int64_t first = two_rows && fused ? (t > 1024 ? 34 : 41) : fused && t <= 896 ? 57 : 49;
    const bool filled = quads >= first ? quads <= 64 || (last >= 24 && t > 512) || (fused && t > 1024)
                                       : !fused && t <= 896 && quads >= 24 && quads <= 30;
    const bool staged = t > 256 && few_repeated && (whole_lines(lda) && whole_lines(ldb) ? quads >= 32 : filled);
    if (staged)
        return two_rows ? launch_splitk_rows<2, true>(A, lda, B, ldb, C, ldc, M, N, K, fused, bn, s)
                        : launch_splitk_rows<1, true>(A, lda, B, ldb, C, ldc, M, N, K, fused, bn, s);
    return two_rows ? launch_splitk_rows<2, false>(A, lda, B, ldb, C, ldc, M, N, K, fused, bn, s)
                    : launch_splitk_rows<1, false>(A, lda, B, ldb, C, ldc, M, N, K, fused, bn, s);
}

}  // namespace bnn

// First hidden layer of Alg. 4 on real inputs at small batches, in one launch:
//     a^b_0 = Sign(x), packed;   a^b_1 = Sign(BatchNorm(XnorDotProduct(a^b_0, W^b_1)))
//
// A launch costs the host 3.6 us and the device 2.1 us before it has done anything, more than packing 100 x 784 reals takes: a
// network of five launches is bound by their number (784-4096-4096-4096-10 at batch 100: 19.2 us in five launches, 16.8 in four).  So
// every workgroup binarizes the 16 rows it needs itself, 50 KB of reals from L2, and goes on to multiply: 100 x 4096 x 784 4.0 us
// replayed from a graph, 5.2 in two launches.
//
// A workgroup is eight wavefronts and owns 16 rows x 128 columns (v_mfma_f32_16x16x128_f8f6f4: 16 rows rather than 32 halve the reals
// that go through a compute unit at 64 bytes a cycle).  Lane l of a 64-element piece of a row compares element l with zero, so the
// comparison's lane mask is two packed words as they stand.  What bounds it is the number of instructions: with four wavefronts of
// twice the rows and columns, clamped addresses and bits counted piece by piece it took 5.0 us; now a buffer load checks a row's end
// itself, masks are applied to whole words and the words' bits are counted by the lanes that multiply them.  The words meet in
// LDS, planes [word][row]; the filters' words go straight from memory to the lanes that widen them, their loads in flight before the
// reals'.  Arithmetic and folded thresholds are those of mfma_fp4.h.
#include "bnn_internal.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"

namespace bnn {
namespace sign_gemm {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int BM = 16, BN = 128, T = 512, WAVES = 8;
constexpr int ROWS = BM / WAVES;                           // rows a wavefront binarizes
constexpr int PITCH = BM + 1;                              // words per plane: the pieces of a row fall into different banks

// 4 bytes at `offset` bytes from `base` (uniform), zero from `bytes` on: the unit checks the bound, and steps of `offset` that the
// compiler knows are part of the instruction.
__device__ inline uint32_t load_below(const void* base, uint32_t bytes, uint32_t offset) {
    constexpr int kWords = 0x00027000;                     // data format: 32 bits
    return __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, kWords), offset, 0, 0);
}

// Sum (or OR) of a value over the four lanes of every 16 that hold the same row: lanes r, r + 16, r + 32, r + 48.
template <typename F>
__device__ inline uint32_t over_groups(uint32_t v, F&& join) {
    const auto s16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t pair = join(s16[0], s16[1]);
    const auto s32 = __builtin_amdgcn_permlane32_swap(pair, pair, false, false);
    return join(s32[0], s32[1]);
}

// PIECES: 64-element pieces of a row, all of K.
template <int PIECES>
__global__ __launch_bounds__(T) void sign_gemm_kernel(const float* __restrict__ x, int64_t ldx, const uint32_t* __restrict__ B,
                                                      int64_t ldb, int M, int N, int K, int tiles_n, FastDiv by_tiles_n,
                                                      BnSignArgs bn, uint32_t* __restrict__ a_bits, int64_t ld_a) {
    constexpr int STEPS = (PIECES + 1) / 2;                // of 128 elements
    __shared__ uint32_t bits_s[4 * STEPS * PITCH];
    __shared__ __attribute__((aligned(16))) float col_s[BN];
    const int tile_m = by_tiles_n(int(blockIdx.x)), tile_n = int(blockIdx.x) - tile_m * tiles_n;
    const int row0 = tile_m * BM, col0 = tile_n * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int kw = (K + 31) >> 5;
    const uint32_t tmask = tail_mask(K);

    // Filters: words 4s + g of column r of the wavefront's 16; past a row's end words of the next one, which meet zeros.
    const int col = min(col0 + 16 * wave, N - 1), cols = min(16, N - col);
    uint32_t w[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
        w[s] = load_below(B + int64_t(col) * ldb, uint32_t((cols - 1) * int(ldb) + kw) * 4u,
                          uint32_t(min(r, cols - 1)) * uint32_t(ldb) * 4u + 4u * g + 16u * s);
    const int word = (col0 >> 5) + (wave >> 1), nw = (N + 31) >> 5, half = wave & 1;
    const int thr = bn.thr[min(col0 + 16 * wave + r, N - 1)];
    const uint32_t flip = bn.flip_bits[min(word, nw - 1)];

    // Reals, and their signs as words.
    uint32_t v[ROWS][PIECES];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)
#pragma unroll
        for (int c = 0; c < PIECES; ++c)
            v[i][c] = load_below(x + int64_t(min(row0 + ROWS * wave + i, M - 1)) * ldx, uint32_t(K) * 4u, 4u * lane + 256u * c);
    const int at = 2 * lane;                               // lane c ends up with words 2c and 2c + 1 of the row
    const uint32_t low_mask = at < kw - 1 ? ~0u : at == kw - 1 ? tmask : 0u, high_mask = at + 1 < kw - 1 ? ~0u : at + 1 == kw - 1 ? tmask : 0u;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        int low = 0, high = 0;
#pragma unroll
        for (int c = 0; c < PIECES; ++c) {
            const uint64_t m = __ballot(__uint_as_float(v[i][c]) >= 0.0f);
            low = bnn_llvm_writelane(int(uint32_t(m)), c, low);
            high = bnn_llvm_writelane(int(uint32_t(m >> 32)), c, high);
        }
        if (lane < 2 * STEPS) {
            bits_s[at * PITCH + ROWS * wave + i] = uint32_t(low) & low_mask;
            bits_s[(at + 1) * PITCH + ROWS * wave + i] = uint32_t(high) & high_mask;
        }
    }

    // Column terms.
    {
        int pop = 0;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (4 * s + 4 < kw) pop += __popc(w[s]);
            else pop += __popc(w[s] & (4 * s + g < kw - 1 ? ~0u : 4 * s + g == kw - 1 ? tmask : 0u));
        }
        pop = int(over_groups(uint32_t(pop), [](uint32_t a, uint32_t b) { return a + b; }));
        if (lane < 16) col_s[16 * wave + r] = fold_column_term(max(-K - 1, min(K + 1, thr)), K, 2 * pop);
    }
    __syncthreads();

    if (tile_n == 0)                                       // the packed input, once per row tile
        for (int i = threadIdx.x; i < BM * kw; i += T)
            if (row0 + (i & 15) < M) a_bits[int64_t(row0 + (i & 15)) * ld_a + (i >> 4)] = bits_s[(i >> 4) * PITCH + (i & 15)];

    v4f acc = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    int pop = 0;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const uint32_t a = bits_s[(4 * s + g) * PITCH + r];
        pop += __popc(a);
        // operands swapped: lane l holds columns 4g .. 4g + 3 of row r of the block
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(operand8(widen4_b(w[s])), operand8(widen4_a(a)), acc, 4, 4, 0, 0, 0, 0);
    }
    const float row_term = -0.5f * float(int(over_groups(uint32_t(pop), [](uint32_t a, uint32_t b) { return a + b; })));
    const float4 c = *reinterpret_cast<const float4*>(&col_s[16 * wave + 4 * g]);
    uint32_t neg = 0u;
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[3] + (c.w + row_term)), 31);
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[2] + (c.z + row_term)), 31);
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[1] + (c.y + row_term)), 31);
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(acc[0] + (c.x + row_term)), 31);
    const uint32_t bits = over_groups((~neg & 0xFu) << (4 * g), [](uint32_t a, uint32_t b) { return a | b; });
    const int left = N - 32 * word - 16 * half;
    const uint32_t live = left >= 16 ? 0xFFFFu : left <= 0 ? 0u : (1u << left) - 1u;
    // A wavefront's 16 columns are half a word.
    if (lane < BM && row0 + r < M && word < nw)
        reinterpret_cast<uint16_t*>(bn.out + int64_t(row0 + r) * bn.ld_out + word)[half] = uint16_t((bits ^ (flip >> (16 * half))) & live);
}

constexpr int kFewPieces = 13, kMostPieces = 16;           // 784 inputs (28 x 28), 1024; shorter rows compare and multiply zeros up to 13
// Whether one launch is faster than two: up to two workgroups per compute unit, where the reals that all column tiles read again cost
// less than a launch.  us replayed from a graph, two launches and one: 16 x 4096 x 784 (32 tiles) 4.8 and 3.9, 256 x 4096 x 784 (512) 5.95 and
// 5.4, 2000 x 512 x 100 (500) 6.2 and 5.3, 100 x 4096 x 1024 (224) 5.3 and 5.0; 400 x 4096 x 784 (800) 6.9 and 8.2.
constexpr int64_t kMaxTiles = 512;

static bool preferred(int64_t M, int64_t N, int64_t K, int64_t ldb) {
    return ldb < (1 << 24) && K > 32 && K <= 64 * kMostPieces && ceil_div(M, BM) * ceil_div(N, BN) <= kMaxTiles;
}

// Whether two matrices of 4-byte elements share memory, from their first element to their last.
struct Operand {
    const void* first;
    int64_t rows, cols, ld;
};
static bool overlap(const Operand& a, const Operand& b) {
    auto begin = [](const Operand& o) { return reinterpret_cast<uintptr_t>(o.first); };
    auto end = [&](const Operand& o) { return begin(o) + 4u * (uint64_t(o.rows - 1) * uint64_t(o.ld) + uint64_t(o.cols)); };
    return begin(a) < end(b) && begin(b) < end(a);
}

}  // namespace sign_gemm
}  // namespace bnn

extern "C" int bnn_sign_gemm_bn_sign_pack(const float* x, int64_t ldx, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                          const int32_t* thr, const uint32_t* flip_bits, uint32_t* a_bits, int64_t ld_a, uint32_t* out,
                                          int64_t ld_out, void* stream) {
    using namespace bnn;
    using namespace bnn::sign_gemm;
    const int64_t kw = ceil_div(K, 32), nw = ceil_div(N, 32);
    // What either call would refuse is left to it.
    const bool plain = M > 0 && N > 0 && M <= kMaxDim && N <= kMaxDim && K > 0 && K <= kMaxK && ldx >= K && ldb >= kw && ld_a >= kw &&
                       ld_out >= nw && x && B && thr && flip_bits && a_bits && out && aligned_to(x, 4) && aligned_to(B, 4) &&
                       aligned_to(thr, 4) && aligned_to(flip_bits, 4) && aligned_to(a_bits, 4) && aligned_to(out, 4);
    // So is what they read before they write it: here workgroups write results while others still read reals and filters.
    auto separate = [&] {
        const Operand bits{a_bits, M, kw, ld_a};
        return !overlap({x, M, K, ldx}, {out, M, nw, ld_out}) && !overlap(bits, {B, N, kw, ldb}) && !overlap(bits, {thr, 1, N, N}) &&
               !overlap(bits, {flip_bits, 1, nw, nw});
    };
    if (plain && preferred(M, N, K, ldb) && separate()) {
        const int64_t tiles_n = ceil_div(N, BN);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(unsigned(ceil_div(M, BM) * tiles_n)), dim3(T), 0, static_cast<hipStream_t>(stream), x, ldx, B,
                               ldb, int(M), int(N), int(K), int(tiles_n), fast_div(tiles_n), BnSignArgs{thr, flip_bits, out, ld_out},
                               a_bits, ld_a);
            return check_launch();
        };
        return K <= 64 * kFewPieces ? launch(sign_gemm_kernel<kFewPieces>) : launch(sign_gemm_kernel<kMostPieces>);
    }
    const int st = bnn_pack_sign(x, M, K, ldx, a_bits, ld_a, stream);
    return st != BNN_OK ? st : bnn_xnor_gemm_bn_sign_pack(a_bits, ld_a, B, ldb, M, N, K, thr, flip_bits, out, ld_out, stream);
}

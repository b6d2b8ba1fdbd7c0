// Bits-in, matrix-engine-inside kernels for the products of Alg. 4:
//
//   binary  a_k = XnorDotProduct(a^b_{k-1}, W^b_k), Sec. 4 Eq. (5)
//   conv    (CONV = true)     the binary product whose A rows are the receptive fields of a
//                             kh x kw convolution (3 x 3 in the paper's nets, Sec. 3.3), gathered
//                             from the packed NHWC input while the tile is staged (implicit
//                             GEMM: the im2col matrix is never written); taps outside the image
//                             are +1, i.e. all-ones words (zero padding through Eq. (1))
//
// Operands stay packed 32 per word in HBM and LDS (the 32x smaller footprint the
// paper argues for); only inside registers is each bit widened to a 4-bit float
// and fed to v_mfma_f32_32x32x64_f8f6f4, whose fp32 accumulation of small integers is exact below 2^24.
// With a, b in {0,1} standing for -1/+1:
//
//   sum_k (2a-1)(2b-1) = K - 2*popcount(A_m) - 2*popcount(B_n) + 4 * sum_k a*b
//
// so the product is the matrix-engine sum S plus row and column popcounts, which
// the staging threads gather for free while they copy the tile.
// Pad bits and words beyond K are zeroed at staging and therefore contribute to
// neither S nor the popcounts; tile rows beyond the matrix are computed on a copy
// of its last row and never stored.
//
// Widening: element k of a word lands in operand register k%4, nibble k/4, for
// both operands (the sum over k does not depend on its order).  The E2M1 codes
// 0b0001, 0b0010, 0b0100 are 0.5, 1.0, 2.0, so most registers are a bare mask of
// the word and only the product of the two sides has to be 1:
//   register   0                      1                  2                        3
//   A side     w & 0x1111.. (0.5)     w & 0x2222.. (1)   w & 0x4444.. (2)         (w>>2) & 0x2222.. (1)
//   B side     (w<<2) & 0x4444.. (2)  w & 0x2222.. (1)   (w>>2) & 0x1111.. (0.5)  (w>>2) & 0x2222.. (1)
// i.e. 5 vector-ALU operations per 32 elements on the A side, 6 on the B side.
//
// Workgroup = 256 threads = 2 x 2 wavefronts; a wavefront owns WM x WN blocks
// of 32 x 32 outputs (fp32 accumulators).  A advances 16 words per staged tile =
// 8 MFMA steps: lane (row r = l%32, half h = l/32) of a fragment owns words
// [8h, 8h+8) of its tile row, read with two ds_read_b128.
// Those 16 words are 512 consecutive bits of K; B is staged the same way.
// The tile is long enough that the global loads of the next tile, issued
// before the MFMA steps, have landed when they are staged.
#include "bnn_internal.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"

namespace bnn {

// TINY: rows of fewer than 4 words (K <= 96), which have no whole quad to load.
// ROWS: the int32 form stores rows through LDS (mfma_epilogue_rows).
template <int WM, int WN, bool FUSED, bool CONV, bool TINY, bool ROWS>
__global__ __launch_bounds__(256, WM >= 4 ? 2 : 3) void xnor_gemm_mfma_kernel(
    const uint32_t* __restrict__ A, int64_t lda, const uint32_t* __restrict__ B, int64_t ldb,
    int32_t* __restrict__ C, int64_t ldc, int M, int N, int K, TileMap tiles, BnSignArgs bn,
    ConvArgs cv) {
    constexpr int BM = 64 * WM, BN = 64 * WN;          // 2 x 2 wavefronts
    constexpr int PLANE_A = BM + 2, PLANE_B = BN + 2;  // 16-byte slots per quad plane (2 pad slots)
    constexpr int ST_ROWS = 256 / kMfmaKQ;             // rows covered by one staging pass
    constexpr int LOADS_A = BM / ST_ROWS;
    constexpr int LOADS_B = BN / ST_ROWS;
    static_assert(BM % ST_ROWS == 0 && BN % ST_ROWS == 0, "tile rows must divide among the staging threads");
    static_assert(kMfmaKQ == 4, "the row-popcount reduction below assumes 4 staging lanes per row");
    __shared__ uint4 lds[2 * kMfmaKQ * (PLANE_A + PLANE_B)];
    auto lds_a = [&](int buf) { return lds + buf * (kMfmaKQ * PLANE_A); };
    auto lds_b = [&](int buf) { return lds + 2 * kMfmaKQ * PLANE_A + buf * (kMfmaKQ * PLANE_B); };
    static_assert(sizeof(lds) >= 4 * kStoreScratch * sizeof(float), "the int32 rows leave through the operand buffers");
    __shared__ __attribute__((aligned(16))) int pop_a[BM];
    __shared__ __attribute__((aligned(16))) int pop_b[BN];
    __shared__ __attribute__((aligned(16))) float pop_af[FUSED ? BM : 4];   // row term of the float threshold
    __shared__ __attribute__((aligned(16))) int thr_s[FUSED ? BN : 1];                  // the tile's thresholds and flip words, fetched
    __shared__ uint32_t flip_s[FUSED ? BN / 32 : 1];       // before the K loop (read in the epilogue)
    // With the operands swapped the accumulator blocks are the transposes of the output blocks, which lets the fused
    // epilogue pack a row's bits inside a lane and the int32 one store 4 columns of a row at a time.
    constexpr bool SWAPPED = FUSED || ROWS;
    __shared__ float colfix_s[FUSED ? BN : 1];              // column term of the folded threshold

    int tile_m, tile_n;
    tile_of_block(blockIdx.x, tiles, tile_m, tile_n);
    const int row0 = tile_m * BM, col0 = tile_n * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fh = lane >> 5;
    const int kw = (K + 31) >> 5;
    const uint32_t tmask = tail_mask(K);
    const int n_ktiles = (kw + kMfmaKT - 1) / kMfmaKT;
    const int n_full_ktiles = (K >> 5) / kMfmaKT;      // K-tiles made only of complete, unmasked words

    const int st_q = tid % kMfmaKQ, st_r = tid / kMfmaKQ;
    // conv: per staged row the word offset of its image and its output pixel (oy << 16 | ox);
    // otherwise the row pointer.  fill_a: what staging writes for a fetched quad
    // (0 = the loaded words, 1 = all ones: tap outside the image, 2 = zeros: no such row or word).
    const uint32_t* pa[LOADS_A];
    uint32_t img_off[LOADS_A];
    int pix[LOADS_A];
    bool live_a[LOADS_A];
    int fill_a[LOADS_A];
#pragma unroll
    for (int l = 0; l < LOADS_A; ++l) {
        const int r = row0 + st_r + l * ST_ROWS;
        live_a[l] = r < M;
        fill_a[l] = 0;
        const int rc = min(r, M - 1);
        if (CONV) {
            const int ox = rc % cv.Wo, t = rc / cv.Wo;
            const int oy = t % cv.Ho, b = t / cv.Ho;
            img_off[l] = uint32_t(b) * uint32_t(cv.H * cv.W * cv.Cw);
            pix[l] = (oy << 16) | ox;
            pa[l] = A;
        } else {
            pa[l] = A + int64_t(rc) * lda;
        }
    }
    const uint32_t* pb[LOADS_B];
#pragma unroll
    for (int l = 0; l < LOADS_B; ++l) pb[l] = B + int64_t(min(col0 + st_r + l * ST_ROWS, N - 1)) * ldb;

    uint4 ra[LOADS_A], rb[LOADS_B];
    int cnt_a[LOADS_A], cnt_b[LOADS_B];
#pragma unroll
    for (int l = 0; l < LOADS_A; ++l) cnt_a[l] = 0;
#pragma unroll
    for (int l = 0; l < LOADS_B; ++l) cnt_b[l] = 0;

    // conv: quad `quad` of a receptive field is 4 channel words of one tap; the load address is
    // clamped into the image and the choice between the loaded words, all-ones and zeros is made
    // at staging, so the loads themselves are unconditional.
    auto fetch_conv = [&](int quad) {
        const int w0 = min(quad * 4, kw - 4);
        const int tap = w0 / cv.Cw, cw = w0 - tap * cv.Cw;
        const int ky = tap / cv.kw, kx = tap - ky * cv.kw;
#pragma unroll
        for (int l = 0; l < LOADS_A; ++l) {
            const int y = (pix[l] >> 16) * cv.stride - cv.pad + ky;
            const int x = (pix[l] & 0xFFFF) * cv.stride - cv.pad + kx;
            const bool inside = y >= 0 && y < cv.H && x >= 0 && x < cv.W;
            const int yc = min(max(y, 0), cv.H - 1), xc = min(max(x, 0), cv.W - 1);
            ra[l] = *reinterpret_cast<const uint4*>(A + img_off[l] + uint32_t((yc * cv.W + xc) * cv.Cw + cw));
            fill_a[l] = (!live_a[l] || quad * 4 >= kw) ? 2 : (inside ? 0 : 1);
        }
    };
    // The loads carry no control flow: a branch around them makes the compiler wait for them where the branches
    // meet, which exposes the whole memory latency in every iteration (and checked loads in the last K-tile are a chain
    // of such waits).  What is not a whole quad is put right when it is staged.
    auto load_words = [&](const uint32_t* row, int quad) {
        if (!TINY) return load_row_quad(row, quad, kw);
        return make_uint4(row[0], row[min(1, kw - 1)], row[min(2, kw - 1)], 0u);      // one K-tile, quad 0 only
    };
    auto place_words = [&](uint4 v, int quad) {
        return TINY ? mask_row_quad(v, kw - 4 * quad, tmask) : place_row_quad(v, quad, kw, tmask);
    };
    auto fetch = [&](int kt) {
        const int quad = kt * kMfmaKQ + st_q;
        if (CONV) {
            fetch_conv(quad);
        } else {
#pragma unroll
            for (int l = 0; l < LOADS_A; ++l) ra[l] = load_words(pa[l], quad);
        }
#pragma unroll
        for (int l = 0; l < LOADS_B; ++l) rb[l] = load_words(pb[l], quad);
    };
    // Writes the fetched words to LDS and adds their set bits to this thread's row sums.
    auto stage = [&](int kt, int buf) {
        if (kt >= n_full_ktiles) {
            const int quad = kt * kMfmaKQ + st_q;
#pragma unroll
            for (int l = 0; l < LOADS_A; ++l)
                if (!CONV) ra[l] = place_words(ra[l], quad);
#pragma unroll
            for (int l = 0; l < LOADS_B; ++l) rb[l] = place_words(rb[l], quad);
        }
#pragma unroll
        for (int l = 0; l < LOADS_A; ++l) {
            // Rows beyond the matrix hold a copy of its last row (clamped load): their sums and
            // outputs are computed and never stored, so nothing has to be zeroed here.
            uint4 v = ra[l];
            if (CONV) {
                const bool keep = fill_a[l] == 0;
                const uint32_t fill = fill_a[l] == 1 ? ~0u : 0u;
                v = make_uint4(keep ? ra[l].x : fill, keep ? ra[l].y : fill, keep ? ra[l].z : fill,
                               keep ? ra[l].w : fill);
            }
            cnt_a[l] += popc4(v);
            lds_a(buf)[st_q * PLANE_A + st_r + l * ST_ROWS] = v;
        }
#pragma unroll
        for (int l = 0; l < LOADS_B; ++l) {
            const uint4 v = rb[l];
            cnt_b[l] += popc4(v);
            lds_b(buf)[st_q * PLANE_B + st_r + l * ST_ROWS] = v;
        }
    };

    v16f acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    if (FUSED) {
        // No result exceeds lim in magnitude, so clamping a threshold to [-lim, lim] changes no output
        // bit and keeps the bounds the epilogue derives from it inside int32 for any caller-given value.
        const int lim = K + 1;
        if (tid < BN) thr_s[tid] = col0 + tid < N ? max(-lim, min(lim, bn.thr[col0 + tid])) : 0;
        if (tid < BN / 32) flip_s[tid] = col0 + 32 * tid < N ? bn.flip_bits[(col0 >> 5) + tid] : 0u;
    }
    if (n_ktiles > 0) {
        fetch(0);
        stage(0, 0);
    }
    __syncthreads();

    for (int kt = 0; kt < n_ktiles; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < n_ktiles) fetch(kt + 1);

        // The lane's 8 words are quads 2*fh and 2*fh+1 of its tile row; each quad feeds 4 steps.
#pragma unroll
        for (int hq = 0; hq < 2; ++hq) {
            uint4 aw[WM], bw[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) aw[i] = lds_a(buf)[(2 * fh + hq) * PLANE_A + wm * 32 * WM + i * 32 + fr];
#pragma unroll
            for (int j = 0; j < WN; ++j) bw[j] = lds_b(buf)[(2 * fh + hq) * PLANE_B + wn * 32 * WN + j * 32 + fr];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                v8i fa[WM], fb[WN];
#pragma unroll
                for (int i = 0; i < WM; ++i) fa[i] = widen_fp4_a(quad_word(aw[i], s));
#pragma unroll
                for (int j = 0; j < WN; ++j) fb[j] = widen_fp4_b(quad_word(bw[j], s));
                // Both block scales are 1: literal zero scale operands make the compiler emit the
                // plain v_mfma_f32_32x32x64_f8f6f4 (unit scale, half the encoding size and no
                // scale-register reads) instead of the scaled pair.
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        if (SWAPPED)
                            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                fb[j], fa[i], acc[i][j], 4 /* fp4 */, 4 /* fp4 */, 0, 0, 0, 0);
                        else
                            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                fa[i], fb[j], acc[i][j], 4 /* A: fp4 */, 4 /* B: fp4 */, 0, 0, 0, 0);
                    }
            }
        }

        // Ordering pin: without it the compiler hoists the staging of the next tile (and with it
        // the wait for the global loads issued at the top of this iteration) above the MFMA steps,
        // which exposes the whole memory latency every iteration.  The empty asm "uses" the
        // accumulators, so all MFMAs precede it, and clobbers memory, so the LDS stores follow it.
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) asm volatile("" : "+v"(acc[i][j]) : : "memory");

        if (kt + 1 < n_ktiles) stage(kt + 1, buf ^ 1);
        __syncthreads();
    }

    // Row sums: the kMfmaKQ threads that staged the quads of one row are neighbouring lanes.
    // pop_a / pop_b hold 2*popcount.
#pragma unroll
    for (int l = 0; l < LOADS_A; ++l) {
        int c = cnt_a[l];
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        if (st_q == 0) {
            pop_a[st_r + l * ST_ROWS] = 2 * c;
            if (FUSED) pop_af[st_r + l * ST_ROWS] = 0.5f * float(c);       // 2pa/4
        }
    }
#pragma unroll
    for (int l = 0; l < LOADS_B; ++l) {
        int c = cnt_b[l];
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);
        if (st_q == 0) {
            pop_b[st_r + l * ST_ROWS] = 2 * c;
            if (FUSED) colfix_s[st_r + l * ST_ROWS] = fold_column_term(thr_s[st_r + l * ST_ROWS], K, 2 * c);
        }
    }
    __syncthreads();

    if constexpr (FUSED)
        mfma_epilogue_bits<WM, WN>(acc, pop_a, pop_af, pop_b, thr_s, flip_s, colfix_s, bn, M, N, K, row0, col0, wm, wn,
                                   fr, fh);
    else if constexpr (ROWS)
        mfma_epilogue_rows<WM, WN>(acc, reinterpret_cast<float*>(lds) + wave * kStoreScratch, pop_a, pop_b, C, ldc, M, N, K,
                                   row0, col0, wm, wn, lane);
    else
        mfma_epilogue<WM, WN>(acc, pop_a, pop_b, C, ldc, M, N, K, row0, col0, wm, wn, fr, fh);
}

template <int WM, bool FUSED, bool CONV, bool TINY = false>
static int launch_mfma(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                       int64_t M, int64_t N, int64_t K, BnSignArgs bn, ConvArgs cv, void* stream) {
    constexpr int WN = 2;
    const int64_t tiles_m = ceil_div(M, 64 * WM), tiles_n = ceil_div(N, 64 * WN);
    if (tiles_m * tiles_n > kMaxDim) return BNN_ERR_UNSUPPORTED;
    const dim3 grid{unsigned(tiles_m * tiles_n)};
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream), A, lda, B, ldb, C, ldc, int(M),
                           int(N), int(K), tile_map(tiles_m, tiles_n), bn, cv);
    };
    // The 64 x 128 tiles are for grids that are over before stores queue up: straight from the accumulators
    // (834 x 2414 x 1343 6.9 vs 7.4 us through LDS).
    if (!FUSED && WM >= 2 && wants_row_stores(C, ldc))
        launch(xnor_gemm_mfma_kernel<WM, WN, FUSED, CONV, TINY, !FUSED && (WM >= 2)>);
    else
        launch(xnor_gemm_mfma_kernel<WM, WN, FUSED, CONV, TINY, false>);
    return check_launch();
}

// 128 x 128 tiles (2 x 2 blocks per wavefront, 3 workgroups per compute unit): more, smaller
// workgroups for products whose K is short or whose 256 x 128 grid would leave units idle.  Grids
// of fewer than 256 such tiles take 64 x 128 tiles (1 x 2 blocks per wavefront) instead: with so few
// workgroups every one of them waits on its own K-tile loads, and twice as many share that wait
// (256 x 1024 x 8192 fused: 17.3 -> 13.0 us, 512 x 4096 x 4096: 10.3 -> 8.2 us).
static bool wants_half_tiles(int64_t M, int64_t N) { return ceil_div(M, 128) * ceil_div(N, 128) < 256; }

// Rows of fewer than 4 words (K <= 96).  The fused form follows the rule above (1000000 x 128 x 64 42 us on 128 x 128 tiles,
// 58 on 64 x 128; 10000 x 4096 x 64 16.6 and 21.5; 512 x 512 x 96 4.3 and 3.9); the int32 form, all stores, is faster on the
// smaller tiles whatever the grid (10000 x 4096 x 64 26.6 and 28.8, 50176 x 64 x 32 6.3 and 6.7), while one launch holds them.
template <bool FUSED>
static int launch_tiny(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                       int64_t N, int64_t K, BnSignArgs bn, void* stream) {
    const bool small = FUSED ? wants_half_tiles(M, N) : ceil_div(M, 64) * ceil_div(N, 128) <= max_blocks(256);
    return small ? launch_mfma<1, FUSED, false, true>(A, lda, B, ldb, C, ldc, M, N, K, bn, ConvArgs{}, stream)
                 : launch_mfma<2, FUSED, false, true>(A, lda, B, ldb, C, ldc, M, N, K, bn, ConvArgs{}, stream);
}

// Entry points used by the dispatchers.  The callers have validated the arguments.
bool mfma_path_supports(int64_t K) { return K <= kMfmaMaxAcc; }

int launch_xnor_gemm_mfma(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C,
                          int64_t ldc, int64_t M, int64_t N, int64_t K, void* stream) {
    if (K <= 96) return launch_tiny<false>(A, lda, B, ldb, C, ldc, M, N, K, BnSignArgs{}, stream);
    return launch_mfma<4, false, false>(A, lda, B, ldb, C, ldc, M, N, K, BnSignArgs{}, ConvArgs{}, stream);
}

int launch_xnor_gemm_mfma_fused(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int64_t M,
                                int64_t N, int64_t K, BnSignArgs bn, void* stream) {
    if (K <= 96) return launch_tiny<true>(A, lda, B, ldb, nullptr, 0, M, N, K, bn, stream);
    return launch_mfma<4, true, false>(A, lda, B, ldb, nullptr, 0, M, N, K, bn, ConvArgs{}, stream);
}

int launch_xnor_gemm_mfma128(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int32_t* C,
                             int64_t ldc, int64_t M, int64_t N, int64_t K, void* stream) {
    if (K <= 96) return launch_tiny<false>(A, lda, B, ldb, C, ldc, M, N, K, BnSignArgs{}, stream);
    if (wants_half_tiles(M, N))
        return launch_mfma<1, false, false>(A, lda, B, ldb, C, ldc, M, N, K, BnSignArgs{}, ConvArgs{}, stream);
    return launch_mfma<2, false, false>(A, lda, B, ldb, C, ldc, M, N, K, BnSignArgs{}, ConvArgs{}, stream);
}

int launch_xnor_gemm_mfma128_fused(const uint32_t* A, int64_t lda, const uint32_t* B, int64_t ldb, int64_t M,
                                   int64_t N, int64_t K, BnSignArgs bn, void* stream) {
    if (K <= 96) return launch_tiny<true>(A, lda, B, ldb, nullptr, 0, M, N, K, bn, stream);
    if (wants_half_tiles(M, N))
        return launch_mfma<1, true, false>(A, lda, B, ldb, nullptr, 0, M, N, K, bn, ConvArgs{}, stream);
    return launch_mfma<2, true, false>(A, lda, B, ldb, nullptr, 0, M, N, K, bn, ConvArgs{}, stream);
}

// Implicit-GEMM convolution: `in` is the packed NHWC input, B the packed filters [N][kh*kw*Cw].
// The conv kernel reads A in unaligned-tolerant fashion only through 16-byte quads, so the
// caller guarantees in is 16-byte aligned and Cw % 4 == 0.
// Tile choice as for the plain product: 256 x 128 when that grid fills the chip's 512 workgroup
// slots, else 128 x 128 (three workgroups per compute unit).
static bool conv_wants_small_tiles(int64_t M, int64_t N) { return ceil_div(M, 256) * ceil_div(N, 128) < 512; }

// Short receptive fields (K <= 1152: 3 x 3 over 128 channels) go to the conv mode of the short-K
// organisation (xnor_gemm_mfma_shortk.hip).
bool conv_shortk_supports(const uint32_t* B, int64_t ldb, int64_t K);
int launch_conv_mfma_shortk(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                            int64_t N, int64_t K, ConvArgs cv, void* stream);
int launch_conv_mfma_shortk_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N,
                                  int64_t K, BnSignArgs bn, ConvArgs cv, void* stream);

// Convolutions whose tiles' input patch fits keep it in LDS (conv_patch.hip); its launchers return
// BNN_ERR_UNSUPPORTED for every other layer.
int launch_conv_patch(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                      int64_t N, int64_t K, ConvArgs cv, void* stream);
int launch_conv_patch_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                            BnSignArgs bn, ConvArgs cv, void* stream);

int launch_conv_mfma(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                     int64_t N, int64_t K, ConvArgs cv, void* stream) {
    const int st = launch_conv_patch(in, B, ldb, C, ldc, M, N, K, cv, stream);
    if (st != BNN_ERR_UNSUPPORTED) return st;
    if (cv.Cw % 4 != 0) return BNN_ERR_UNSUPPORTED;     // the gathering loaders move whole 16-byte channel quads
    if (conv_shortk_supports(B, ldb, K)) return launch_conv_mfma_shortk(in, B, ldb, C, ldc, M, N, K, cv, stream);
    if (conv_wants_small_tiles(M, N))
        return launch_mfma<2, false, true>(in, 0, B, ldb, C, ldc, M, N, K, BnSignArgs{}, cv, stream);
    return launch_mfma<4, false, true>(in, 0, B, ldb, C, ldc, M, N, K, BnSignArgs{}, cv, stream);
}

int launch_conv_mfma_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                           BnSignArgs bn, ConvArgs cv, void* stream) {
    const int st = launch_conv_patch_fused(in, B, ldb, M, N, K, bn, cv, stream);
    if (st != BNN_ERR_UNSUPPORTED) return st;
    if (cv.Cw % 4 != 0) return BNN_ERR_UNSUPPORTED;
    if (conv_shortk_supports(B, ldb, K)) return launch_conv_mfma_shortk_fused(in, B, ldb, M, N, K, bn, cv, stream);
    if (conv_wants_small_tiles(M, N))
        return launch_mfma<2, true, true>(in, 0, B, ldb, nullptr, 0, M, N, K, bn, cv, stream);
    return launch_mfma<4, true, true>(in, 0, B, ldb, nullptr, 0, M, N, K, bn, cv, stream);
}

}  // namespace bnn

// Binary convolution (the 3 x 3, pad 1 layers of the paper's ConvNets, Sec. 3.3, and any other geometry whose input
// patch fits) with the input patch of a tile resident in LDS.
//
// The GEMM view of the layer is C[pixel][filter] = XnorDotProduct(receptive field, filter) (Alg. 4)
// with K = kh*kw*Cin.  The receptive fields of neighbouring pixels overlap kh*kw-fold, so instead
// of staging every K-tile of the (implicit) im2col matrix, a workgroup loads each input pixel its
// tile needs ONCE: a tile is BM consecutive output pixels, its patch the input rows under their
// windows with a halo of `pad` pixels all around, kept in LDS for the workgroup's life.  Halo cells
// outside the image hold all-ones words (+1, zero padding through Eq. (1)).  The A operand of an MFMA step for tap (ky, kx) is then a plain LDS read at
//     slot(pixel) + ky * PW + kx          (PW = W + 2*pad, patch row pitch in pixels)
// with no per-tap bounds logic, and only the filters (B) stream through LDS K-tile by K-tile.
// Arithmetic, widening, fix-up and epilogues are those of xnor_gemm_mfma.hip; the row popcounts are
// sums of per-pixel popcounts over the taps.
//
// Patch layout: planes [channel quad cq][half h] of 8-byte slots, slot s = words 4*cq + 2*h, +1 of
// patch pixel s; lanes of an operand read consecutive pixels, hence consecutive slots.
// B K-tile layout: planes [quad][half] of 8-byte slots, as in the short-K kernel.
//
// Pooled layers (POOL = true): the paper's ConvNets max-pool the pre-activations 2 x 2 between a
// convolution and its BatchNorm + Sign.  Sign(BatchNorm(.)) is monotone per channel, so the pooled
// output bit is the OR of the window's four output bits where the folded flip bit is 0 and their
// AND where it is 1.  The rows of a pooled layer are its pixels window by window (row 4 * window + 2 * dy + dx), so a
// window is four neighbouring lanes of one accumulator block whatever the size of the image, and only the pooled words are
// stored.  Nothing but the cell of a row depends on that order.
//
// Channel counts that are multiples of 32 but not of 128 (WORDS = true; the 64-channel block of the
// half-width SVHN net of Sec. 2.3): a tap is then not a whole number of 16-byte quads, so the patch is
// kept as planes [channel word][slot] of single words, and the K-word that lane half h consumes at step
// (quad q, s), word 4q + 2h + s of the receptive field, is looked up in a small LDS table that maps
// a K-word to (channel word plane, tap offset).  Filter words beyond the receptive field's last word
// are zeroed at staging.  Everything else is shared.
//
// The padded images (pad rows and columns all around) follow each other without a gap, so the patch of ANY run of BM
// consecutive output pixels is a run of their rows: kernel size, stride, padding and image size are free, tiles may start
// and end inside image rows and span images (the halo rows between two images are then part of the patch).
//
// What this kernel takes (the launcher checks; everything else goes to the gathering kernels): filters 16-byte aligned
// with ldb % 4 == 0, a patch within kPatchMaxBytes of LDS, and Cin % 128 == 0 - or Cin % 32 == 0 for same-size stride-1
// layers whose tiles are whole image rows or images, with a receptive field of at most kResidentKTiles * 512 bits.
// Some layers that would fit are faster gathered (better_gathered).
// Fused 3 x 3 layers, and others that fill the chip in strips, leave before these tiles are chosen (conv_strip.hip).
// Against gathering the receptive fields K-tile by K-tile, fused, on layers that now run in strips: 128 images of 28 x 28, 128 -> 256
// channels 22.4 -> 18.9 us, 200 of 13 x 13, 128 -> 396 17.8 -> 13.9, 100 of 14 x 14, 256 -> 256 13.4 -> 11.7, 256 of 32 x 32, 128 -> 256
// at stride 2 15.5 -> 13.0, 128 of 56 x 56, 128 -> 128 37.0 -> 31.6; as int32, which stays here, 128 of 28 x 28, 128 -> 256 30.1 -> 25.6.
#include "bnn_internal.h"
#include "conv_patch_geometry.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"

namespace bnn {

// Fused layers in strips (conv_strip.hip): BNN_ERR_UNSUPPORTED, with nothing launched, for those it leaves to this kernel.
int launch_conv_strip_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                            BnSignArgs bn, ConvArgs cv, bool pool, ConvUse use, void* stream);

constexpr int kPatchMaxBytes = 40 * 1024;

// Word offset of the K-word table behind the word-granular patch ([Cw][slots] words + slots pixel popcounts).
__host__ __device__ inline size_t words_patch_koff_offset(int Cw, int slots) {
    return (size_t(Cw + 1) * size_t(slots) + 1) & ~size_t(1);
}

// RES > 0: the filters' whole K extent (at most RES K-tiles of 4 quads) is staged once, next to the patch, and the K
// loop runs without a barrier; RES = 0: B streams through two K-tile buffers.  kResidentKTiles fit beside the patches of
// two or three workgroups.  kResidentKTilesAlone (3 x 3 over 512 channels) fill a compute unit by themselves: for grids
// that give a compute unit one workgroup at most, where every K-tile streamed is a memory round trip that nothing else
// covers (52 images of 8 x 8, 512 -> 512 pooled 13.9 -> 12.8 us, 20 of 16 x 16, 384 -> 256 11.5 -> 10.7).
constexpr int kResidentKTiles = 5, kResidentKTilesAlone = 9;
constexpr int64_t kLoneGrid = 224;        // workgroups that leave no compute unit with two
constexpr int64_t kComputeUnits = 256;

// KS = 2: eight wavefronts, the second four taking the second half of K of the same tile; their sums join the first
// four's in LDS.  For grids that give a compute unit one workgroup at most: a wavefront alone on its SIMD waits for every
// LDS read, widening and product in turn (16 images of 8 x 8, 512 -> 512 12.6 -> 10.4 us, 20 of 16 x 16, 256 -> 256 8.1 ->
// 7.6).  Not for 128-pixel tiles with a short K, where joining the sums costs what it saves (26 of 32 x 32, 128 -> 128
// 6.7 -> 7.2).
template <int WM, bool FUSED, bool POOL, int RES, bool WORDS, int KS>
__global__ __launch_bounds__(256 * KS, KS > 1 ? 2 : RES > kResidentKTiles ? 1 : WM >= 4 ? 2 : 3) void conv_patch_mfma_kernel(
    const uint32_t* __restrict__ in, const uint32_t* __restrict__ B, int64_t ldb, int32_t* __restrict__ C,
    int64_t ldc, int M, int N, int K, TileMap tiles, BnSignArgs bn, ConvArgs cv, PatchGeom pg,
    int n_images) {
    constexpr int WN = 2, BM = 64 * WM, BN = 64 * WN;
    constexpr int PLANE_B = BN + 2;                     // 8-byte slots per B plane (2 pad slots)
    constexpr int T = 256 * KS;
    constexpr int ST_ROWS = T / 4;                      // filter rows per staging pass (4 threads per row)
    static_assert(KS == 1 || (RES > 0 && WM <= 2), "K is split over wavefronts for small tiles with resident filters");
    constexpr int LOADS_B = BN / ST_ROWS;
    constexpr bool BRES = RES > 0;
    static_assert(!WORDS || BRES, "the word-granular patch is built for resident filters only");
    extern __shared__ __attribute__((aligned(16))) uint2 patch[];                    // [cqn][2][slots], int pix_pop[slots], resident B tiles
                                                        // WORDS: uint32 [Cw][slots], pix_pop, int koff[4*kq], B tiles
    __shared__ uint2 lds_b_stream[BRES ? 1 : 2 * 8 * PLANE_B];
    __shared__ __attribute__((aligned(16))) int pop_a[BM];
    __shared__ __attribute__((aligned(16))) float pop_af[FUSED ? BM : 4];
    __shared__ __attribute__((aligned(16))) int pop_b[BN];
    __shared__ __attribute__((aligned(16))) int thr_s[FUSED ? BN : 1];
    __shared__ uint32_t flip_s[FUSED ? BN / 32 : 1];
    __shared__ float colfix_s[FUSED ? BN : 1];
    __shared__ int slot_s[BM];
    uint32_t* patchw = reinterpret_cast<uint32_t*>(patch);
    int* pix_pop = WORDS ? reinterpret_cast<int*>(patchw + size_t(cv.Cw) * pg.slots)
                         : reinterpret_cast<int*>(patch + size_t(2) * pg.cqn * pg.slots);
    // WORDS: K-word -> plane and tap offset into patchw, read two at a time (hence the even word offset)
    const size_t koff_at = words_patch_koff_offset(cv.Cw, pg.slots);
    int* koff_s = reinterpret_cast<int*>(patchw) + koff_at;
    uint2* lds_b = !BRES ? lds_b_stream                 // [buffer][8 planes]
                   : WORDS ? patch + (koff_at + size_t(4) * pg.kq) / 2
                           : patch + size_t(2) * pg.cqn * pg.slots + (pg.slots + 1) / 2;

    int tile_m, tile_n;
    tile_of_block(blockIdx.x, tiles, tile_m, tile_n);
    const int row0 = tile_m * BM, col0 = tile_n * BN;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = KS > 1 ? (wave >> 1) & 1 : wave >> 1, wn = wave & 1, kg = KS > 1 ? wave >> 2 : 0;
    const int fr = lane & 31, fh = lane >> 5;

    // ---- B staging: K-tiles of 4 quads, as planes [quad][half] ---------------------------------
    const int st_q = tid & 3, st_r = tid >> 2;
    const uint32_t* pb[LOADS_B];
#pragma unroll
    for (int l = 0; l < LOADS_B; ++l) pb[l] = B + int64_t(min(col0 + st_r + l * ST_ROWS, N - 1)) * ldb;
    uint4 rb[LOADS_B];
    int cnt_b[LOADS_B];
#pragma unroll
    for (int l = 0; l < LOADS_B; ++l) cnt_b[l] = 0;
    const int n_ktiles = (pg.kq + 3) >> 2;
    auto fetch_b = [&](int kt) {
        const int quad = min(4 * kt + st_q, pg.kq - 1);           // clamped; zeroed at staging if past the row
#pragma unroll
        for (int l = 0; l < LOADS_B; ++l) rb[l] = *reinterpret_cast<const uint4*>(pb[l] + 4 * quad);
    };
    auto stage_b = [&](int kt, int buf) {
        const bool live = 4 * kt + st_q < pg.kq;
#pragma unroll
        for (int l = 0; l < LOADS_B; ++l) {
            uint4 v = zero_unless(live, rb[l]);
            if (WORDS) {                                // words of the quad beyond the receptive field's last one
                const int left = pg.kwords - 4 * (4 * kt + st_q);
                if (left < 4) v.w = 0u;
                if (left < 3) v.z = 0u;
                if (left < 2) v.y = 0u;
            }
            cnt_b[l] += popc4(v);
            lds_b[(8 * buf + 2 * st_q) * PLANE_B + st_r + l * ST_ROWS] = make_uint2(v.x, v.y);
            lds_b[(8 * buf + 2 * st_q + 1) * PLANE_B + st_r + l * ST_ROWS] = make_uint2(v.z, v.w);
        }
    };

    // The tile's first output pixel is (image b0, row y0, ...); the patch starts at the padded row its window starts at,
    // row patch_row0 of image b0 (rows are counted from there: all images' together may be more than 2^31).
    // Output pixel r of the tile as a patch cell: the divisions are done once per pixel here, not once per use.
    // POOL: cv.Wo, cv.Ho and the divisions are those of the map of windows (pooled_units).
    constexpr int PF = POOL ? 2 : 1;
    const int row_first = pg.by_wo(POOL ? row0 >> 2 : row0), b0 = pg.by_ho(row_first), y0 = row_first - b0 * cv.Ho;
    const int patch_row0 = PF * y0 * cv.stride;
    // Cells to load: up to the end of the last pixel's window where that may be far fewer than the tile that needs most has.
    int slots_here = pg.slots;
    if (pg.trim) {
        const int last = min(row0 + BM, M) - 1;
        const int row_last = pg.by_wo(POOL ? last >> 2 : last), b_last = pg.by_ho(row_last), y_last = row_last - b_last * cv.Ho;
        slots_here = ((b_last - b0) * pg.img_rows + PF * (y_last - y0) * cv.stride + (PF - 1) * cv.stride + cv.kh) * pg.pw;
    }
    if (tid < BM) {
        const int m = min(row0 + tid, M - 1), unit = POOL ? m >> 2 : m;
        const int t = pg.by_wo(unit), x = unit - t * cv.Wo;
        const int b = pg.by_ho(t), y = t - b * cv.Ho;
        const int dy = POOL ? (m >> 1) & 1 : 0, dx = POOL ? m & 1 : 0;
        slot_s[tid] = ((b - b0) * pg.img_rows + (PF * y + dy) * cv.stride - patch_row0) * pg.pw + (PF * x + dx) * cv.stride;
    }
    // Thresholds and flip words go to registers here and to LDS after the patch loads have been issued: every
    // global load of the prologue (these, the filters, the patch) is in flight before the first one is waited for.
    int thr_reg = 0;
    uint32_t flip_reg = 0u;
    if (FUSED) {
        if (tid < BN && col0 + tid < N) thr_reg = bn.thr[col0 + tid];
        if (tid < BN / 32 && col0 + 32 * tid < N) flip_reg = bn.flip_bits[(col0 >> 5) + tid];
    }
    // The filter loads are issued first, so that they are in flight while the patch is addressed and loaded.
    uint4 all_b[BRES ? RES : 1][LOADS_B];
    if (BRES) {
#pragma unroll
        for (int kt = 0; kt < RES; ++kt)
            if (kt < n_ktiles) {
                fetch_b(kt);
#pragma unroll
                for (int l = 0; l < LOADS_B; ++l) all_b[kt][l] = rb[l];
            }
    } else {
        fetch_b(0);
    }

    // ---- patch: every slot once ------------------------------------------------------------
    // Slot s is column s % pw of row patch_row0 + s / pw of the padded images from b0 on, which follow each other without a
    // gap.
    const uint32_t* in_b0 = in + size_t(b0) * uint32_t(cv.H * cv.W) * uint32_t(cv.Cw);
    const int images_left = n_images - b0;
    if (WORDS || !FUSED) {
        // Slot by slot (the word-granular patch, and the int32 form, whose epilogue leaves no registers for
        // more loads in flight).
        for (int s = tid; s < slots_here; s += T) {
            const int py = pg.by_pw(s), px = s - py * pg.pw;
            const int b = pg.by_img_rows(patch_row0 + py), y = patch_row0 + py - b * pg.img_rows - cv.pad, x = px - cv.pad;
            const bool inside = b < images_left && y >= 0 && y < cv.H && x >= 0 && x < cv.W;
            const uint32_t pix = inside ? uint32_t((b * cv.H + y) * cv.W + x) : 0u;
            const uint32_t* p = in_b0 + size_t(pix) * uint32_t(cv.Cw);
            int pop = 0;
            if (WORDS) {
                for (int cw = 0; cw < cv.Cw; ++cw) {
                    const uint32_t v = inside ? p[cw] : ~0u;
                    patchw[cw * pg.slots + s] = v;
                    pop += __popc(v);
                }
            } else {
                for (int cq = 0; cq < pg.cqn; ++cq) {
                    uint4 v = *reinterpret_cast<const uint4*>(p + 4 * cq);
                    if (!inside) v = make_uint4(~0u, ~0u, ~0u, ~0u);
                    patch[(2 * cq) * pg.slots + s] = make_uint2(v.x, v.y);
                    patch[(2 * cq + 1) * pg.slots + s] = make_uint2(v.z, v.w);
                    pop += popc4(v);
                }
            }
            pix_pop[s] = pop;
        }
    } else {
        // Two slots per thread and pass, up to four channel quads of each at a time: all (up to eight) loads
        // of a pass are issued before the first LDS write waits for one.  Slots that do not exist and cells
        // outside the image load input pixel 0 (a valid address) and are not written / written as all ones.
        constexpr int kSlotsPerPass = 2, kQuadsPerPass = 4;
        for (int s_base = 0; s_base < slots_here; s_base += kSlotsPerPass * T) {
            const uint32_t* p[kSlotsPerPass];
            bool live[kSlotsPerPass], inside[kSlotsPerPass];
            int pop[kSlotsPerPass];
#pragma unroll
            for (int u = 0; u < kSlotsPerPass; ++u) {
                const int s = s_base + u * T + tid;
                live[u] = s < slots_here;
                const int py = pg.by_pw(s), px = s - py * pg.pw;
                const int b = pg.by_img_rows(patch_row0 + py), y = patch_row0 + py - b * pg.img_rows - cv.pad, x = px - cv.pad;
                inside[u] = live[u] && b < images_left && y >= 0 && y < cv.H && x >= 0 && x < cv.W;
                const uint32_t pix = inside[u] ? uint32_t((b * cv.H + y) * cv.W + x) : 0u;
                p[u] = in_b0 + size_t(pix) * uint32_t(cv.Cw);
                pop[u] = 0;
            }
            for (int cq0 = 0; cq0 < pg.cqn; cq0 += kQuadsPerPass) {
                uint4 v[kSlotsPerPass][kQuadsPerPass];
#pragma unroll
                for (int u = 0; u < kSlotsPerPass; ++u)
#pragma unroll
                    for (int c = 0; c < kQuadsPerPass; ++c)
                        if (cq0 + c < pg.cqn) v[u][c] = *reinterpret_cast<const uint4*>(p[u] + 4 * (cq0 + c));
#pragma unroll
                for (int u = 0; u < kSlotsPerPass; ++u) {
                    const int s = s_base + u * T + tid;
#pragma unroll
                    for (int c = 0; c < kQuadsPerPass; ++c)
                        if (cq0 + c < pg.cqn) {
                            const uint4 w = inside[u] ? v[u][c] : make_uint4(~0u, ~0u, ~0u, ~0u);
                            if (live[u]) {
                                patch[(2 * (cq0 + c)) * pg.slots + s] = make_uint2(w.x, w.y);
                                patch[(2 * (cq0 + c) + 1) * pg.slots + s] = make_uint2(w.z, w.w);
                            }
                            pop[u] += popc4(w);
                        }
                }
            }
#pragma unroll
            for (int u = 0; u < kSlotsPerPass; ++u)
                if (live[u]) pix_pop[s_base + u * T + tid] = pop[u];
        }
    }
    if (FUSED) {
        if (tid < BN) thr_s[tid] = max(-K - 1, min(K + 1, thr_reg));
        if (tid < BN / 32) flip_s[tid] = flip_reg;
    }
    if (WORDS) {
        // K-word kwi of a receptive field = channel word kwi % Cw of tap kwi / Cw; words past the field's
        // end point at a valid cell (their filter words are zero).
        for (int kwi = tid; kwi < 4 * pg.kq; kwi += T) {
            int off = 0;
            if (kwi < pg.kwords) {
                const int tap = kwi / cv.Cw, cw = kwi - tap * cv.Cw;
                const int ty = tap / cv.kw, tx = tap - ty * cv.kw;
                off = cw * pg.slots + ty * pg.pw + tx;
            }
            koff_s[kwi] = off;
        }
    }

    if (BRES) {
#pragma unroll
        for (int kt = 0; kt < RES; ++kt)
            if (kt < n_ktiles) {
#pragma unroll
                for (int l = 0; l < LOADS_B; ++l) rb[l] = all_b[kt][l];
                stage_b(kt, kt);
            }
    } else {
        stage_b(0, 0);
    }
    __syncthreads();                                    // patch, pixel popcounts and the first (or every) B tile are in LDS

    // Row popcounts: sum of the pixel popcounts under the kh x kw window (read before the epilogue,
    // which follows at least one more barrier).  Nine taps at a time, their loads in flight together and their offsets
    // stepped in scalar registers: one tap after the other, nine round trips to LDS stood between staging and the first
    // product (of the 31200 cycles of a 256-pixel tile of 256 x 16 x 16 x 256, 256 -> 256, this phase took 2050).
    if (tid < BM) {
        constexpr int kTaps = 9;
        const int* at = pix_pop + slot_s[tid];
        const int taps = cv.kh * cv.kw;
        int sum = 0, off = 0, kx = 0;
        if (taps == 1) sum = at[0];
        for (int t0 = 0; t0 < taps && taps > 1; t0 += kTaps) {
            int v[kTaps];
#pragma unroll
            for (int u = 0; u < kTaps; ++u) {
                v[u] = at[off];                         // past the last tap: the last one again
                if (t0 + u + 1 < taps) {
                    ++off;
                    if (++kx == cv.kw) {
                        kx = 0;
                        off += pg.pw - cv.kw;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kTaps; ++u) sum += t0 + u < taps ? v[u] : 0;
        }
        pop_a[tid] = 2 * sum;
        if (FUSED) pop_af[tid] = 0.5f * float(sum);
    }

    // Column popcounts and column terms of the epilogue, once every filter word has been staged.
    auto publish_columns = [&] {
#pragma unroll
        for (int l = 0; l < LOADS_B; ++l) {
            int c = cnt_b[l];
            c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
            c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
            if (st_q == 0) {
                pop_b[st_r + l * ST_ROWS] = 2 * c;
                if (FUSED) colfix_s[st_r + l * ST_ROWS] = fold_column_term(thr_s[st_r + l * ST_ROWS], K, 2 * c);
            }
        }
    };
    if (BRES) publish_columns();

    // This lane's A operands: pixel wm*32*WM + i*32 + fr, words of lane half fh.
    const uint2* rd_a[WM];
    const uint32_t* rd_aw[WM];                          // WORDS: the pixel's cell in plane 0
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int slot = slot_s[wm * 32 * WM + i * 32 + fr];
        rd_a[i] = patch + fh * pg.slots + slot;
        rd_aw[i] = patchw + slot;
    }
    const int rd_b = fh * PLANE_B + wn * 32 * WN + fr;

    v16f acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // (tap row, tap column, channel quad) of the next quad of K, stepped with carries.
    int ky = 0, kx = 0, cq = 0;
    // KS > 1: this wavefront's half of the K-tiles' quads.
    const int kt_first = KS > 1 && kg == 1 ? n_ktiles / 2 : 0, kt_end = KS > 1 && kg == 0 ? n_ktiles / 2 : n_ktiles;
    if (KS > 1 && !WORDS && kt_first > 0) {
        const int tap = 4 * kt_first / pg.cqn;
        cq = 4 * kt_first - tap * pg.cqn;
        ky = tap / cv.kw;
        kx = tap - ky * cv.kw;
    }
    for (int kt = kt_first; kt < kt_end; ++kt) {
        const int buf = BRES ? kt : kt & 1;
        if (!BRES && kt + 1 < n_ktiles) fetch_b(kt + 1);
        const int quads_here = min(4, pg.kq - 4 * kt);
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            if (qq >= quads_here) break;
            uint2 aw[WM], bw[WN];
            if (WORDS) {
                // this lane half's two K-words of the quad: 4q + 2*fh and the next one
                const int2 off = *reinterpret_cast<const int2*>(&koff_s[4 * (4 * kt + qq) + 2 * fh]);
#pragma unroll
                for (int i = 0; i < WM; ++i) aw[i] = make_uint2(rd_aw[i][off.x], rd_aw[i][off.y]);
            } else {
                const int a_off = (2 * cq) * pg.slots + ky * pg.pw + kx;
#pragma unroll
                for (int i = 0; i < WM; ++i) aw[i] = rd_a[i][a_off];
            }
#pragma unroll
            for (int j = 0; j < WN; ++j) bw[j] = lds_b[(8 * buf + 2 * qq) * PLANE_B + rd_b + j * 32];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                v8i fa[WM], fb[WN];
#pragma unroll
                for (int i = 0; i < WM; ++i) fa[i] = widen_fp4_a(s == 0 ? aw[i].x : aw[i].y);
#pragma unroll
                for (int j = 0; j < WN; ++j) fb[j] = widen_fp4_b(s == 0 ? bw[j].x : bw[j].y);
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        // fused: operands swapped, the accumulators hold the transposed blocks (mfma_epilogue_bits)
                        if (FUSED)
                            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                fb[j], fa[i], acc[i][j], 4 /* fp4 */, 4 /* fp4 */, 0, 0, 0, 0);
                        else
                            acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                fa[i], fb[j], acc[i][j], 4 /* A: fp4 */, 4 /* B: fp4 */, 0, 0, 0, 0);
                    }
            }
            if (!WORDS && ++cq == pg.cqn) {
                cq = 0;
                if (++kx == cv.kw) {
                    kx = 0;
                    ++ky;
                }
            }
        }
        if (!BRES) {
            // Keep the staging of the next B tile (and the wait for its loads) behind the MFMA steps.
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) asm volatile("" : "+v"(acc[i][j]) : : "memory");
            if (kt + 1 < n_ktiles) stage_b(kt + 1, buf ^ 1);
            __syncthreads();
        }
    }

    if constexpr (KS > 1) {
        // The second half's sums, through the memory of the filters, which every wavefront has finished reading.
        // (16-byte aligned: dynamic LDS starts so, lds_b is 8-byte aligned in it.)
        const size_t at = (size_t(lds_b - patch) + 1) & ~size_t(1);
        float4* sums = reinterpret_cast<float4*>(patch + at) + (wave & 3) * (WM * WN * 4 * kWave);
        __syncthreads();
        if (kg == 1) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        sums[((i * WN + j) * 4 + g) * kWave + lane] =
                            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float4 v = sums[((i * WN + j) * 4 + g) * kWave + lane];
                        acc[i][j][4 * g] += v.x;
                        acc[i][j][4 * g + 1] += v.y;
                        acc[i][j][4 * g + 2] += v.z;
                        acc[i][j][4 * g + 3] += v.w;
                    }
        }
    }

    if (!BRES) publish_columns();
    __syncthreads();
    if (KS > 1 && kg > 0) return;                       // no barrier follows

    if constexpr (POOL) {
        static_assert(FUSED, "pooling acts on output bits");
        uint32_t words[WM];
        mfma_output_words<WM, WN>(acc, pop_a, pop_af, pop_b, thr_s, flip_s, colfix_s, N, K, col0, wm, wn, fr, fh, words);
        const uint32_t flip_word = flip_s[wn * WN + fh];
        const int64_t nw = (int64_t(N) + 31) >> 5;
        const int64_t w = ((int64_t(col0) + wn * 32 * WN) >> 5) + fh;
        // Lane i of the four that hold a window stores block i's word.
        uint32_t pooled = 0u;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const uint32_t p = pool_words(words[i], flip_word);              // by every lane
            pooled = (fr & 3) == i ? p : pooled;
        }
        const int m = row0 + wm * 32 * WM + (fr & 3) * 32 + (fr & 28);
        if ((fr & 3) < WM && m < M && w < nw) bn.out[int64_t(m >> 2) * bn.ld_out + w] = pooled;
    } else if constexpr (FUSED)
        mfma_epilogue_bits<WM, WN>(acc, pop_a, pop_af, pop_b, thr_s, flip_s, colfix_s, bn, M, N, K, row0, col0, wm, wn,
                                   fr, fh);
    else
        mfma_epilogue<WM, WN>(acc, pop_a, pop_b, C, ldc, M, N, K, row0, col0, wm, wn, fr, fh);
}

// Same-size stride-1 layers whose tiles of BM pixels are whole image rows that divide into images, or whole images.
static bool whole_row_tiles(const ConvArgs& cv, int BM) {
    if (cv.stride != 1 || cv.Ho != cv.H || cv.Wo != cv.W) return false;
    if (cv.kh != 2 * cv.pad + 1 || cv.kw != 2 * cv.pad + 1) return false;
    if (cv.W > BM || BM % cv.W != 0) return false;
    const int rows = BM / cv.W;
    return cv.H % rows == 0 || rows % cv.H == 0;
}

// The layers with whole channel words only (Cin % 128 != 0) that this kernel takes: whole-row tiles, resident filters.
static bool words_layer_fits(const ConvArgs& cv, int BM) {
    return whole_row_tiles(cv, BM) && (int64_t(cv.kh) * cv.kw * cv.Cw + 15) / 16 <= kResidentKTiles;
}

template <int WM, bool FUSED, bool POOL>
static int launch_patch(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                        int64_t N, int64_t K, BnSignArgs bn, ConvArgs cv, PatchGeom pg, void* stream) {
    const int64_t tiles_m = ceil_div(M, 64 * WM), tiles_n = ceil_div(N, 128);
    if (tiles_m * tiles_n > max_blocks(256)) return BNN_ERR_UNSUPPORTED;        // (the larger tiles of the gathering kernels)
    const bool words = cv.Cw % 4 != 0;                  // a tap is not a whole number of 16-byte quads
    const size_t patch_bytes = words ? (words_patch_koff_offset(cv.Cw, pg.slots) + size_t(4) * pg.kq) * 4
                                     : size_t(pg.slots) * size_t(cv.Cw) * 4 + size_t((pg.slots + 1) / 2) * 8;
    const int n_ktiles = (pg.kq + 3) / 4;
    const bool alone = WM <= 2 && n_ktiles > kResidentKTiles && n_ktiles <= kResidentKTilesAlone && tiles_m * tiles_n <= kLoneGrid;
    const bool few = n_ktiles <= kResidentKTiles;
    // Filters stay resident unless a compute unit then holds fewer workgroups than streaming them would leave it with, and the
    // grid needs more than it holds: 30 images of 100 x 100, 256 -> 256, stride 2 43.6 us resident, 30.5 streamed, 10 of 70 x 70
    // 17.9 and 14.7, 151 of 14 x 124, 256 -> 512 (256-pixel tiles, one resident workgroup) 179 and 119, 255 of 16 x 16, 256 ->
    // 256 (1020 tiles, three and four workgroups) 19.4 and 17.7; but 10 of 70 x 70 at stride 2 (192 tiles) 9.1 and 10.3, 100 of
    // 28 x 28 on 256 pixels (two either way) 24.9 and 24.8.
    const size_t tile_bytes = size_t(8) * (128 + 2) * sizeof(uint2);
    auto per_unit = [&](size_t filters) {
        const int64_t fit = int64_t(size_t(160) * 1024 / (patch_bytes + filters + (2 + WM) * 1024)), most = WM >= 4 ? 2 : 4;
        return fit < most ? fit : most;
    };
    const bool streams = !words && few && tiles_m * tiles_n > kComputeUnits * per_unit(n_ktiles * tile_bytes) &&
                         per_unit(n_ktiles * tile_bytes) < per_unit(2 * tile_bytes);
    const bool resident = (few && !streams) || alone;
    const bool split = WM <= 2 && resident && !words && tiles_m * tiles_n <= kLoneGrid &&
                       n_ktiles >= (WM == 1 ? 2 : 4);
    const size_t filter_bytes = resident ? n_ktiles * tile_bytes : 0;
    const size_t sum_bytes = split ? size_t(4) * WM * 2 * 4 * kWave * sizeof(float4) + 16 : 0;   // of the second half of K
    const size_t lds_bytes = patch_bytes + (filter_bytes > sum_bytes ? filter_bytes : sum_bytes);
    const int n_images = int(M / (int64_t(cv.Ho) * cv.Wo * (POOL ? 4 : 1)));
    const dim3 grid(unsigned(tiles_m * tiles_n));
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto launch = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), lds_bytes, s, in, B, ldb, C, ldc, int(M), int(N), int(K),
                           tile_map(tiles_m, tiles_n), bn, cv, pg, n_images);
    };
    constexpr int WS = WM <= 2 ? WM : 2;                // the forms below this line are for small tiles
    if (words) launch(conv_patch_mfma_kernel<WM, FUSED, POOL, kResidentKTiles, true, 1>, 256);   // resident: words_layer_fits
    else if (alone) launch(conv_patch_mfma_kernel<WS, FUSED, POOL, kResidentKTilesAlone, false, 2>, 512);
    else if (split) launch(conv_patch_mfma_kernel<WS, FUSED, POOL, kResidentKTiles, false, 2>, 512);
    else if (resident) launch(conv_patch_mfma_kernel<WM, FUSED, POOL, kResidentKTiles, false, 1>, 256);
    else launch(conv_patch_mfma_kernel<WM, FUSED, POOL, 0, false, 1>, 256);
    return check_launch();
}

// Pixels per tile: 256 (two workgroups per compute unit) when that grid fills the chip's 512 workgroup slots, else 128
// (three).  64 with resident filters where even that grid leaves 3/8 of the compute units without a workgroup: 51 images
// of 8 x 8, 256 -> 128 channels (26 tiles of 128) 8.8 -> 8.0 us, 20 of 16 x 16, 256 -> 256 (80) 9.0 -> 8.4, 128 -> 256 of
// 16 x 16 at stride 2 (128) 7.8 -> 6.6; but 52 of 16 x 16, 256 -> 256 pooled (208) 9.6 -> 9.9, and filters that stream
// through LDS (512 channels, 188 tiles) 17.0 -> 20.6: a K-tile of 64 pixels is over before the next one's loads are back.
//
// The shortest fields keep to 64 pixels up to 320 tiles of 128 (256 images of 14 x 14, 256 -> 256, 2 x 2 at stride 2, 196
// tiles, 7.2 -> 6.7 us, gathered 6.8; 128 of 28 x 28, 128 -> 256, 2 x 2 at stride 3, 162 tiles, 6.6 -> 6.0, gathered 6.3; 3 x 3
// over 128 channels in the int32 form 8.8 -> 7.7, but fused 6.6 -> 6.8).  The int32 form, whose stores take most of its time,
// gathers faster than 256-pixel tiles and slower than 128-pixel ones where the field is short (128 of 28 x 28, 128 -> 256: 1 x 1
// 21.4 gathered, 23.3, 18.2; 2 x 2 22.0, 24.2, 19.1; 3 x 3 30.1, 32.9, 25.6); whole-row layers keep the larger tiles.
constexpr int64_t kShortField = 1152;     // the longest receptive field of the short-K kernel
static bool wants_big_tiles(int64_t M, int64_t N) { return ceil_div(M, 256) * ceil_div(N, 128) >= 512; }
static bool wants_small_tiles(int64_t M, int64_t N, int64_t K, bool fused) {
    return ceil_div(M, 128) * ceil_div(N, 128) <= (K <= (fused ? 1024 : kShortField) ? 320 : 160) &&
           (K <= kResidentKTiles * 512 || (K <= kResidentKTilesAlone * 512 && ceil_div(M, 64) * ceil_div(N, 128) <= kLoneGrid));
}

// Layers of other than whole-row tiles that are faster gathered:
//  - patches of a few, wide rows hold many cells that no window of the tile reads: stride 1 and a receptive field that the
//    short-K kernel gathers, fused, 300 x 300 x 128 -> 128 14.8 us and 12.4 gathered (1812 cells), 2 images of 200 x 250 15.5 and
//    14.1 (1512); but 2 of 300 x 160 10.1 and 12.3 (972).  At stride 2 patches of 2034 cells still gain (4 of 224 x 224 9.4 and
//    10.3), and 256-pixel tiles read more of theirs (4 of 224 x 224 20.9 and 22.2).
//  - a patch that leaves a compute unit with two workgroups, streamed filters beside it, where three would take all tiles in one
//    round: 31 images of 28 x 28, 1024 -> 512 (760 tiles) 53.0 and 49.9, int32 57.2 and 50.2, 24 of them (588) 50.2 and 46.1; but
//    40 (980) 61.9 and 62.8.
//  - 1 x 1 windows over many channels, which reuse nothing: 200 images of 14 x 14, 1024 -> 512 19.4 and 14.4, int32 23.9 and
//    19.9, 768 channels int32 22.0 and 19.6; but fused 512 -> 256 over 64 of 28 x 28 8.6 and 9.6.
static bool better_gathered(const ConvArgs& cv, int BM, int64_t M, int64_t N, int64_t K, const PatchGeom& pg, bool fused) {
    if (whole_row_tiles(cv, BM)) return false;
    if (cv.kh * cv.kw == 1 && cv.Cw >= (fused ? 32 : 20)) return true;
    if (BM > 128) return false;
    if (cv.stride == 1 && K <= kShortField && pg.slots > 1280) return true;
    const int64_t tiles = ceil_div(M, BM) * ceil_div(N, 128);
    return K > kResidentKTiles * 512 && tiles > 512 && tiles <= 768 && int64_t(pg.slots) * (cv.Cw * 4 + 4) > 32 * 1024;
}

// BNN_ERR_UNSUPPORTED if the layer is not one this kernel takes (the caller then uses the gathering kernels).
template <bool FUSED>
static int launch_conv_patch_any(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc,
                                 int64_t M, int64_t N, int64_t K, BnSignArgs bn, ConvArgs cv, void* stream) {
    if (!aligned_to(B, 16) || ldb % 4 != 0) return BNN_ERR_UNSUPPORTED;
    PatchGeom pg;
    auto fits = [&](int BM) {
        return (cv.Cw % 4 == 0 || words_layer_fits(cv, BM)) && patch_geometry(cv, BM, BM, kPatchMaxBytes, false, pg) && !better_gathered(cv, BM, M, N, K, pg, FUSED);
    };
    if (wants_small_tiles(M, N, K, FUSED) && fits(128) && fits(64))
        return launch_patch<1, FUSED, false>(in, B, ldb, C, ldc, M, N, K, bn, cv, pg, stream);
    if (wants_big_tiles(M, N) && (FUSED || K > kShortField || whole_row_tiles(cv, 256)) && fits(256))
        return launch_patch<4, FUSED, false>(in, B, ldb, C, ldc, M, N, K, bn, cv, pg, stream);
    if (fits(128)) return launch_patch<2, FUSED, false>(in, B, ldb, C, ldc, M, N, K, bn, cv, pg, stream);
    return BNN_ERR_UNSUPPORTED;
}

// What bnn_conv_pool_bn_sign_pack takes: tiles of 64 * WM pixels that are whole image rows, even H and W, W a power of two
// below 32 or 32 * k with k <= WM / 2, and an even number of image rows per tile.
static bool pool_fits(const ConvArgs& cv, int WM) {
    const int BM = 64 * WM;
    if (!whole_row_tiles(cv, BM) || (cv.Cw % 4 != 0 && !words_layer_fits(cv, BM))) return false;
    const int rows = BM / cv.W < cv.H ? BM / cv.W : cv.H;
    if ((cv.H & 1) || (cv.W & 1) || (rows & 1)) return false;
    if (cv.W < 32) return (cv.W & (cv.W - 1)) == 0;
    return cv.W % 32 == 0 && 2 * (cv.W / 32) <= WM;
}

// Pooled layers of other than the maps of pool_fits that are faster as a convolution and a pooling of its output bits (2 to 3 us):
//  - windows lie in two image rows at least, so a pooled patch has more rows than the plain one; where a compute unit holds fewer
//    workgroups of 128 pixels with it (beside two K-tiles of streamed filters) and the grid then takes another round of them: one image
//    of 56 x 56, 512 -> 21028 (3795 tiles, 8 rounds and 5) 117 us, apart 103, 93 of 28 x 28, 768 -> 32 (570) 38.2 and 34.4, 5 of 56 x
//    183, 128 -> 17696 at stride 2 218 and 160; but 77 of 28 x 28, 768 -> 32 (472, one round) 25.1 and 27.4, and 1 x 1
//    windows win all the same (45 of 28 x 28, 768 -> 384 11.7 and 12.6);
//  - patches that only tiles of 256 pixels can hold (their windows fill whole rows) on fewer than 192 of those: 1, 3, 7 images of 32 x
//    128, 512 -> 128 19.3 and 14.5 to 15.5, 14 of 16 x 128, 128 -> 128, 7 x 7 25.2 and 21.6; but 30 (240 tiles) 25.3 and 27.4;
//  - what better_gathered says of 1 x 1 windows, beyond one round: 59 of 26 x 26, 1024 -> 384 14.8 and 13.6; but 15 of 28 x 14,
//    1024 -> 1718 (644 tiles) 10.4 and 12.0.
static bool better_pooled_apart(const ConvArgs& cv, const ConvArgs& units, int64_t M, int64_t N) {
    const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128), tiles256 = ceil_div(M, 256) * ceil_div(N, 128);
    if (cv.kh * cv.kw == 1) return cv.Cw >= 32 && tiles > 3 * kComputeUnits && !whole_row_tiles(cv, 128);
    PatchGeom pooled, plain;
    const bool fits256 = patch_geometry(units, 256, 256, kPatchMaxBytes, true, pooled);
    if (wants_big_tiles(M, N) && fits256) return false;
    if (!patch_geometry(units, 128, 128, kPatchMaxBytes, true, pooled)) return fits256 && tiles256 < 192;
    if (!patch_geometry(cv, 128, 128, kPatchMaxBytes, false, plain)) return false;
    auto rounds = [&](const PatchGeom& pg) {
        const int64_t bytes = pg.slots * (int64_t(cv.Cw) * 4 + 4) + 2 * 8 * (128 + 2) * int64_t(sizeof(uint2)) + 4 * 1024;
        const int64_t fit = 160 * 1024 / bytes;
        return ceil_div(tiles, kComputeUnits * (fit < 4 ? fit : 4));
    };
    return rounds(pooled) > rounds(plain);
}

// Whether three tiles of 256 pixels share a compute unit's local memory beside their resident filters (512 bits of K are 8 KB), four
// of 128 where the patch of 256 does not fit; layers that are gathered have no patch.  cv: the layer, its pooled_units if pool.
bool conv_patch_tiles_fill(const ConvArgs& cv, bool pool, int64_t K) {
    PatchGeom pg;
    auto fit = [&](int WM) {
        const int64_t patch = int64_t(pg.slots) * cv.Cw * 4 + (pg.slots + 1) / 2 * 8;
        return 160 * 1024 / (patch + ceil_div(K, 512) * 8 * (128 + 2) * int64_t(sizeof(uint2)) + (2 + WM) * 1024);
    };
    if (patch_geometry(cv, 256, 256, kPatchMaxBytes, pool, pg)) return fit(4) >= 3;
    return !patch_geometry(cv, 128, 128, kPatchMaxBytes, pool, pg) || fit(2) >= 4;
}

int launch_conv_patch(const uint32_t* in, const uint32_t* B, int64_t ldb, int32_t* C, int64_t ldc, int64_t M,
                      int64_t N, int64_t K, ConvArgs cv, void* stream) {
    return launch_conv_patch_any<false>(in, B, ldb, C, ldc, M, N, K, BnSignArgs{}, cv, stream);
}

int launch_conv_patch_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                            BnSignArgs bn, ConvArgs cv, void* stream) {
    const int st = launch_conv_strip_fused(in, B, ldb, M, N, K, bn, cv, false, ConvUse::faster, stream);
    if (st != BNN_ERR_UNSUPPORTED) return st;
    const int st_patch = launch_conv_patch_any<true>(in, B, ldb, nullptr, 0, M, N, K, bn, cv, stream);
    if (st_patch != BNN_ERR_UNSUPPORTED || ceil_div(M, 256) * ceil_div(N, 128) <= max_blocks(256)) return st_patch;
    // More tiles than the gathering kernels can launch: strips, whatever part of the chip they leave idle.
    return launch_conv_strip_fused(in, B, ldb, M, N, K, bn, cv, false, ConvUse::any, stream);
}

// Convolution, 2 x 2 max pooling (stride 2), BatchNorm, Sign in one launch; bn.out is the pooled
// packed NHWC map [B][Ho/2][Wo/2][ld_out].  BNN_ERR_UNSUPPORTED for what it does not take (the caller then pools the unpooled
// output bits with bnn_maxpool_bits).  any_map: any even map of whole channel quads whose patch fits, not only the layers of
// pool_fits.  ConvUse::ask: BNN_OK, with nothing launched, for what it takes and is no slower than the two launches.
int launch_conv_patch_pool_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                                 BnSignArgs bn, ConvArgs cv, bool any_map, ConvUse use, void* stream) {
    if (!aligned_to(B, 16) || ldb % 4 != 0) return BNN_ERR_UNSUPPORTED;
    PatchGeom pg;
    const bool whole_rows = (pool_fits(cv, 2) && patch_geometry(cv, 128, 128, kPatchMaxBytes, false, pg)) ||
                            (pool_fits(cv, 4) && patch_geometry(cv, 256, 256, kPatchMaxBytes, false, pg));
    if (any_map ? cv.Cw % 4 != 0 || ((cv.Ho | cv.Wo) & 1) : !whole_rows) return BNN_ERR_UNSUPPORTED;
    const bool ask = use == ConvUse::ask;
    const int st = launch_conv_strip_fused(in, B, ldb, M, N, K, bn, cv, true, use, stream);
    if (st != BNN_ERR_UNSUPPORTED) return st;
    const ConvArgs units = pooled_units(cv);
    if (ask && !whole_rows && better_pooled_apart(cv, units, M, N)) return BNN_ERR_UNSUPPORTED;
    auto fits = [&](int WM) {
        if (whole_rows && !pool_fits(cv, WM)) return false;
        return patch_geometry(units, 64 * WM, 64 * WM, kPatchMaxBytes, true, pg);
    };
    if (ask) return fits(2) || fits(4) ? BNN_OK : BNN_ERR_UNSUPPORTED;
    int st_patch = BNN_ERR_UNSUPPORTED;
    if (wants_small_tiles(M, N, K, true) && fits(2) && fits(1))
        st_patch = launch_patch<1, true, true>(in, B, ldb, nullptr, 0, M, N, K, bn, units, pg, stream);
    else if (wants_big_tiles(M, N) && fits(4))
        st_patch = launch_patch<4, true, true>(in, B, ldb, nullptr, 0, M, N, K, bn, units, pg, stream);
    else if (fits(2))
        st_patch = launch_patch<2, true, true>(in, B, ldb, nullptr, 0, M, N, K, bn, units, pg, stream);
    else if (fits(4))
        st_patch = launch_patch<4, true, true>(in, B, ldb, nullptr, 0, M, N, K, bn, units, pg, stream);
    if (st_patch != BNN_ERR_UNSUPPORTED) return st_patch;
    // A patch that only the strips' share of local memory holds, or more tiles than one launch does.
    return launch_conv_strip_fused(in, B, ldb, M, N, K, bn, cv, true, ConvUse::any, stream);
}

}  // namespace bnn

// Binary convolution layers on bits (fused with Sign(BatchNorm), with or without 2 x 2 max pooling) in strips:
// one workgroup of eight wavefronts per compute unit, 128 filters resident in LDS, a strip of output pixels walked in tiles
// of 512.
//
// Arithmetic, patch and filter layout are those of conv_patch.hip (an input patch in LDS, the A operand of tap (ky, kx) read at
// slot(pixel) + ky * PW + kx; pooled layers in window order).  What differs is how the work is cut, because at batch 256 these
// layers are bound by what surrounds their products: of the 34500 cycles of a workgroup of 256 pixels x 128 filters (256 -> 256
// channels of 16 x 16, two workgroups per compute unit, all starting together) 18400 were matrix cycles.
//   - Filters are staged once per compute unit instead of once per 256 pixels: loads go through the unit at 64 bytes a
//     cycle, so staging them twice beside two patches took 1500 of the 7500 cycles before the first product, and filters of
//     up to nine K-tiles (3 x 3 over 512 channels) fit instead of streaming.
//   - Strips are equal: the N / 128 column tiles times `groups` strips are at most one workgroup per compute unit, and
//     every workgroup has the same pixels, where whole tiles left the last round of workgroups half empty (392 tiles of 256
//     pixels over 512 slots).  A strip's last tile holds what is left, in block rows of 32 dealt to the wavefronts in turn.
//   - While a tile is multiplied the next one's patch is loaded into registers and stored to another of three buffers, with
//     one barrier per tile, so that a wavefront's epilogue and start of the next tile run under the other wavefront's products.
//   - Everything a wavefront needs for its own rows (patch cells, window popcounts) it computes itself, and the
//     accumulators START as the folded threshold, a product of bf16 pairs (a quarter of the rank-2 fp32 update that
//     conv_patch.hip adds at the end, and neither zeros nor a pass of its own).
//   - The K loop is one quad of channels (two steps of 64) long: the operands of a step are widened between the products of
//     the step before, LDS is read half a step ahead (BNN_STRIP_SCHEDULE).  The two wavefronts of a SIMD take 39 cycles per
//     product together, 36 where one runs alone: alternating operands cost the engine more than the issue of both does.
//   - What comes before the first product is bound by the number of its instructions (two wavefronts of a SIMD take about eight
//     cycles for each): 900 of them, 8000 cycles of 31000, for 256 -> 256 of 16 x 16, 5300 now.  Hence the divisions in float32
//     (strip_cells.h), a kernel for each way of walking a strip (Walk) and for 3 x 3 windows, the arguments that the first loads
//     need in the first line of the argument block, and the pixels' cells held before the barrier, while the loads are in flight.
// Batch 256, us of the kernel replayed from a graph, tiles of conv_patch.hip, strips before that and now: 128 -> 128 of 32 x 32 pooled 19.3, 17.0, 15.7, 128 -> 256 of
// 16 x 16 10.9, 10.1, 9.0, 256 -> 256 16.3, 15.0, 13.6, 256 -> 512 of 8 x 8 11.3, 10.0, 9.5, 512 -> 512 pooled 18.3, 16.2, 15.6;
// 128 images of 28 x 28, 128 -> 256 pooled (on tiles two launches) 21.7, 15.1, 13.6.
// Signs (+-1) for the filters' bits would need no popcounts of the pixels (2600 cycles less before the first product), but operands
// that change sign cost the engine more power than bits: 2.11 GHz where bits hold 2.36, and no gain (15.0 us for 256 -> 256).
// Four wavefronts of 4 x 4 blocks (one per SIMD) were slower at every size (256 -> 256 of 16 x 16 21.4): the allocator does not
// fit 256 accumulators and the next patch's registers, and nothing covers the phases between the tiles.
#include <numeric>

#include "bnn_internal.h"
#include "conv_patch_geometry.h"
#include "gemm_staging.h"
#include "mfma_fp4.h"
#include "strip_cells.h"
#include "strip_cut.h"

namespace bnn {
namespace strip {

constexpr int T = 512, BN = 128, PLANE_B = BN + 2;     // 8-byte slots per filter plane (2 pad slots)
constexpr int WAVE_ROWS = 4;                           // wavefronts along the pixels, two along the filters
constexpr int NB_MAX = 4;                              // block rows of 32 pixels per wavefront
constexpr int BM = 32 * WAVE_ROWS * NB_MAX;            // 512 pixels
constexpr int PF_SLOTS = 2, PF_QUADS = 2;              // patch cells per thread and quads per cell that are loaded ahead
constexpr int FIRST = 4;                               // quads of the first patch that a thread loads before it stores one

// How the layer is cut.
struct Cut {
    FastDiv by_tiles_n;
    int tiles_n, per_die;      // column tiles; workgroups / 8
    int rows;                  // pixels per strip, a multiple of 32
};

// A tile and its patch: unit row and column (in the image) and image of the tile's first unit, first padded row of the patch in
// that image, cells to load (up to the end of the tile's last window where that may be far fewer than the largest patch has), first row
// of the image that can be among them, and that row's address.  Units: pixels, or (POOL) pooling windows, whose maps cv.Wo, cv.Ho and
// the divisions then describe.
struct Origin {
    int y, x, b, row0, slots, top;
    const uint32_t* at;
};

template <bool POOL>
__device__ __forceinline__ Origin origin_of(const uint32_t* in, const PatchGeom& pg, const ConvArgs& cv, int row0, int rows) {
    constexpr int PF = POOL ? 2 : 1;
    const int u0 = POOL ? row0 >> 2 : row0;
    const int first = pg.by_wo(u0), b0 = pg.by_ho(first), y0 = first - b0 * cv.Ho;
    const int row_first = PF * y0 * cv.stride, top = max(min(row_first - cv.pad, cv.H - 1), 0);
    int slots = pg.slots;
    if (pg.trim) {
        const int last = pg.by_wo(POOL ? (row0 + rows - 1) >> 2 : row0 + rows - 1), b1 = pg.by_ho(last), y1 = last - b1 * cv.Ho;
        slots = ((b1 - b0) * pg.img_rows + PF * (y1 - y0) * cv.stride + (PF - 1) * cv.stride + cv.kh) * pg.pw;
    }
    return Origin{y0, u0 - first * cv.Wo, b0, row_first, slots, top,
                  in + (size_t(b0) * uint32_t(cv.H) + uint32_t(top)) * uint32_t(cv.W) * uint32_t(cv.Cw)};
}

// Byte offset of cell s of a patch from o.at, 0 for a cell outside the images.
__device__ __forceinline__ uint32_t cell_of(const Maps& maps, const ConvArgs& cv, int n_images, Origin o, int s, bool& inside) {
    const uint32_t at = input_of_cell(maps, cv.pad, cv.H, cv.W, o.row0, o.top, n_images - o.b, s, inside);
    inside = inside && s < o.slots;
    return inside ? at : 0u;
}

__device__ __forceinline__ uint4 ones_unless(bool keep, uint4 v) {
    return make_uint4(keep ? v.x : ~0u, keep ? v.y : ~0u, keep ? v.z : ~0u, keep ? v.w : ~0u);
}

__device__ __forceinline__ void put_quad(uint2* patch, int slots, int s, int cq, uint4 v) {
    patch[(2 * cq) * slots + s] = make_uint2(v.x, v.y);
    patch[(2 * cq + 1) * slots + s] = make_uint2(v.z, v.w);
}

// Quad cq of the cell at byte offset `at`.
__device__ __forceinline__ uint4 load_at(const uint32_t* image, uint32_t at, int cq) {
    return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(image) + 16 * cq + at);
}

// Cells s0, s0 + T, ... (FIRST / C of them) of a patch, C quads each, on their way into registers ...
template <int C>
__device__ __forceinline__ void load_cells(const PatchGeom& pg, const Maps& maps, const ConvArgs& cv, int n_images, Origin o, int s0,
                                           int cq0, uint4 (&v)[FIRST], uint32_t& inside) {
    inside = 0u;
#pragma unroll
    for (int u = 0; u < FIRST / C; ++u) {
        bool in_image;
        const uint32_t at = cell_of(maps, cv, n_images, o, s0 + u * T, in_image);
        inside |= in_image ? 1u << u : 0u;
#pragma unroll
        for (int c = 0; c < C; ++c) v[u * C + c] = load_at(o.at, at, min(cq0 + c, pg.cqn - 1));
    }
}

// ... and from there to LDS; pop: set bits of the cells' quads before cq0, and afterwards with these.
template <int C>
__device__ __forceinline__ void store_cells(const PatchGeom& pg, Origin o, int s0, int cq0, const uint4 (&v)[FIRST], uint32_t inside,
                                            int (&pop)[FIRST / C], uint2* patch) {
    const int slots = pg.slots, cqn = pg.cqn;
#pragma unroll
    for (int u = 0; u < FIRST / C; ++u) {
        const int s = s0 + u * T;
        const bool keep = (inside >> u) & 1u;
        if (s < o.slots) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (cq0 + c >= cqn) break;
                const uint4 w = ones_unless(keep, v[u * C + c]);
                patch[(2 * (cq0 + c)) * slots + s] = make_uint2(w.x, w.y);
                patch[(2 * (cq0 + c) + 1) * slots + s] = make_uint2(w.z, w.w);
                pop[u] += popc4(w);
            }
            if (cq0 + C >= cqn) reinterpret_cast<int*>(patch + 2 * cqn * slots)[s] = pop[u];
        }
    }
}

// A whole patch but for what load_cells(s0 = tid, cq0 = 0) took.
template <int C>
__device__ __forceinline__ void load_rest(const PatchGeom& pg, const Maps& maps, const ConvArgs& cv, int n_images, Origin o,
                                          int (&pop)[FIRST / C], uint2* patch) {
    for (int base = 0; base < o.slots; base += FIRST / C * T) {
        if (base > 0) {
#pragma unroll
            for (int u = 0; u < FIRST / C; ++u) pop[u] = 0;
        }
        for (int cq0 = base == 0 ? C : 0; cq0 < pg.cqn; cq0 += C) {
            uint4 v[FIRST];
            uint32_t inside;
            load_cells<C>(pg, maps, cv, n_images, o, base + int(threadIdx.x), cq0, v, inside);
            store_cells<C>(pg, o, base + int(threadIdx.x), cq0, v, inside, pop, patch);
        }
    }
}

// Strips of one tile, or longer ones whose next patch is loaded under the products (AHEAD: into another of up to three buffers) or
// between the tiles.  One kernel for all of them keeps up to 51 scalars in lanes of a vector register (none for one tile): 256 -> 256
// of 16 x 16 14.5 us with it, 13.6 with these.
enum class Walk { ONE, AHEAD, BETWEEN };

// C: quads per cell and load of the first patch.  K3: windows of 3 x 3.
template <bool POOL, int RES, int C, Walk WALK, bool K3>
__global__ __launch_bounds__(T, 2) void conv_strip_mfma_kernel(
    const uint32_t* __restrict__ in, const uint32_t* __restrict__ B, int64_t ldb, Cut cut, int M, int N, int K, int n_images,
    BnSignArgs bn, ConvArgs cv, PatchGeom pg, Maps maps) {
    if constexpr (K3) cv.kh = cv.kw = 3;
    constexpr bool MANY = WALK != Walk::ONE;
    constexpr int WN = 2, PF = POOL ? 2 : 1;           // POOL: rows are the pixels of one pooling window after the other
    extern __shared__ __attribute__((aligned(16))) uint2 dyn[];            // filters, then up to three patches with their pixel popcounts
    __shared__ float colfix_s[BN];
    __shared__ uint32_t flip_s[BN / 32];
    const int cqn = pg.cqn, slots = pg.slots, kq = pg.kq;
    const int patch_size = 2 * cqn * slots + (slots + 1) / 2;     // in 8-byte slots
    uint2* patches = dyn + 2 * kq * PLANE_B;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fh = lane >> 5;

    // Consecutive workgroups go to the 8 dies in turn: a die takes neighbouring strips, with all their column tiles.
    int logical = int(blockIdx.x);
    if (logical < 8 * cut.per_die) logical = (logical & 7) * cut.per_die + (logical >> 3);
    const int group = cut.by_tiles_n(logical), col0 = (logical - group * cut.tiles_n) * BN;
    const StripRows strip = strip_rows(group, cut.rows, M);
    const int row_begin = strip.begin, row_end = strip.end;

    // ---- filters: every load of the start is in flight before the first one is waited for -----------------
    const int st_q = tid & 3, st_r = tid >> 2;
    const uint32_t* pb = B + int64_t(min(col0 + st_r, N - 1)) * ldb;
    uint4 all_b[RES];
#pragma unroll
    for (int kt = 0; kt < RES; ++kt)
        if (4 * kt < kq) all_b[kt] = *reinterpret_cast<const uint4*>(pb + 4 * min(4 * kt + st_q, kq - 1));
    const int thr = bn.thr[min(col0 + st_r, N - 1)];
    uint32_t flip_reg = 0u;
    if (tid < BN / 32 && col0 + 32 * tid < N) flip_reg = bn.flip_bits[(col0 >> 5) + tid];

    // ---- patches -------------------------------------------------------------------------------------------
    // Loaded ahead (Walk::AHEAD: at most PF_SLOTS cells per thread of at most PF_QUADS quads): cell u * T + tid of a patch.
    uint4 ahead[PF_QUADS];
    bool ahead_inside = false;
    auto load_ahead = [&](Origin o, int u) __attribute__((always_inline)) {
        const uint32_t at = cell_of(maps, cv, n_images, o, u * T + tid, ahead_inside);
#pragma unroll
        for (int c = 0; c < PF_QUADS; ++c) ahead[c] = load_at(o.at, at, min(c, cqn - 1));
    };
    auto store_ahead = [&](Origin o, int u, uint2* patch) __attribute__((always_inline)) {
        const int s = u * T + tid;
        if (s < o.slots) {
            const uint4 v0 = ones_unless(ahead_inside, ahead[0]);
            put_quad(patch, slots, s, 0, v0);
            int pop = popc4(v0);
            if (cqn > 1) {
                const uint4 v1 = ones_unless(ahead_inside, ahead[1]);
                put_quad(patch, slots, s, 1, v1);
                pop += popc4(v1);
            }
            reinterpret_cast<int*>(patch + 2 * cqn * slots)[s] = pop;
        }
    };

    Origin here = origin_of<POOL>(in, pg, cv, row_begin, min(BM, row_end - row_begin));
    uint4 first[FIRST];
    uint32_t first_inside;
    load_cells<C>(pg, maps, cv, n_images, here, tid, 0, first, first_inside);

    // The lane's rows as patch cells: row (i * WAVE_ROWS + wr) * 32 + fr of the tile.
    int slot[NB_MAX];
    const int in_window = POOL ? (fr & 2 ? cv.stride * pg.pw : 0) + (fr & 1 ? cv.stride : 0) : 0;
    auto find_slots = [&](int row0, Origin o) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB_MAX; ++i) {
            const int r = min((i * WAVE_ROWS + wr) * 32 + fr, row_end - 1 - row0);
            slot[i] = cell_of_unit(maps, o.y, o.x, o.row0, PF * cv.stride, POOL ? r >> 2 : r) + in_window;
        }
    };
    find_slots(row_begin, here);
    // Here, while the loads are in flight: the compiler would move it behind the barrier, to its first use.
#pragma unroll
    for (int i = 0; i < NB_MAX; ++i) asm volatile("" : "+v"(slot[i]));

    // Filters to LDS, planes [quad][half] of 8-byte slots, with their popcounts and column terms.
    {
        int c = 0;
#pragma unroll
        for (int kt = 0; kt < RES; ++kt)
            if (4 * kt + st_q < kq) {
                const uint4 v = all_b[kt];
                c += popc4(v);
                uint2* to = dyn + (2 * (4 * kt + st_q)) * PLANE_B + st_r;
                to[0] = make_uint2(v.x, v.y);
                to[PLANE_B] = make_uint2(v.z, v.w);
            }
        c += __builtin_amdgcn_update_dpp(0, c, 0xB1, 0xF, 0xF, true);       // lane ^ 1
        c += __builtin_amdgcn_update_dpp(0, c, 0x4E, 0xF, 0xF, true);       // lane ^ 2
        if (st_q == 0) colfix_s[st_r] = fold_column_term(max(-K - 1, min(K + 1, thr)), K, 2 * c);
        if (tid < BN / 32) flip_s[tid] = flip_reg;
    }
    {
        int pop[FIRST / C] = {};
        store_cells<C>(pg, here, tid, 0, first, first_inside, pop, patches);
        load_rest<C>(pg, maps, cv, n_images, here, pop, patches);
    }
    __syncthreads();

    // Left factors of the accumulators' start, start = (column term) x 1 + 1 x (row term), each term in two bf16 parts:
    // lane half 0 holds (column hi, column lo, 1, 1) and, on the right, (1, 1, row hi, row lo); half 1 zeros.
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

    // One tile: rows [row0, row0 + rows), the wavefront's NB block rows (block i * WAVE_ROWS + wr).
    auto run = [&](auto nb_tag, int row0, uint2* patch, bool more_tiles, Origin next, uint2* next_patch) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_tag)::value;
        constexpr int VALU = (5 * NB + 6 * WN + NB * WN - 1) / (NB * WN);      // widening of a step, per product
        const bool more = MANY && NB == NB_MAX && more_tiles;                          // a tile before the last one is whole
        const uint2* rd_a[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) rd_a[i] = patch + fh * slots + slot[i];
        v16f acc[NB][WN];
        {
            // Popcounts under the windows: lane half h sums block rows i with i % 2 = h, nine taps at a time.
            const int* pops = reinterpret_cast<int*>(patch + 2 * cqn * slots);
            constexpr int NP = (NB + 1) / 2;
            const int* at[NP];
            int sum[NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int odd = slot[2 * p + 1 < NB ? 2 * p + 1 : 2 * p];
                at[p] = pops + (fh == 0 ? slot[2 * p] : odd);
                sum[p] = 0;
            }
            if constexpr (K3) {
                int v[NP][9];
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int e = 0; e < 9; ++e) v[p][e] = at[p][(e / 3) * pg.pw + e % 3];
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int e = 0; e < 9; ++e) sum[p] += v[p][e];
            } else {
                for (int ky = 0; ky < cv.kh; ky += 3)
                    for (int kx = 0; kx < cv.kw; kx += 3) {
                        int v[NP][9];
#pragma unroll
                        for (int p = 0; p < NP; ++p)
#pragma unroll
                            for (int e = 0; e < 9; ++e)
                                v[p][e] = at[p][min(ky + e / 3, cv.kh - 1) * pg.pw + min(kx + e % 3, cv.kw - 1)];
#pragma unroll
                        for (int p = 0; p < NP; ++p)
#pragma unroll
                            for (int e = 0; e < 9; ++e) sum[p] += ky + e / 3 < cv.kh && kx + e % 3 < cv.kw ? v[p][e] : 0;
                    }
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                short hi, lo;
                split_bf16(-0.5f * float(sum[p]), hi, lo);                 // block row 2p + fh
                const uint32_t mine = uint32_t(uint16_t(hi)) | (uint32_t(uint16_t(lo)) << 16);
                const auto sw = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
                const uint32_t odd = sw[1];                                // lanes 0-31: what lanes 32-63 have
                const v4s right_even = {kOne, kOne, short(mine & 0xFFFFu), short(mine >> 16)};
                const v4s right_odd = {kOne, kOne, short(odd & 0xFFFFu), short(odd >> 16)};
                v16f zero;
#pragma unroll
                for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    acc[2 * p][j] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(left[j], right_even, zero, 0, 0, 0);
                    if (2 * p + 1 < NB)
                        acc[2 * p + 1 < NB ? 2 * p + 1 : 0][j] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(left[j], right_odd, zero, 0, 0, 0);
                }
            }
        }
        const bool piped = WALK == Walk::AHEAD && more;
        if (piped) load_ahead(next, 0);

        // K loop over quads of channels; (ky, kx, cq) of the quad that is read next, stepped with carries.
        int kx = 0, cq = 0, off = 0, q = 0;
        const int row_step = pg.pw - cv.kw + 1, plane_step = 2 * slots;
        auto step_quad = [&]() __attribute__((always_inline)) {
            if (++cq < cqn) {
                off += plane_step;
            } else {
                cq = 0;
                off -= (cqn - 1) * plane_step;
                if (++kx < cv.kw) {
                    ++off;
                } else {
                    kx = 0;
                    off += row_step;
                }
            }
        };
        const uint2* rd_b = rd_b0;
        uint2 aw[NB], bw[WN];
        auto read_words = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NB; ++i) aw[i] = rd_a[i][off];
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
            // operands swapped: the accumulators hold the transposed blocks, a lane 16 columns of one output row
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand8(b[j]), operand8(a[i]), acc[i][j], 4, 4, 0, 0, 0, 0);
        };
        for (int part = piped ? 0 : 2; part < 3; ++part) {
            const int q_end = WALK != Walk::AHEAD || part == 2 ? kq : part == 0 ? kq / 3 : 2 * kq / 3;
            for (; q < q_end; ++q) {
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < kq) {                    // past the end the last quad again, whose products are not taken
                    step_quad();
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
            // The next patch, half of the cells, then the rest (the loop has registers for one cell's quads, not for two).  A
            // buffer is written two tiles after it was read, behind the barrier of the tile in between.
            if (WALK == Walk::AHEAD && part == 0) {
                store_ahead(next, 0, next_patch);
                load_ahead(next, 1);
            } else if (WALK == Walk::AHEAD && part == 1) {
                store_ahead(next, 1, next_patch);
                __syncthreads();
            }
        }
        if (WALK == Walk::BETWEEN && more) {
            __syncthreads();
            int pop[FIRST / C] = {};
            load_cells<C>(pg, maps, cv, n_images, next, tid, 0, first, first_inside);
            store_cells<C>(pg, next, tid, 0, first, first_inside, pop, next_patch);
            load_rest<C>(pg, maps, cv, n_images, next, pop, next_patch);
            __syncthreads();
        }

        // The output bit is the complement of the accumulator's sign (mfma_output_words).
        uint32_t words[NB];
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
            words[i] = ((sw[0] | sw[1]) ^ flip_word) & live_word;
        }
        if (cols_left <= 0) return;
        if constexpr (POOL) {
            // Lane i of the four that hold a window stores block row i's word.
            uint32_t pooled = 0u;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const uint32_t w = pool_words(words[i], flip_word);
                pooled = (fr & 3) == i ? w : pooled;
            }
            const int m = row0 + ((fr & 3) * WAVE_ROWS + wr) * 32 + (fr & 28);
            if ((fr & 3) < NB && m < row_end) out[int64_t(m >> 2) * bn.ld_out] = pooled;
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int m = row0 + (i * WAVE_ROWS + wr) * 32 + fr;
                if (m < row_end) out[int64_t(m) * bn.ld_out] = words[i];
            }
        }
    };

    auto tile = [&](int row0, uint2* patch, bool more, Origin next, uint2* next_patch) __attribute__((always_inline)) {
        const int blocks = (min(BM, row_end - row0) + 31) / 32, mine = (blocks - wr + WAVE_ROWS - 1) / WAVE_ROWS;
        if (__builtin_expect(mine == 4, 1)) run(std::integral_constant<int, 4>{}, row0, patch, more, next, next_patch);
        else if (mine == 3) run(std::integral_constant<int, 3>{}, row0, patch, more, next, next_patch);
        else if (mine == 2) run(std::integral_constant<int, 2>{}, row0, patch, more, next, next_patch);
        else if (mine == 1) run(std::integral_constant<int, 1>{}, row0, patch, more, next, next_patch);
    };
    if constexpr (!MANY) {
        tile(row_begin, patches, false, here, patches);
    } else {
        int buf = 0;
        for (int row0 = row_begin; row0 < row_end; row0 += BM) {
            const int left_rows = row_end - row0 - BM;
            const bool more = left_rows > 0;
            Origin next = here;
            if (more) next = origin_of<POOL>(in, pg, cv, row0 + BM, min(BM, left_rows));
            uint2* patch = patches + buf * patch_size;
            if (WALK == Walk::AHEAD) buf = buf == 2 ? 0 : buf + 1;
            tile(row0, patch, more, next, patches + buf * patch_size);
            if (more) find_slots(row0 + BM, next);
            here = next;
        }
    }
}

}  // namespace strip

// Whether the tiles of conv_patch.hip that the layer would take fill a compute unit (there).
bool conv_patch_tiles_fill(const ConvArgs& cv, bool pool, int64_t K);

constexpr int kStripResident = 5, kStripResidentMost = 9;     // K-tiles of 512 bits of the resident filters
constexpr int64_t kStripLdsBytes = 158 * 1024;                // of 160 KB, beside what the kernel declares itself
static_assert(starts_in_bf16_pairs(kStripResidentMost * 512));
// Which of the layers that fit are faster here than on the tiles of conv_patch.hip and the gathering kernels.  Measured on 4100
// layers, pooled and not, of 1 to 25 taps, 128 to 1024 channels and 32 to 32768 filters; us, tiles and strips:
//  - strips of fewer than 160 rows for 3 x 3 windows, those of 32 and 64 rows however little of the chip they fill: 212 of the layers taken
//    1.01 to 1.53 times as fast, 1.12 in the mean (66 images of 14 x 14, 256 -> 256 8.4 and 7.4; 12 of 28 x 28, 256 -> 256 8.9 and 7.3; 16
//    of 32 x 32, 128 -> 64 5.5 and 4.95).  Windows of other sizes, which have no kernel for strips of one tile, lose more instructions
//    before the first product than they gain (10 of 14 x 14, 128 -> 128, 5 x 5 7.5 and 8.3).
//    Two kinds of them are left to tiles by lines that are coarser than what they separate.  64 rows of K > 2560, where a pair of 32-row
//    blocks shares the filters that tiles of 64 pixels keep for themselves: of 72 layers 35 lose up to 3 % in strips (52 of 14 x 14, 512 -> 99
//    9.75 and 9.99), 28 would gain more than that (4 of 30 x 30, 512 -> 512 12.1 and 10.2).  And strips of several map rows, but not of pairs of them,
//    where these are whole blocks of 32 pixels, so that a pooled layer's patch is no larger than the plain layer's: 72 of 72 layers
//    would be 1.06 to 1.55 times as fast in strips, plain ones as well (20 of 32 x 32, 256 -> 128 8.9 and 7.2);
//  - enough of the chip at work, from 96 rows on: 60 % with strips of one tile, 80 % up to four, 86 % beyond (41 images of 16 x 16, 256 -> 8576,
//    78 %, 75.5 and 79.1; 47 of 14 x 14, 512 -> 12288, 75 %, 169 and 190), 93 % with K <= 1152, whose tiles are short (40 of 28 x 28,
//    128 -> 9984, 91 %, 138 and 148; 58 of 32 x 32, 128 -> 4700 pooled, 87 %, 123 and 139);
//  - K <= 1536: whatever follows holds only for layers whose tiles fill a compute unit (conv_patch_tiles_fill: three of 256 pixels or
//    four of 128; gathered layers).  Of 5700 layers, those whose larger patches leave it with fewer are 1.02 to 1.45 times faster in
//    strips (225 of 28 x 28, 128 -> 512 at stride 2, two tiles, 19.6 and 16.1; 228 of 34 x 92, 256 -> 512, 3 x 1, pooled 154 and 130),
//    but for K <= 512 with a patch that is mostly not read (14685 of 28 x 19, 128 -> 64, 4 x 1 at stride 3 0.82 times as fast);
//  - K <= 1152 not with 577 to 768 rows: the three tiles of a compute unit are one round (3 x 3, 185 of 16 x 16, 128 -> 512, 740 rows,
//    13.7 and 14.9; 73 of 14 x 51, 256 -> 512, 1 x 4, 12.6 and 14.8; 800 rows and more 1.1 to 1.25 times faster in strips);
//  - fewer than nine taps reuse little of a patch.  Their tiles win where most of the strip's patch is not read (more than eight
//    cells per pixel: 571 of 32 x 32, 384 -> 128, 1 x 4 at stride 3 8.8 and 10.9), in strips of more than two tiles with K < 1152
//    (145 of 89 x 89, 128 -> 128, 7 x 1 65.3 and 75.2), two taps (189 of 56 x 56, 1024 -> 128, 2 x 1 64.5 and 74.2) or up to four of
//    K <= 1536 on dense patches (493 of 28 x 28, 384 -> 384, 4 x 1 93.8 and 109), and in the shortest strips with K <= 512 (64 of
//    32 x 32, 128 -> 128, 1 x 4 5.7 and 6.0).
// cv: the layer, its pooled_units if pool.
static bool strips_preferred(const ConvArgs& cv, bool pool, int64_t M, int64_t K, int64_t tiles_n, int64_t rows, int64_t cells,
                             int64_t pixels) {
    const int64_t tiles = ceil_div(rows, strip::BM), taps = int64_t(cv.kh) * cv.kw, row = pool ? 2 * int64_t(cv.Wo) : cv.Wo;
    if (rows < 5 * kStripStep && (cv.kh != 3 || cv.kw != 3)) return false;
    if (rows == 2 * kStripStep && K > kStripResident * 512) return false;
    if (rows < 5 * kStripStep && row % kStripStep == 0 && rows > row && rows % (2 * row) != 0) return false;
    if (rows > 2 * kStripStep && !strips_fill(M, tiles_n, rows, tiles == 1 ? 60 : tiles <= 4 ? 80 : K <= 1152 ? 93 : 86)) return false;
    if (taps < 9 && K <= 512 && cells > 8 * pixels) return false;
    if (K <= 1536 && !conv_patch_tiles_fill(cv, pool, K)) return true;
    if (K <= 1152 && rows > 576 && rows <= 768) return false;
    if (taps >= 9) return true;
    if (K <= 1536 && cells > 8 * pixels) return false;
    if (tiles > 2 && (K < 1152 || taps <= 2 || (taps <= 4 && K <= 1536 && 2 * cells < 3 * pixels))) return false;
    return K > 512 || rows > 256;
}

// BNN_ERR_UNSUPPORTED, with nothing launched, for a layer that this kernel does not take or, but for ConvUse::any, that is faster
// elsewhere.
int launch_conv_strip_fused(const uint32_t* in, const uint32_t* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                            BnSignArgs bn, ConvArgs cv, bool pool, ConvUse use, void* stream) {
    using namespace strip;
    if (!aligned_to(B, 16) || ldb % 4 != 0 || cv.Cw % 4 != 0 || K > kStripResidentMost * 512) return BNN_ERR_UNSUPPORTED;
    if (pool && ((cv.Ho | cv.Wo) & 1)) return BNN_ERR_UNSUPPORTED;
    const int64_t tiles_n = ceil_div(N, BN);
    if (tiles_n > kStripUnits) return BNN_ERR_UNSUPPORTED;
    const int n_images = int(M / (int64_t(cv.Ho) * cv.Wo));
    PatchGeom pg;
    Cut cut;
    const StripPlan plan = strip_plan(M, tiles_n);
    const int64_t rows = plan.rows, groups = plan.groups;
    // Windows that do not overlap reuse nothing of a patch: 1 x 1, 64 of 32 x 32, 256 -> 256 6.6 us on tiles and 7.4, 2 x 2 at stride 2, 233
    // of 16 x 16, 128 -> 512 7.7 and 7.95; but 2 x 2 at stride 1, 128 of 28 x 28, 256 -> 256 17.3 and 14.9.
    if (cv.kh <= cv.stride && cv.kw <= cv.stride) return BNN_ERR_UNSUPPORTED;
    if (pool) cv = pooled_units(cv);
    // Tiles start at multiples of the strips' rows, and 512 pixels further on.
    const int64_t tile = rows < BM ? rows : BM, align = rows <= BM ? rows : std::gcd(rows, int64_t(BM));
    if (!patch_geometry(cv, tile, align, kStripLdsBytes, pool, pg)) return BNN_ERR_UNSUPPORTED;
    if (use != ConvUse::any && !strips_preferred(cv, pool, M, K, tiles_n, rows, pg.slots, tile)) return BNN_ERR_UNSUPPORTED;
    const int64_t filters = int64_t(2) * pg.kq * PLANE_B * 8, patch = (int64_t(2) * pg.cqn * pg.slots + (pg.slots + 1) / 2) * 8;
    if (filters + patch > kStripLdsBytes) return BNN_ERR_UNSUPPORTED;
    if (use == ConvUse::ask) return BNN_OK;
    const int64_t tiles = ceil_div(rows, BM), buffers = tiles < 3 ? tiles : 3;
    const bool ahead = tiles > 1 && pg.slots <= PF_SLOTS * T && pg.cqn <= PF_QUADS && filters + buffers * patch <= kStripLdsBytes;
    cut.tiles_n = int(tiles_n);
    cut.by_tiles_n = fast_div(tiles_n);
    cut.per_die = int(groups * tiles_n / 8);
    cut.rows = int(rows);
    const Maps maps = maps_of(cv.Wo, cv.Ho, pg.img_rows, pg.pw, cv.H, cv.W, cv.Cw);
    const size_t lds = size_t(filters + (ahead ? buffers : 1) * patch);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(unsigned(groups * tiles_n)), dim3(T), lds, static_cast<hipStream_t>(stream), in, B, ldb, cut,
                           int(M), int(N), int(K), n_images, bn, cv, pg, maps);
        return check_launch();
    };
    auto of_size = [&](auto pool_tag, auto res_tag, auto c_tag) {
        constexpr bool POOL = decltype(pool_tag)::value;
        constexpr int RES = decltype(res_tag)::value, C = decltype(c_tag)::value;
        constexpr bool K3 = RES == kStripResident || C != 2;            // two quads of 3 x 3 taps are at most 4.5 K-tiles
        const bool three = K3 && cv.kh == 3 && cv.kw == 3;
        if constexpr (C == PF_QUADS) {
            if (ahead) return three ? launch(conv_strip_mfma_kernel<POOL, RES, C, Walk::AHEAD, K3>)
                                    : launch(conv_strip_mfma_kernel<POOL, RES, C, Walk::AHEAD, false>);
        }
        if (!three) return launch(conv_strip_mfma_kernel<POOL, RES, C, Walk::BETWEEN, false>);
        return tiles > 1 ? launch(conv_strip_mfma_kernel<POOL, RES, C, Walk::BETWEEN, K3>)
                         : launch(conv_strip_mfma_kernel<POOL, RES, C, K3 ? Walk::ONE : Walk::BETWEEN, K3>);
    };
    using Two = std::integral_constant<int, PF_QUADS>;
    using Four = std::integral_constant<int, 4>;
    using Few = std::integral_constant<int, kStripResident>;
    using Most = std::integral_constant<int, kStripResidentMost>;
    auto launch_as = [&](auto pool_tag) {
        if (K > kStripResident * 512) return pg.cqn <= 2 ? of_size(pool_tag, Most{}, Two{}) : of_size(pool_tag, Most{}, Four{});
        return pg.cqn <= 2 ? of_size(pool_tag, Few{}, Two{}) : of_size(pool_tag, Few{}, Four{});
    };
    return pool ? launch_as(std::true_type{}) : launch_as(std::false_type{});
}

}  // namespace bnn

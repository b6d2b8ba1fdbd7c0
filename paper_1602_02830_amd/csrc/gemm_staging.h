// Pieces shared by the packed-operand GEMM kernels: staging loads of packed
// rows, the die-aware tile order, and the arguments of the fused epilogue.
#pragma once

#include "bnn_internal.h"

namespace bnn {

// Loads words [4*quad, 4*quad+4) of row `row` (quad counted from the matrix's
// first word), zero where the row or word does not exist, pad bits masked.
template <bool VEC>
__device__ inline uint4 load_quad(const uint32_t* __restrict__ P, int64_t ld, int rows, int kw,
                                  uint32_t tmask, int row, int quad) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    const int w0 = quad * 4;
    if (row < rows && w0 < kw) {
        const uint32_t* p = P + int64_t(row) * ld + w0;
        if (VEC && w0 + 4 <= kw) {
            v = *reinterpret_cast<const uint4*>(p);
        } else {
            v.x = p[0];
            if (w0 + 1 < kw) v.y = p[1];
            if (w0 + 2 < kw) v.z = p[2];
            if (w0 + 3 < kw) v.w = p[3];
        }
        const int last = kw - 1 - w0;     // position of the row's last word inside this quad
        if (last == 0) v.x &= tmask;
        else if (last == 1) v.y &= tmask;
        else if (last == 2) v.z &= tmask;
        else if (last == 3) v.w &= tmask;
    }
    return v;
}

// Words [4*quad, 4*quad+4) of the row starting at `row_ptr`, with no checks: the caller
// guarantees the row exists and the quad is complete.  One 16-byte load when VEC.
template <bool VEC>
__device__ inline uint4 load_quad_unchecked(const uint32_t* __restrict__ row_ptr, int quad) {
    const uint32_t* p = row_ptr + quad * 4;
    if (VEC) return *reinterpret_cast<const uint4*>(p);
    return make_uint4(p[0], p[1], p[2], p[3]);
}

// 16-byte load from an address that is only known to be 4-byte aligned (rows whose leading dimension is not a
// multiple of 4 words): one global_load_dwordx4, which needs dword alignment alone.
__device__ inline uint4 load_quad_any(const uint32_t* __restrict__ p) {
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));
    const quad_t v = *reinterpret_cast<const quad_t*>(p);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ inline void store_quad_any(uint32_t* p, uint4 v) {
    typedef uint32_t quad_t __attribute__((ext_vector_type(4), aligned(4)));
    *reinterpret_cast<quad_t*>(p) = quad_t{v.x, v.y, v.z, v.w};
}

// Quad `quad` of a row of kw >= 4 words, loaded without any check: a quad that is not whole, or not there, loads the
// row's last four words instead, and place_row_quad puts them right - words in place, words past the row's end zero,
// the last word's pad bits masked.
__device__ inline uint4 load_row_quad(const uint32_t* __restrict__ row, int quad, int kw) {
    return load_quad_any(row + min(4 * quad, kw - 4));
}

// left: words of the row from the quad's first one on.
__device__ inline uint4 mask_row_quad(uint4 v, int left, uint32_t tmask) {
    auto mask = [&](int w) { return left > w + 1 ? ~0u : left == w + 1 ? tmask : 0u; };
    return make_uint4(v.x & mask(0), v.y & mask(1), v.z & mask(2), v.w & mask(3));
}

__device__ inline uint4 place_row_quad(uint4 v, int quad, int kw, uint32_t tmask) {
    const int left = kw - 4 * quad;
    const bool down1 = left == 3 || left == 1, down2 = left == 2 || left == 1;     // left <= 0: all masked below
    v = make_uint4(down1 ? v.y : v.x, down1 ? v.z : v.y, down1 ? v.w : v.z, v.w);
    v = make_uint4(down2 ? v.z : v.x, down2 ? v.w : v.y, v.z, v.w);
    return mask_row_quad(v, left, tmask);
}

// Rows that allow aligned 16-byte loads (what the kernels chosen by id ask for; the automatic choice does not).
inline bool rows_16_byte_aligned(const uint32_t* P, int64_t ld) { return aligned_to(P, 16) && ld % 4 == 0; }

__device__ inline uint4 zero_unless(bool keep, uint4 v) {
    return make_uint4(keep ? v.x : 0u, keep ? v.y : 0u, keep ? v.z : 0u, keep ? v.w : 0u);
}

// Division of n < 2^31 by a number that the host knows: a multiply-high, an add and a shift (Granlund & Montgomery,
// "Division by Invariant Integers using Multiplication") instead of the 30 dependent operations of an integer division,
// which a workgroup would go through several times in a row before it can issue its first load.
struct FastDiv {
    uint32_t magic, shift;
    __device__ inline int operator()(int n) const {
        return int((__umulhi(uint32_t(n), magic) + uint32_t(n)) >> shift);
    }
};

inline FastDiv fast_div(int64_t d) {
    if (d > kMaxDim) d = kMaxDim;      // n / d is 0 either way
    uint32_t l = 0;
    while ((int64_t(1) << l) < d) ++l;
    return FastDiv{uint32_t((uint64_t((int64_t(1) << l) - d) << 32) / uint64_t(d) + 1), l};
}

// Maps the hardware's round-robin placement of consecutive workgroups on the 8
// accelerator dies (each with its own L2) to compact panels of tiles: die d
// gets the contiguous range [d*per, (d+1)*per) of logical tile ids, and
// logical ids walk the tile grid in column-major bands of 8 tile-rows, so the
// tiles resident on one die at a time share a few A panels and B panels.
constexpr int kDies = 8, kBand = 8;

struct TileMap {
    int tiles_m, tiles_n;
    int per_die;
    FastDiv band;      // by the tiles of a whole band
    FastDiv tail;      // by the rows of the last, partial band
};

inline TileMap tile_map(int64_t tiles_m, int64_t tiles_n) {
    return TileMap{int(tiles_m), int(tiles_n), int(tiles_m * tiles_n / kDies), fast_div(kBand * tiles_n),
                   fast_div(tiles_m % kBand ? tiles_m % kBand : kBand)};
}

__device__ inline void tile_of_block(int bid, const TileMap& t, int& tm, int& tn) {
    int logical = bid;
    if (bid < t.per_die * kDies) logical = (bid % kDies) * t.per_die + bid / kDies;
    const int band = t.band(logical);
    const int in_band = logical - band * kBand * t.tiles_n;
    const int rows_in_band = min(kBand, t.tiles_m - band * kBand);
    tn = rows_in_band == kBand ? in_band / kBand : t.tail(in_band);
    tm = band * kBand + (in_band - tn * rows_in_band);
}

// Arguments of the fused epilogue (Alg. 4: a^b_k = Sign(BatchNorm(a_k, theta_k)) on folded
// thresholds), used when FUSED: the tile's pre-activations never leave registers.
struct BnSignArgs {
    const int32_t* thr;        // [N]
    const uint32_t* flip_bits; // [ceil(N/32)]
    uint32_t* out;             // [M][ld_out] packed bits
    int64_t ld_out;
};

// Geometry of a convolution whose receptive fields are gathered on the fly (implicit GEMM):
// input packed NHWC [B][H][W][Cw words], taps kh x kw, row m = (b*Ho + oy)*Wo + ox.
struct ConvArgs {
    int H, W, Cw, kh, kw, stride, pad, Ho, Wo;
};

// What a launcher of one of several kernels is to do: launch if it takes the layer and is the faster one (for whom this is asked),
// launch if it takes the layer at all, or answer only, with nothing launched.
enum class ConvUse { faster, any, ask };

}  // namespace bnn

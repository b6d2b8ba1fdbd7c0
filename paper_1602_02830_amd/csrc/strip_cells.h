// Pixels, patch cells and input pixels of a strip's tile (conv_strip.hip).  Arithmetic alone, no HIP types, so that the kernels and a
// plain C++ test share it.
//
// All are counted from the tile's first image and its first padded row: at most a patch's cells (what LDS holds), a map's rows and
// columns (32767 and the padding) and a tile's pixels on from there, hence far below 2^22, where a division is exact in float32:
// with n + 0.5 held, trunc((n + 0.5) / d) has 0.5 / d of room and errs by less than (n + 0.5) / d * 2^-23.  That takes three operations
// of four cycles, where one by multiply-high takes 24 and every 32-bit product 16: with the patch cells of a lane's four pixels in
// integers, they took 1850 of the 8000 cycles before a workgroup's first product.
#pragma once

#include <math.h>
#include <stdint.h>

namespace bnn {
namespace strip {

// Sizes and reciprocals.  Wo, Ho: of the map of units (pixels or pooling windows).
struct Maps {
    float wo, ho, img_rows, pw, by_wo, by_ho, by_img_rows, by_pw;
    float h, w, cell_bytes;
};

inline Maps maps_of(int wo, int ho, int img_rows, int pw, int h, int w, int channel_words) {
    return Maps{float(wo),         float(ho),        float(img_rows), float(pw), 1.0f / float(wo),         1.0f / float(ho),
                1.0f / float(img_rows), 1.0f / float(pw), float(h),        float(w),  float(4 * channel_words)};
}

// Cell under the first tap of unit `n` of a tile that starts at unit (y, x) of its first image and at padded row row0; step: cells
// from one unit to the next.
__host__ __device__ inline int cell_of_unit(const Maps& maps, int y, int x, int row0, int step, int n) {
    const float s = float(step), u = float(n) + (float(x) + 0.5f), t = truncf(u * maps.by_wo), ux = fmaf(-t, maps.wo, u);
    const float v = t + (float(y) + 0.5f), b = truncf(v * maps.by_ho), uy = fmaf(-b, maps.ho, v);
    const float row = fmaf(b, maps.img_rows, fmaf(uy, s, -float(row0) - 0.5f * s));
    return int(fmaf(row, maps.pw, fmaf(ux, s, -0.5f * s)));
}

// Byte offset of cell `s` from row `top` of the tile's first image, 0 for a cell outside of the `images` that follow from there.
__host__ __device__ inline uint32_t input_of_cell(const Maps& maps, int pad, int h, int w, int row0, int top, int images, int s,
                                                  bool& inside) {
    const float sh = float(s) + 0.5f, py = truncf(sh * maps.by_pw), x = fmaf(-py, maps.pw, sh) - (0.5f + float(pad));
    const float rh = py + (float(row0) + 0.5f), b = truncf(rh * maps.by_img_rows);
    const float y = fmaf(-b, maps.img_rows, rh) - (0.5f + float(pad));
    const int most = images < 1 << 20 ? images : 1 << 20;
    inside = b < float(most) && uint32_t(int(y)) < uint32_t(h) && uint32_t(int(x)) < uint32_t(w);
    const float pixel = fmaf(fmaf(b, maps.h, y - float(top)), maps.w, x);
    return uint32_t(int(inside ? pixel * maps.cell_bytes : 0.0f));
}

}  // namespace strip
}  // namespace bnn

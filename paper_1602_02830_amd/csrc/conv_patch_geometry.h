// Geometry of an input patch in LDS: what the kernels that keep the pixels of a tile's receptive fields resident share.
#pragma once

#include "bnn_internal.h"
#include "gemm_staging.h"

namespace bnn {

struct PatchGeom {
    int img_rows;      // H + 2*pad: rows of a padded image
    int pw;            // W + 2*pad: patch row pitch (pixels)
    int slots;         // cells of the largest patch a tile of this layer has
    bool trim;         // most tiles need far fewer
    int cqn;           // channel quads per pixel (Cw / 4); unused when a tap is not a whole number of quads
    int kq;            // quads of K per filter row: kh * kw * cqn, or ceil(kwords / 4)
    int kwords;        // words of K per filter row: kh * kw * Cw
    FastDiv by_wo, by_ho, by_img_rows, by_pw;
};

// Rows of the padded images that the windows of BM consecutive output pixels can span, at most; the first of them is any
// multiple of `align`.
inline int64_t patch_rows(const ConvArgs& cv, int64_t BM, int64_t align) {
    const bool whole = BM % cv.Wo == 0 && align % cv.Wo == 0;                    // tiles are whole output rows
    const int64_t rows = whole ? BM / cv.Wo : (BM - 2) / cv.Wo + 2;              // output rows a tile touches
    // Image boundaries among them: none or rows / Ho - 1 where tiles follow each other from row 0 on and divide into images
    // or the reverse.
    int64_t cross = ceil_div(rows - 1, cv.Ho);
    if (whole && align % BM == 0 && cv.Ho % rows == 0) cross = 0;
    else if (whole && align % BM == 0 && rows % cv.Ho == 0) cross = rows / cv.Ho - 1;
    // From one output row to the next the window moves by `stride` rows, across a boundary by what is left of the image.
    const int64_t over = int64_t(cv.H) + 2 * cv.pad - int64_t(cv.Ho - 1) * cv.stride;
    const int64_t within = (rows - 1) * cv.stride, crossing = (rows - 1 - cross) * cv.stride + cross * over;
    return (within > crossing ? within : crossing) + cv.kh;
}

// The layer as its pooling windows see it (2 x 2, stride 2; even Ho and Wo): a map of windows, each of them the receptive
// field of a kernel with one more stride of rows and columns.  The row order of the pooled kernels is window by window.
inline ConvArgs pooled_units(ConvArgs cv) {
    cv.Ho /= 2;
    cv.Wo /= 2;
    return cv;
}

// Fills the patch geometry for tiles of BM output pixels that start at multiples of align; false if the patch takes more than
// max_bytes.  windows: cv is pooled_units of the layer and a tile BM / 4 pooling windows.
inline bool patch_geometry(const ConvArgs& cv, int64_t BM, int64_t align, int64_t max_bytes, bool windows, PatchGeom& pg) {
    const int64_t img_rows = int64_t(cv.H) + 2 * cv.pad, pw = int64_t(cv.W) + 2 * cv.pad;
    ConvArgs unit = cv;
    if (windows) {
        unit.stride *= 2;
        unit.kh += cv.stride;
        BM /= 4;
        align /= 4;
    }
    const int64_t slots = patch_rows(unit, BM, align) * pw;
    if (slots * (int64_t(cv.Cw) * 4 + 4) > max_bytes) return false;
    pg.img_rows = int(img_rows);
    pg.pw = int(pw);
    pg.slots = int(slots);
    // The largest patch crosses from image to image and starts in the middle of a row.  Counting a tile's own cells costs
    // 0.1 - 0.2 us and pays from about 1.4 times (8 images of 112 x 112, 128 -> 128 channels 15.1 -> 13.7 us, 64 of 56 x 56
    // 19.6 -> 18.7; 100 of 16 x 16, whose patches are all alike, 6.8 -> 6.9).
    pg.trim = 5 * slots >= 7 * ((ceil_div(BM, unit.Wo) - 1) * unit.stride + unit.kh) * pw;
    pg.cqn = cv.Cw / 4;
    pg.kwords = cv.kh * cv.kw * cv.Cw;
    pg.kq = (pg.kwords + 3) / 4;
    pg.by_wo = fast_div(cv.Wo);
    pg.by_ho = fast_div(cv.Ho);
    pg.by_img_rows = fast_div(img_rows);
    pg.by_pw = fast_div(pw);
    return true;
}

}  // namespace bnn

// How the strip kernels (conv_strip.hip, xnor_gemm_mfma_strip.hip, the strips of bitplane_gemm.hip) cut an output: one workgroup
// per compute unit at most, for every column tile the same number of equal strips of rows.  Arithmetic alone, no HIP types, so
// that the host, the kernels and a plain C++ test share it.
#pragma once

#include <stdint.h>

namespace bnn {

constexpr int64_t kStripUnits = 256;       // compute units
constexpr int64_t kStripStep = 32;         // strips are whole blocks of 32 rows

// Rows per strip and strips per column tile; tiles_n is at most kStripUnits.
struct StripPlan {
    int64_t rows, groups;
};
inline StripPlan strip_plan(int64_t M, int64_t tiles_n) {
    const int64_t most = kStripUnits / tiles_n, even = (M + most - 1) / most;
    const int64_t rows = (even + kStripStep - 1) / kStripStep * kStripStep;
    return StripPlan{rows, (M + rows - 1) / rows};
}

// Whether the strips keep at least `percent` of the chip at work: the rows there are against kStripUnits strips of `rows` rows.
// (kStripUnits / tiles_n is rounded down and rows up: 129 column tiles leave 127 units without a strip, 52 leave 48.)
inline bool strips_fill(int64_t M, int64_t tiles_n, int64_t rows, int percent) {
    return 100 * M * tiles_n >= percent * kStripUnits * rows;
}

// Rows [begin, end) of strip `group`.  `rows` is rounded up for every strip, so begin + rows can pass M by thousands of rows and,
// near the largest M, 2^31 (not 2^32): that sum is unsigned.
struct StripRows {
    int begin, end;
};
__host__ __device__ inline StripRows strip_rows(int group, int rows, int M) {
    const int begin = group * rows;
    const uint32_t past = uint32_t(begin) + uint32_t(rows);
    return StripRows{begin, int(past < uint32_t(M) ? past : uint32_t(M))};
}

}  // namespace bnn

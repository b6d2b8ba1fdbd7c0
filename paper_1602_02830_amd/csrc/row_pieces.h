// Rows of any length in pieces of 128 elements, of which a row's last may be partial (pack_sign.hip, bn_sign_pack.hip): what the lanes of a
// group of eight load and store.  Arithmetic alone, no HIP types, so that the host, the kernels and a plain C++ test share it.
#pragma once

#include <stdint.h>

namespace bnn {

// A row of n <= 2^31 - 1 elements, at least 4 of them.  Its words come from the host: n + 31 does not fit the 32 bits that a kernel
// holds n in.
struct PieceRow {
    int n, words;

    __host__ __device__ int pieces() const { return (words + 3) >> 2; }

    // Elements 32 u + 4 q on of a piece: loaded from `at`, with the `past` elements before them, four where there are none.
    struct Quad {
        int at, past;
    };
    __host__ __device__ Quad quad(int piece, int u, int q) const {
        const int first = piece * 128 + q * 4 + 32 * u, at = first < n - 4 ? first : n - 4;
        return Quad{at, first - at < 4 ? first - at : 4};
    }

    // Word u of a piece, the row's last where there is none.
    __host__ __device__ int word(int piece, int u) const {
        const int w = piece * 4 + u;
        return w < words ? w : words - 1;
    }

    // Whether lane q of a group stores one: word q of the piece.
    __host__ __device__ bool stores(int piece, int q) const { return q < 4 && piece * 4 + q < words; }
};

inline PieceRow piece_row(int64_t n) { return PieceRow{int(n), int((n + 31) >> 5)}; }

// Pieces of a row of so many words; none where more than a fifth of their words would not exist (hence rows of 97 elements and more).
inline int64_t pieces_of(int64_t words) {
    const int64_t pieces = (words + 3) / 4;
    return 16 * pieces <= 5 * words ? pieces : 0;
}

}  // namespace bnn

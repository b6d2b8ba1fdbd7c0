"""CPU-only tests of rows in pieces of 128 elements (csrc/row_pieces.h): what the lanes load and store, built by the host compiler with
every signed overflow an error, and the row that the entry points hand to their kernels."""
import os
import subprocess

from test_launch_limits import A, C, FLIP, OUT, THR
from test_strip_cut import seen_by_launch  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_02830_amd", "csrc")
LONGEST = 2 ** 31 - 1

PIECES = r"""
#include <stdlib.h>
#define __host__
#define __device__
#include "row_pieces.h"
/* n ...: the first and last pieces of a row of n elements, every element against its own division */
int main(int argc, char** argv) {
    for (int a = 1; a < argc; ++a) {
        const int64_t n = atoll(argv[a]), words = n / 32 + (n % 32 != 0), pieces = words / 4 + (words % 4 != 0);
        const bnn::PieceRow row = bnn::piece_row(n);
        if (row.n != n || row.words != words || row.pieces() != pieces) return 1;
        if (bnn::pieces_of(words) != (5 * words >= 16 * pieces ? pieces : 0)) return 2;
        for (int64_t p = 0; p < pieces; p = p == 3 && pieces > 8 ? pieces - 4 : p + 1)
            for (int q = 0; q < 8; ++q) {
                if (row.stores(int(p), q) != (q < 4 && 4 * p + q < words)) return 3;
                for (int u = 0; u < 4; ++u) {
                    const int64_t first = 128 * p + 32 * u + 4 * q, w = 4 * p + u;
                    const bnn::PieceRow::Quad quad = row.quad(int(p), u, q);
                    if (quad.at < 0 || quad.at + int64_t(4) > n || quad.past < 0 || quad.past > 4) return 4;
                    for (int e = 0; e < 4; ++e) {                        /* bit e of the nibble comes from loaded element past + e */
                        if (first + e < n ? quad.past + e > 3 || quad.at + quad.past + e != first + e : quad.past + e <= 3) return 5;
                    }
                    if (row.word(int(p), u) != (w < words ? w : words - 1)) return 6;
                }
            }
    }
    return 0;
}
"""


def test_pieces_take_every_element_of_rows_of_any_length(tmp_path):
    src, exe = tmp_path / "pieces.cpp", tmp_path / "pieces"
    src.write_text(PIECES)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", f"-I{CSRC}", str(src),
                    "-o", str(exe)], check=True)
    for sizes in (range(4, 700), (784, 4095, 6001, 8191, 2 ** 24 + 5), range(LONGEST - 160, LONGEST + 1)):
        r = subprocess.run([str(exe), *map(str, sizes)], stderr=subprocess.PIPE, text=True)
        assert r.returncode == 0, (sizes, r.returncode, r.stderr)


def test_long_rows_reach_their_kernels_with_their_words(seen_by_launch):  # noqa: F811
    """Rows of integers up to the ABI's longest, rows of reals up to what the last-level cache holds."""
    for n in (97, 1000, 2 ** 26 - 5, LONGEST - 31, LONGEST - 30, LONGEST):
        got = seen_by_launch("piece_row", ("bnn_bn_sign_pack", (C, n, 1, n, THR, FLIP, OUT, (n + 31) // 32, 0)))
        assert got == [n | (n + 31) // 32 << 32], n
    for n in (97, 1000, 2 ** 26 - 5):
        assert seen_by_launch("piece_row_2", ("bnn_pack_sign", (A, 1, n, n, OUT, (n + 31) // 32, 0))) == [n | (n + 31) // 32 << 32], n

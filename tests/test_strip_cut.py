"""CPU-only tests of how the strip kernels cut an output (csrc/strip_cut.h, csrc/strip_cells.h): the functions that give a workgroup
its rows and a pixel its patch cell, built by the host compiler with every signed overflow an error, and the launches of the entry
points at the sizes where the strips' ends lie beyond 2^31."""
import json
import os
import subprocess
import sys

import pytest

from test_launch_limits import A, B, C, CHILD, FLIP, LIB, OUT, RUNTIME, THR, WB, launches_of  # noqa: F401

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_02830_amd", "csrc")

COVER = r"""
#include <stdio.h>
#include <stdlib.h>
#define __host__
#define __device__
#include "strip_cut.h"
int main(int argc, char** argv) {                   /* M tiles_n ...: the strips of each, in order, cover [0, M) */
    for (int a = 1; a + 1 < argc; a += 2) {
        const int64_t M = atoll(argv[a]), tiles_n = atoll(argv[a + 1]);
        const bnn::StripPlan plan = bnn::strip_plan(M, tiles_n);
        if (plan.groups * tiles_n > bnn::kStripUnits || plan.rows % bnn::kStripStep != 0 || plan.rows > M + 31) return 1;
        int64_t next = 0;
        for (int group = 0; group < int(plan.groups); ++group) {
            const bnn::StripRows r = bnn::strip_rows(group, int(plan.rows), int(M));
            if (r.begin != next || r.end <= r.begin || r.end - r.begin > plan.rows || r.end > M) {
                fprintf(stderr, "M %lld, %lld column tiles: strip %d is [%d, %d)\n", (long long)M, (long long)tiles_n, group, r.begin, r.end);
                return 2;
            }
            next = r.end;
        }
        if (next != M) return 3;
    }
    return 0;
}
"""

CELLS = r"""
#include <stdio.h>
#include <stdlib.h>
#define __host__
#define __device__
#include "strip_cells.h"
/* Wo Ho H W pad stride channel_words units: float divisions against integer ones, for tiles of 512 units that start anywhere */
int main(int, char** argv) {
    int a[8];
    for (int i = 0; i < 8; ++i) a[i] = atoi(argv[1 + i]);
    const int Wo = a[0], Ho = a[1], H = a[2], W = a[3], pad = a[4], step = a[5], cw = a[6], tile = a[7];
    const int img_rows = H + 2 * pad, pw = W + 2 * pad;
    const bnn::strip::Maps maps = bnn::strip::maps_of(Wo, Ho, img_rows, pw, H, W, cw);
    unsigned seed = 12345u;
    auto below = [&](int n) { seed = seed * 1664525u + 1013904223u; return int((uint64_t(seed) * uint64_t(n)) >> 32); };
    for (int trial = 0; trial < 400; ++trial) {
        const int y = trial < 2 ? (trial ? Ho - 1 : 0) : below(Ho), x = trial < 4 ? (trial & 2 ? Wo - 1 : 0) : below(Wo);
        const int row0 = y * step, images = trial % 3 ? 1 + below(600) : 1, top = row0 - pad < 0 ? 0 : row0 - pad < H ? row0 - pad : H - 1;
        int cells = 1;
        for (int n = 0; n < tile; ++n) {
            const int t = (x + n) / Wo, ux = (x + n) % Wo, b = (y + t) / Ho, uy = (y + t) % Ho;
            const int want = (b * img_rows + uy * step - row0) * pw + ux * step;
            if (bnn::strip::cell_of_unit(maps, y, x, row0, step, n) != want) return 1;
            if (want > cells) cells = want;
        }
        cells = cells + 3 * pw < 16384 ? cells + 3 * pw : 16384;             /* more cells than that do not fit LDS */
        for (int s = 0; s < cells; ++s) {
            const int r = row0 + s / pw, b = r / img_rows, cy = r % img_rows - pad, cx = s % pw - pad;
            const bool there = b < images && cy >= 0 && cy < H && cx >= 0 && cx < W;
            bool inside;
            const uint32_t at = bnn::strip::input_of_cell(maps, pad, H, W, row0, top, images, s, inside);
            if (inside != there) return 2;
            if (there && b == 0 && cy < top) continue;                        /* before the patch's first row: never asked for */
            if (at != (there ? 4u * cw * ((uint32_t(b) * H + cy - top) * W + cx) : 0u)) return 3;
        }
    }
    return 0;
}
"""

# The last strip's unclamped end reaches 2^31 from here on.
PAST_INT = {1: 2147475457, 2: 2147479553, 4: 2147481601}
LARGEST = 2 ** 31 - 1025


@pytest.fixture(scope="module")
def cover(tmp_path_factory):
    folder = tmp_path_factory.mktemp("strips")
    src, exe = folder / "cover.cpp", folder / "cover"
    src.write_text(COVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", f"-I{CSRC}", str(src),
                    "-o", str(exe)], check=True)
    return lambda sizes: subprocess.run([str(exe), *(str(v) for pair in sizes for v in pair)], stderr=subprocess.PIPE, text=True)


def test_cells_in_float32_are_the_integer_ones(tmp_path):
    src, exe = tmp_path / "cells.cpp", tmp_path / "cells"
    src.write_text(CELLS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", f"-I{CSRC}", str(src),
                    "-o", str(exe)], check=True)
    # Wo, Ho, H, W, pad, step, channel words, units of a tile: the ConvNet's maps, single pixels, the tallest and widest maps and
    # paddings that are admitted, strides of pooling windows
    for sizes in ((16, 16, 16, 16, 1, 1, 8, 512), (14, 14, 28, 28, 1, 2, 4, 128), (1, 1, 1, 1, 0, 1, 144, 512), (3, 1, 2, 4, 1, 2, 4, 512),
                  (30, 1030, 1030, 34, 1, 1, 4, 512), (7, 32767, 32767, 9, 0, 1, 4, 512), (5, 32767, 32767, 7, 0, 1, 4, 512),
                  (8000, 3, 3, 8000, 1, 1, 4, 512), (2670, 13589, 32767, 5, 4000, 3, 4, 32), (333, 127, 1000, 2667, 3, 8, 36, 128)):
        assert subprocess.run([str(exe), *map(str, sizes)]).returncode == 0, sizes


def test_strips_cover_the_rows_of_every_size(cover):
    sizes = [(M + d, t) for t, M in PAST_INT.items() for d in (-1, 0, 1)] + [(LARGEST, t) for t in (1, 2, 3, 4, 52, 129, 256)]
    sizes += [(M, t) for M in (1, 31, 32, 33, 8191, 8192, 8193, 40960, 100001) for t in (1, 3, 8, 31, 128, 129, 255, 256)]
    r = cover(sizes)
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("tiles_n,M", sorted(PAST_INT.items()) + [(t, LARGEST) for t in PAST_INT])
def test_strip_kernels_take_rows_up_to_the_limit(launches_of, tiles_n, M):  # noqa: F811
    """One workgroup of 512 threads per strip and column tile: a convolution of 2 x 2 maps (window 3 x 3, padding 2, 16 outputs an
    image), the same with its pooling, and a fused layer of K = 600 (whose call refuses four column tiles of that many rows)."""
    N, K = 128 * tiles_n, 600
    images = min(-(-M // 16), LARGEST // 16)
    conv = (A, images, 2, 2, 128, WB, 36, N, 3, 3, 1, 2)
    runs = launches_of(("bnn_conv_bn_sign_pack", (*conv, THR, FLIP, OUT, N // 32, 0)),
                       ("bnn_conv_pool_windows_bn_sign_pack", (*conv, 2, THR, FLIP, OUT, N // 32, 0)),
                       ("bnn_xnor_gemm_bn_sign_pack", (A, 19, B, 19, M, N, K, THR, FLIP, OUT, N // 32, 0)))
    for st, log in runs if tiles_n <= 2 else runs[:2]:
        assert st == 0 and log == [[256, 512, A]]


def strips(M, N, tile_n):
    """Workgroups of 512 threads that an M x N output in strips has."""
    t = -(-N // tile_n)
    rows = -(-(-(-M // (256 // t))) // 32) * 32
    return [[-(-M // rows) * t, 512, A]]


@pytest.mark.parametrize("M,N,K,taken", [
    (2000, 6656, 784, True), (2000, 5504, 600, True), (1164, 19579, 600, False), (3060, 16512, 600, False), (1853, 4224, 1002, False),
    (1853, 4224, 800, True), (5105, 1732, 862, True), (36308, 238, 926, True), (795, 10452, 991, True), (15227, 512, 987, False), (609, 12519, 912, False), (609, 12519, 832, True), (10000, 4096, 784, True), (10000, 3000, 700, True), (4000, 6656, 784, True), (4000, 12000, 784, False), (10000, 6656, 784, False), (10000, 12000, 600, False),
    (4000, 16512, 784, False), (10000, 16640, 784, False), (4141, 7168, 810, False), (4112, 15104, 784, True), (4000, 32768, 784, True),
    (343, 21148, 784, False), (352, 20480, 832, False), (384, 21248, 705, False), (384, 21248, 704, True), (343, 21148, 640, True),
    (310, 20480, 784, True), (404, 20839, 800, True)])
def test_row_strips_are_taken_where_they_fill_the_chip(launches_of, M, N, K, taken):  # noqa: F811
    kw = (K + 31) // 32
    (st, log), = launches_of(("bnn_xnor_gemm_bn_sign_pack", (A, kw, B, kw, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)))
    assert st == 0 and (log == strips(M, N, 128)) == taken


@pytest.mark.parametrize("M,N,lda,ldb,ld_out", [
    (160, 32768, 453437, 19, 1024), (160, 32768, 453438, 19, 1024), (160, 32768, 19, 19, 453438), (160, 32768, 2 ** 40, 19, 1024),
    (40960, 33, 19, 2 ** 22 - 1, 2), (40960, 33, 19, 2 ** 22, 2), (2000, 8000, 360000, 19, 250)])
def test_row_strips_are_taken_however_far_apart_rows_lie(launches_of, M, N, lda, ldb, ld_out):  # noqa: F811
    """On both sides of the distances whose byte offsets fit 32 bits."""
    (st, log), = launches_of(("bnn_xnor_gemm_bn_sign_pack", (A, lda, B, ldb, M, N, 600, THR, FLIP, OUT, ld_out, 0)))
    assert st == 0 and log == strips(M, N, 128)


@pytest.mark.parametrize("M,N,K,taken", [
    (10000, 4096, 784, True), (10000, 4096, 300, True), (2400, 8192, 257, False), (12300, 1226, 440, False), (5190, 3247, 258, False),
    (8192, 4096, 300, True), (16412, 3697, 309, True), (2539, 8192, 496, False), (2539, 8192, 513, True), (9101, 1701, 743, False),
    (9633, 1920, 788, True), (1500, 66048, 300, False), (6000, 16640, 784, True)])
def test_byte_layer_strips_are_taken_where_they_fill_the_chip(launches_of, M, N, K, taken):  # noqa: F811
    kw = (K + 31) // 32
    (st, log), = launches_of(("bnn_bitplane_gemm_bn_sign_pack", (A, 8 * kw, B, kw, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)))
    assert st == 0 and (log == strips(M, N, 512)) == taken


@pytest.mark.parametrize("B_,H,W,Cin,Cout,window,stride,pad,taken", [
    (256, 16, 16, 256, 256, (3, 3), 1, 1, True), (256, 32, 32, 128, 128, (3, 3), 1, 1, True), (128, 28, 28, 128, 256, (3, 3), 1, 1, True),
    (256, 16, 16, 128, 256, (3, 3), 1, 1, True),                                                       # the ConvNet's layers
    (47, 14, 14, 512, 12288, (3, 3), 1, 1, False), (54, 14, 14, 256, 5632, (3, 3), 1, 1, False), (18, 14, 14, 512, 8448, (3, 3), 1, 1, False),
    (5, 14, 14, 512, 8704, (3, 3), 1, 1, True), (40, 28, 28, 128, 9984, (3, 3), 1, 1, False), (29, 28, 28, 512, 3840, (3, 3), 1, 1, True),
    (185, 16, 16, 128, 512, (3, 3), 1, 1, False), (140, 16, 16, 128, 512, (3, 3), 1, 1, True), (200, 16, 16, 128, 512, (3, 3), 1, 1, True),
    (185, 16, 16, 256, 512, (3, 3), 1, 1, True), (73, 14, 51, 256, 512, (1, 4), 1, 0, False),
    (571, 32, 32, 384, 128, (1, 4), 3, 0, False), (145, 89, 89, 128, 128, (7, 1), 1, 3, False), (189, 56, 56, 1024, 128, (2, 1), 1, 0, False),
    (493, 28, 28, 384, 384, (4, 1), 1, 2, False), (64, 32, 32, 128, 128, (1, 4), 1, 0, False), (100, 32, 32, 256, 128, (1, 4), 1, 0, True),
    (225, 28, 28, 128, 512, (3, 3), 2, 1, True), (356, 32, 32, 128, 256, (3, 3), 2, 1, False), (17, 96, 96, 128, 512, (3, 3), 2, 0, True),
    (283, 34, 74, 256, 256, (3, 1), 2, 0, True), (1520, 12, 20, 128, 512, (4, 1), 3, 1, False), (14685, 28, 19, 128, 64, (4, 1), 3, 1, False)])
def test_convolution_strips_are_taken_where_they_are_faster(launches_of, B_, H, W, Cin, Cout, window, stride, pad, taken):  # noqa: F811
    kh, kw = window
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    args = (A, B_, H, W, Cin, WB, kh * kw * Cin // 32, Cout, kh, kw, stride, pad)
    tail = (THR, FLIP, OUT, (Cout + 31) // 32, 0)
    (st, log), (st_pool, log_pool) = launches_of(("bnn_conv_bn_sign_pack", (*args, *tail)),
                                                 ("bnn_conv_pool_windows_bn_sign_pack", (*args, 2, *tail)))
    want = strips(B_ * Ho * Wo, Cout, 128)
    assert st == 0 and (log == want) == taken
    if (Ho | Wo) % 2 == 0:
        assert st_pool in (0, 3) and (log_pool != want or taken)


def test_pooled_strips_are_taken_where_pooled_tiles_leave_units_unfilled(launches_of):  # noqa: F811
    """228 images of 34 x 92, 256 -> 512, 3 x 1: three plain tiles share a compute unit, of the pooled ones not."""
    args, tail = (A, 228, 34, 92, 256, WB, 24, 512, 3, 1, 1, 0), (THR, FLIP, OUT, 16, 0)
    (st, log), (st_pool, log_pool) = launches_of(("bnn_conv_bn_sign_pack", (*args, *tail)),
                                                 ("bnn_conv_pool_windows_bn_sign_pack", (*args, 2, *tail)))
    want = strips(228 * 32 * 92, 512, 128)
    assert (st, st_pool) == (0, 0) and log != want and log_pool == want


@pytest.mark.parametrize("B_,H,W,Cin,Cout,stride", [(38836, 96, 96, 384, 5410, 1), (131071, 64, 64, 256, 11136, 1),
                                                    (280956, 14, 84, 128, 21632, 1), (44239, 96, 172, 128, 16640, 2)])
def test_convolutions_of_more_tiles_than_one_launch_holds_take_strips(launches_of, B_, H, W, Cin, Cout, stride):  # noqa: F811
    """Strips that leave much of the chip idle, and no tiled kernel that could launch."""
    args = (A, B_, H, W, Cin, WB, 9 * Cin // 32, Cout, 3, 3, stride, 1)
    tail = (THR, FLIP, OUT, (Cout + 31) // 32, 0)
    want = strips(B_ * (H // stride) * (W // stride), Cout, 128)
    plain, pooled, windows = launches_of(("bnn_conv_bn_sign_pack", (*args, *tail)), ("bnn_conv_pool_bn_sign_pack", (*args, 2, *tail)),
                                         ("bnn_conv_pool_windows_bn_sign_pack", (*args, 2, *tail)))
    assert plain == windows == [0, want] and pooled == ([0, want] if H == W == 64 else [3, []])


@pytest.mark.parametrize("B_,H,W,Cin,Cout,k,stride,pad,faster", [
    (93, 28, 28, 768, 32, 3, 1, 1, False), (77, 28, 28, 768, 32, 3, 1, 1, True), (1, 56, 56, 512, 21028, 3, 1, 0, False),
    (5, 56, 183, 128, 17696, 3, 2, 1, False), (3, 32, 128, 512, 128, 3, 1, 1, False), (14, 16, 128, 128, 128, 7, 1, 3, False),
    (30, 16, 128, 128, 128, 7, 1, 3, True), (59, 26, 26, 1024, 384, 1, 1, 0, False), (15, 28, 14, 1024, 1718, 1, 1, 0, True),
    (2, 6, 6, 128, 70, 3, 1, 1, True), (8, 60, 60, 96, 64, 3, 1, 1, False)])
def test_pooled_maps_are_taken_and_advised_where_one_launch_is_faster(launches_of, B_, H, W, Cin, Cout, k, stride, pad, faster):  # noqa: F811
    """The call takes any even map of whole channel quads; bnn_conv_pool_form names it where it is the faster form."""
    words = -(-k * k * Cin // 128) * 4
    (st, log), (form, none) = launches_of(
        ("bnn_conv_pool_windows_bn_sign_pack", (A, B_, H, W, Cin, WB, words, Cout, k, k, stride, pad, 2, THR, FLIP, OUT,
                                                (Cout + 31) // 32, 0)),
        ("bnn_conv_pool_form", (B_, H, W, Cin, Cout, k, k, stride, pad, 2)))
    assert (st, len(log)) == ((0, 1) if Cin % 128 == 0 else (3, 0))
    assert (form, none) == (2 if faster else 0, [])


@pytest.mark.parametrize("B_,H,W,Cin", [(4, 32, 32, 96), (3, 8, 8, 64), (40, 32, 32, 768), (2, 64, 64, 128)])
def test_pooled_maps_of_whole_rows_keep_their_call(launches_of, B_, H, W, Cin):  # noqa: F811
    """What bnn_conv_pool_bn_sign_pack takes, the call for any map takes as well with the same launch where Cin is a multiple of 128."""
    words = -(-9 * Cin // 128) * 4
    args = (A, B_, H, W, Cin, WB, words, 64, 3, 3, 1, 1, 2, THR, FLIP, OUT, 2, 0)
    (st, log), (st_any, log_any), (form, _) = launches_of(("bnn_conv_pool_bn_sign_pack", args),
                                                          ("bnn_conv_pool_windows_bn_sign_pack", args),
                                                          ("bnn_conv_pool_form", (B_, H, W, Cin, 64, 3, 3, 1, 1, 2)))
    assert form == 1
    assert st == 0 and len(log) == 1
    assert (st_any, log_any) == ((0, log) if Cin % 128 == 0 else (3, []))


@pytest.fixture(scope="module")
def seen_by_launch(tmp_path_factory):
    """(what, calls) -> that expression of the stand-in for every call's launch: its local memory beside what the kernel declares, its
    kernel, its workgroups, the PieceRow among its arguments."""
    folder = tmp_path_factory.mktemp("seen")
    line = "launch_log[launches][2] = *(uint64_t*)args[0];"
    assert line in RUNTIME and "(void)f; (void)shared;" in RUNTIME

    def run(what, *calls):
        src, so = folder / f"{what}.c", folder / f"{what}.so"
        if not so.exists():
            expression = {"local_memory": "shared", "kernel": "(uint64_t)f", "workgroups": "g.x",
                          "piece_row": "*(uint64_t*)args[3]", "piece_row_2": "*(uint64_t*)args[2]"}[what]
            src.write_text(RUNTIME.replace(line, f"launch_log[launches][2] = {expression};"))
            subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
        r = subprocess.run([sys.executable, "-c", CHILD, str(so), LIB], input=json.dumps([[n, list(a)] for n, a in calls]),
                           stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
        assert r.returncode == 0, r.stderr
        return [log[0][2] for status, log in json.loads(r.stdout) if status == 0 and len(log) == 1]

    return run


@pytest.mark.parametrize("B_,H,W,Cin,Cout,k,rows,taken", [
    (1, 8, 8, 256, 128, 3, 32, True), (10, 14, 14, 256, 256, 3, 32, True), (10, 14, 14, 512, 256, 3, 32, True),
    (63, 16, 16, 128, 64, 3, 64, True), (4, 30, 30, 256, 512, 3, 64, True), (4, 30, 30, 512, 512, 3, 64, False),    # 64 rows: K <= 2560
    (27, 30, 30, 256, 64, 3, 96, True), (25, 30, 30, 512, 128, 3, 96, True),
    (22, 32, 32, 256, 64, 3, 96, False), (44, 16, 32, 256, 64, 3, 96, False), (30, 32, 32, 256, 64, 3, 128, True),    # map rows of whole blocks: pairs of them
    (12, 28, 28, 256, 264, 3, 128, True), (41, 28, 28, 512, 128, 3, 128, True),
    (1, 15, 15, 256, 11264, 3, 128, True), (1, 15, 15, 256, 11008, 3, 128, False),                                   # 60 % of the chip
    (1, 13, 10, 256, 11008, 3, 96, False), (1, 10, 10, 256, 11008, 3, 64, True),                                     # asked from 96 rows on
    (10, 14, 14, 128, 128, 5, 32, False), (156, 14, 14, 128, 128, 5, 128, False), (190, 14, 14, 128, 128, 5, 160, True)])
def test_short_convolution_strips_are_taken_where_they_are_faster(seen_by_launch, B_, H, W, Cin, Cout, k, rows, taken):
    """By the kernel that is launched, against that of a layer of the same channels in strips of 256 or 512 rows."""
    def call(B_, H, W, Cout):
        return ("bnn_conv_bn_sign_pack", (A, B_, H, W, Cin, WB, k * k * Cin // 32, Cout, k, k, 1, k // 2, THR, FLIP, OUT,
                                          (Cout + 31) // 32, 0))

    assert strips(B_ * H * W, Cout, 128) == [[-(-B_ * H * W // rows) * -(-Cout // 128), 512, A]]
    got, strip = seen_by_launch("kernel", call(B_, H, W, Cout), call(256, 16, 16, 256) if Cin <= 256 else call(256, 8, 8, 512))
    assert (got == strip) == taken


@pytest.mark.parametrize("B_,HW,Cin", [(100, 32, 768), (168, 32, 1024), (22, 32, 256), (8, 16, 512)])
def test_pooled_patches_of_whole_rows_are_no_larger_than_plain_ones(seen_by_launch, B_, HW, Cin):
    """Tiles of pooling windows that are whole image rows cover the same rows as the tiles of the unpooled layer."""
    args = (A, B_, HW, HW, Cin, WB, 9 * Cin // 32, 64, 3, 3, 1, 1)
    plain, pooled = seen_by_launch("local_memory", ("bnn_conv_bn_sign_pack", (*args, THR, FLIP, OUT, 2, 0)),
                                   ("bnn_conv_pool_bn_sign_pack", (*args, 2, THR, FLIP, OUT, 2, 0)))
    assert 0 < pooled <= plain


def product(fused, M, N, K, ld=0):
    ld = ld or (K + 31) // 32
    return (("bnn_xnor_gemm_bn_sign_pack", (A, ld, B, ld, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)) if fused else
            ("bnn_xnor_gemm", (A, ld, B, ld, C, N, M, N, K, 0)))


@pytest.mark.parametrize("fused,M,N,K,ld,staged", [
    (True, 512, 1024, 4096, 128, True), (False, 512, 1024, 4096, 128, True), (True, 512, 1024, 4097, 129, True), (True, 512, 1024, 4064, 127, True),
    (True, 800, 960, 4160, 130, False), (False, 800, 960, 4160, 130, False), (True, 800, 960, 4168, 131, False),     # 33 quads
    (True, 800, 960, 4097, 132, False), (True, 800, 960, 5120, 160, True), (True, 800, 960, 3968, 124, False),
    (False, 512, 640, 6200, 194, True), (True, 512, 640, 6200, 194, False), (True, 512, 640, 7300, 229, True), (False, 512, 640, 8704, 272, False),
    (False, 800, 960, 12000, 375, True), (False, 512, 640, 12000, 375, False), (True, 200, 1000, 4096, 128, False),
    (False, 512, 640, 3500, 110, True), (True, 512, 640, 3500, 110, False), (False, 512, 640, 3900, 122, False)])
def test_k_split_products_are_staged_where_that_is_faster(seen_by_launch, fused, M, N, K, ld, staged):
    got, direct, lines = seen_by_launch("kernel", product(fused, M, N, K, ld), product(fused, 512, 640, 2000), product(fused, 512, 640, 4096))
    assert direct != lines and got == (lines if staged else direct)


@pytest.mark.parametrize("fused,M,N,K,ld,rest", [
    (False, 1000, 1000, 4097, 129, True), (False, 1000, 1000, 4500, 160, True), (False, 1000, 1000, 4900, 160, True),        # 1, 4, 7 quads
    (False, 1000, 1000, 5120, 160, True), (False, 1000, 1000, 5121, 161, False), (False, 1000, 1000, 4096, 129, False),     # 8, 9, none
    (False, 1000, 1000, 1024, 33, False),                                                                                   # less than a round
    (False, 512, 640, 4500, 160, True), (False, 512, 640, 4900, 160, True), (False, 512, 640, 5121, 161, False),
    (True, 1000, 1000, 4500, 160, True), (True, 1000, 1000, 4900, 160, True), (True, 1280, 1200, 4352, 136, True),
    (True, 1280, 1200, 4600, 144, True), (True, 512, 640, 4500, 160, False), (True, 512, 640, 4900, 160, False)])
def test_a_short_rest_of_k_is_loaded_with_the_first_round(seen_by_launch, fused, M, N, K, ld, rest):
    """Products staged in rounds of 32 quads, one to eight quads past whole rounds; not fused 32 x 32 tiles."""
    tiles = (512, 640) if (M, N) == (512, 640) else (1000, 1000)
    got, with_rest, whole = seen_by_launch("kernel", product(fused, M, N, K, ld), product(fused, *tiles, 4097, 129), product(fused, *tiles, 4096))
    assert (got == with_rest != whole) == rest


@pytest.mark.parametrize("fused,M,N,K,workgroups", [
    (True, 416, 2368, 4580, 13 * 74), (False, 539, 1883, 8704, 17 * 59), (False, 1000, 1000, 4097, 16 * 32), (True, 1000, 1000, 4097, 16 * 32),
    (True, 1280, 1200, 4352, 20 * 38), (True, 672, 2235, 4480, None), (True, 1292, 1184, 4352, None), (False, 800, 1947, 6528, None)])
def test_k_split_tiles_of_two_rows_fill_the_compute_units(seen_by_launch, fused, M, N, K, workgroups):
    """As many 64 x 32 tiles as two (three, with more than 1024 tiles of 32 x 32) fill every compute unit; else 32 x 32 tiles up to 1024
    of them, and the tiles with K in one piece above."""
    (got,) = seen_by_launch("workgroups", product(fused, M, N, K))
    if workgroups is None:
        assert got <= -(-M // 64) * -(-N // 128)
    else:
        assert got == workgroups

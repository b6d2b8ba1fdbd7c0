"""CPU-only tests of the launches themselves: what grid an entry point asks the runtime for at sizes near the limits of the
ABI.  A child process puts a stand-in for the runtime's launch call in front of the real one - it notes each launch,
refuses what the runtime refuses (a dimension of 2^32 work items or more) and runs nothing - and calls the library with
addresses that nothing reads."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1602_02830_amd", "libbnn_hip.so")

RUNTIME = r"""
#include <stddef.h>
#include <stdint.h>
typedef struct { uint32_t x, y, z; } dim3;
static dim3 next_grid, next_block;
static size_t next_shared;
static void* next_stream;
static int error;
int64_t launches;
uint64_t launch_log[64][3];          /* workgroups, threads, first kernel argument */

int __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, void* stream) {
    next_grid = g; next_block = b; next_shared = shared; next_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, void** stream) {
    *g = next_grid; *b = next_block; *shared = next_shared; *stream = next_stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t shared, void* stream) {
    (void)f; (void)shared; (void)stream;
    if ((uint64_t)g.x * b.x >> 32 || g.x == 0 || g.y == 0 || g.z == 0) return error = 9;
    if (launches < 64) {
        launch_log[launches][0] = (uint64_t)g.x * g.y * g.z;
        launch_log[launches][1] = (uint64_t)b.x * b.y * b.z;
        launch_log[launches][2] = *(uint64_t*)args[0];
    }
    ++launches;
    return 0;
}
int hipGetLastError(void) { int e = error; error = 0; return e; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int* value, int attribute, int device) { (void)attribute; (void)device; *value = 256; return 0; }
"""

CHILD = r"""
import ctypes, json, sys
runtime = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
count = ctypes.c_int64.in_dll(runtime, "launches")
log = (ctypes.c_uint64 * 3 * 64).in_dll(runtime, "launch_log")
out = []
for name, args in json.load(sys.stdin):
    # integers of the ABI that are not int64 (window sizes, kernel ids) are passed as such in registers or stack slots alike
    count.value = 0
    status = getattr(lib, name)(*[ctypes.c_int64(a) for a in args])
    out.append([status, [list(log[i]) for i in range(min(count.value, 64))]])
print(json.dumps(out))
"""

A, B, C, THR, FLIP, OUT = (i << 44 for i in range(1, 7))          # operand addresses
WB = B


@pytest.fixture(scope="module")
def launches_of(tmp_path_factory):
    """calls -> [(status, [[workgroups, threads, first argument], ...]), ...]"""
    folder = tmp_path_factory.mktemp("runtime")
    src, so = folder / "runtime.c", folder / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)

    def run(*calls):
        r = subprocess.run([sys.executable, "-c", CHILD, str(so), LIB], input=json.dumps([[n, list(a)] for n, a in calls]),
                           stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout)

    return run


def test_the_stand_in_sees_launches(launches_of):
    (st, log), (st_empty, log_empty) = launches_of(("bnn_pack_sign", (A, 4, 100, 100, OUT, 4, 0)),
                                                   ("bnn_pack_sign", (A, 0, 100, 100, OUT, 4, 0)))
    assert st == 0 and log == [[1, 256, A]]
    assert st_empty == 0 and log_empty == []


@pytest.mark.parametrize("rows,cols", [(2 ** 31 - 1, 33), (2 ** 31 - 1, 1), (2 ** 26, 2 ** 12), (2 ** 24, 2 ** 31 - 1), (10 ** 6, 10 ** 5)])
def test_bit_plane_packer_stays_below_the_work_item_limit(launches_of, rows, cols):
    kw = (cols + 31) // 32
    (st, log), = launches_of(("bnn_pack_bitplanes", (A, rows, cols, cols, OUT, 8 * kw, 0)))
    assert st == 0 and len(log) == 1 and log[0][1] == 256
    assert log[0][0] >= min(-(-rows * kw // 256), 2 ** 23)


@pytest.mark.parametrize("rows,cols", [(2 ** 22, 2 ** 14), (2 ** 24 - 1, 4096), (2 ** 31 - 1, 128), (2 ** 20, 2 ** 18)])
def test_streaming_kernels_stay_below_the_work_item_limit(launches_of, rows, cols):
    """On both sides of the sizes whose rows of whole 128-element units still fit one launch (2^24 - 1 workgroups)."""
    kw = cols // 32
    for st, log in launches_of(("bnn_pack_sign", (A, rows, cols, cols, OUT, kw, 0)),
                               ("bnn_bn_sign_pack", (C, cols, rows, cols, THR, FLIP, OUT, kw, 0))):
        assert st == 0 and len(log) == 1 and log[0][1] == 256


def covers(log, first, ld, M, tiles_n, tile_m):
    """Launches of tiles of tile_m rows that start at consecutive rows of the first operand and take all M of them."""
    row = 0
    for blocks, threads, address in log:
        assert address == first + 4 * ld * row and blocks % tiles_n == 0 and blocks * threads < 2 ** 32
        row += blocks // tiles_n * tile_m
    return M <= row < M + tile_m


@pytest.mark.parametrize("M,N,K", [(2 ** 22, 4096, 64), (33_500_000, 512, 27), (2 ** 31 - 1025, 33, 96), (2 ** 31 - 1025, 300, 33),
                                   (2 ** 22, 4096, 0), (2 ** 31 - 1025, 33, 128), (2 ** 31 - 1025, 600, 200), (5, 2 ** 31 - 1025, 96)])
@pytest.mark.parametrize("fused", [False, True])
def test_first_layers_of_any_size_stay_below_the_work_item_limit(launches_of, M, N, K, fused):
    """8-bit first layers of 2^34 outputs and more, few words in K among them: every row once, in launches the runtime takes."""
    kw = (K + 31) // 32
    call = (("bnn_bitplane_gemm_bn_sign_pack", (A, 8 * kw, B, kw, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)) if fused else
            ("bnn_bitplane_gemm", (A, 8 * kw, B, kw, C, N, M, N, K, 0)))
    (st, log), = launches_of(call)
    assert st == 0 and log
    tile_n, tile_m = {256: (256, 64), 512: (512, 128)}[log[0][1]]
    assert covers(log, A, 8 * kw, M, -(-N // tile_n), tile_m)


@pytest.mark.parametrize("M,N,K", [(2 ** 25, 4096, 64), (2 ** 31 - 1025, 33, 32), (2 ** 31 - 1025, 64, 96), (2 ** 20, 2 ** 17, 96)])
def test_fused_products_of_few_words_stay_below_the_work_item_limit(launches_of, M, N, K):
    """Fused layers with K <= 96 of up to 2^38 outputs: one launch that the runtime takes."""
    kw = (K + 31) // 32
    (st, log), = launches_of(("bnn_xnor_gemm_bn_sign_pack", (A, kw, B, kw, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)))
    assert st == 0 and len(log) == 1


@pytest.mark.parametrize("M,N,K", [(2 ** 31 - 1025, 17, 32), (2 ** 31 - 1025, 33, 96)])
def test_int32_products_of_few_words_stay_below_the_work_item_limit(launches_of, M, N, K):
    kw = (K + 31) // 32
    (st, log), = launches_of(("bnn_xnor_gemm", (A, kw, B, kw, C, N, M, N, K, 0)))
    assert st == 0 and len(log) == 1


@pytest.mark.parametrize("B,H,W,k,pad", [(2 ** 30, 1, 1, 3, 1), (2 ** 29, 2, 1, 5, 2), (2 ** 28, 2, 2, 7, 3), (2 ** 29 - 300, 1, 2, 5, 2)])
def test_layers_of_whole_channel_words_take_any_number_of_images(launches_of, B, H, W, k, pad):
    """Small images in batches whose padded rows are more than 2^31 together."""
    assert B * (H + 2 * pad) >= 2 ** 31 - 2 ** 8
    (st, log), (st_pool, log_pool) = launches_of(
        ("bnn_conv_bn_sign_pack", (A, B, H, W, 32, WB, 256, 32, k, k, 1, pad, THR, FLIP, OUT, 1, 0)),
        ("bnn_conv_pool_bn_sign_pack", (A, B, H, W, 32, WB, 256, 32, k, k, 1, pad, 2, THR, FLIP, OUT, 1, 0)))
    assert st == 0 and len(log) == 1
    assert (st_pool, len(log_pool)) == ((0, 1) if H % 2 == 0 and W % 2 == 0 else (3, 0))


@pytest.mark.parametrize("fused", [False, True])
def test_convolutions_whose_patch_tiles_do_not_fit_one_launch_are_gathered(launches_of, fused):
    """171000 images of 28 x 28 x 1024, 2176 filters: 17.8 million tiles of 128 pixels, half as many of 256."""
    B, Cin, Cout, words = 171000, 1024, 2176, 9 * 32
    call = (("bnn_conv_bn_sign_pack", (A, B, 28, 28, Cin, WB, words, Cout, 3, 3, 1, 1, THR, FLIP, OUT, Cout // 32, 0)) if fused else
            ("bnn_conv_xnor", (A, B, 28, 28, Cin, WB, words, Cout, 3, 3, 1, 1, C, Cout, 0)))
    (st, log), = launches_of(call)
    assert st == 0 and len(log) == 1


@pytest.mark.parametrize("M,N,K,fused,id_", [
    (12783, 992, 480, True, 7), (12783, 992, 481, True, 6), (12783, 992, 512, True, 6), (12783, 992, 513, True, 7),
    (30000, 4000, 512, True, 6), (10000, 4096, 1024, True, 7), (30000, 4000, 1152, True, 7),
    (98304, 130, 480, False, 7), (98304, 130, 512, False, 6), (98304, 130, 992, False, 7), (98304, 130, 1000, False, 6),
    (40000, 1024, 1152, False, 6), (12783, 992, 1024, False, 7), (12783, 992, 512, False, 7), (200000, 128, 1100, False, 7),
    (2 ** 26, 4096, 512, True, 7), (2 ** 26 - 128, 4096, 512, True, 6)])
def test_short_rows_at_any_alignment_take_the_tiles_that_fit_them(launches_of, M, N, K, fused, id_):
    """Rows that do not start at 16 bytes: K of one 512-bit step, and long int32 rows over whole rounds of tiles, take a
    workgroup per 128 x 128 tile (kernel 6, while one launch holds them); the rest, and aligned rows, the short-K kernel."""
    def call(kernel, ld):
        if fused:
            return ("bnn_xnor_gemm_bn_sign_pack_kernel", (A, ld, B, ld, M, N, K, THR, FLIP, OUT, (N + 31) // 32, kernel, 0))
        return ("bnn_xnor_gemm_kernel", (A, ld, B, ld, C, N, M, N, K, kernel, 0))
    kw = (K + 31) // 32
    odd, aligned = kw | 1, kw + 3 & ~3
    (st, log), (st7, log7), (st_aligned, log_aligned) = launches_of(call(0, odd), call(7, aligned), call(0, aligned))
    assert st == st7 == st_aligned == 0 and log_aligned == log7 != [[-(-M // 128) * -(-N // 128), 256, A]]
    assert log == (log7 if id_ == 7 else [[-(-M // 128) * -(-N // 128), 256, A]])


def first_layer(M=100, N=4096, K=784, ldx=None, ldb=None, ld_a=None, ld_out=None, x=A, b=B, thr=THR, flip=FLIP, bits=C, out=OUT):
    kw, nw = (K + 31) // 32, (N + 31) // 32
    return ("bnn_sign_gemm_bn_sign_pack", (x, ldx or K, b, ldb or kw, M, N, K, thr, flip, bits, ld_a or kw, out, ld_out or nw, 0))


@pytest.mark.parametrize("written,read", [("out", "x"), ("bits", "b"), ("bits", "thr"), ("bits", "flip")])
def test_first_layer_whose_operands_overlap_takes_two_launches(launches_of, written, read):
    """What the two calls read before they write is read before it is written: a matrix that reaches into another by four bytes, and the
    same right beside it."""
    size = {"x": 100 * 784, "b": 4096 * 25, "thr": 4096, "flip": 128, "bits": 100 * 25, "out": 100 * 128}
    at = {"x": A, "b": B, "thr": THR, "flip": FLIP}[read]
    runs = launches_of(*(first_layer(**{written: at + d}) for d in (0, 4 * size[read] - 4, 4 - 4 * size[written], 4 * size[read],
                                                                     -4 * size[written])))
    assert [st for st, _ in runs] == [0] * 5 and [len(log) for _, log in runs] == [2, 2, 2, 1, 1]


def test_first_layer_rows_apart_overlap_as_they_lie(launches_of):
    """Rows 1000 reals, 200 words of bits and 300 of results apart."""
    def run(**at):
        (st, log), = launches_of(first_layer(ldx=1000, ld_a=200, ld_out=300, **at))
        return st, len(log)

    assert run(out=A + 4 * (99 * 1000 + 784)) == run(out=A - 4 * (99 * 300 + 128)) == (0, 1)
    assert run(out=A + 4 * (99 * 1000 + 783)) == run(out=A - 4 * (99 * 300 + 127)) == (0, 2)
    assert run(bits=THR - 4 * (99 * 200 + 25)) == (0, 1) and run(bits=THR - 4 * (99 * 200 + 24)) == (0, 2)


@pytest.mark.parametrize("M,N,K,one", [
    (16, 128, 32, False), (16, 128, 33, True),                      # rows of one word keep to the product of few words
    (100, 4096, 832, True), (100, 4096, 833, True), (100, 4096, 1024, True), (100, 4096, 1025, False),
    (256, 4096, 784, True), (257, 4096, 784, False),                # 512 tiles of 16 x 128
    (1, 65536, 784, True), (1, 65537, 784, False), (8192, 128, 784, True), (8193, 128, 784, False)])
def test_first_layers_of_few_tiles_take_one_launch(launches_of, M, N, K, one):
    kw = (K + 31) // 32
    (st, log), pack, product = launches_of(
        first_layer(M, N, K), ("bnn_pack_sign", (A, M, K, K, C, kw, 0)),
        ("bnn_xnor_gemm_bn_sign_pack", (C, kw, B, kw, M, N, K, THR, FLIP, OUT, (N + 31) // 32, 0)))
    assert st == pack[0] == product[0] == 0
    assert log == ([[-(-M // 16) * -(-N // 128), 512, A]] if one else pack[1] + product[1])


def test_first_layer_rows_of_filters_far_apart_take_two_launches(launches_of):
    for ldb, n in ((2 ** 24 - 1, 1), (2 ** 24, 2)):
        (st, log), = launches_of(first_layer(ldb=ldb))
        assert (st, len(log)) == (0, n)


@pytest.mark.parametrize("change", [
    {"M": 0}, {"N": 0}, {"M": -1}, {"N": -1}, {"K": -5}, {"ldx": 783}, {"ldb": 24}, {"ld_a": 24}, {"ld_out": 127}, {"x": 0}, {"b": 0},
    {"thr": 0}, {"flip": 0}, {"bits": 0}, {"out": 0}, {"x": A + 2}, {"b": B + 2}, {"thr": THR + 1}, {"flip": FLIP + 2}, {"bits": C + 2},
    {"out": OUT + 2}, {"M": 2 ** 31}, {"N": 2 ** 31}, {"K": 2 ** 31 - 31}])
def test_first_layer_answers_as_the_two_calls(launches_of, change):
    """The first status that is not good, and what was launched before it."""
    name, args = first_layer(**change)
    x, ldx, b, ldb, M, N, K, thr, flip, bits, ld_a, out, ld_out, stream = args
    one, pack, product = launches_of((name, args), ("bnn_pack_sign", (x, M, K, ldx, bits, ld_a, stream)),
                                     ("bnn_xnor_gemm_bn_sign_pack", (bits, ld_a, b, ldb, M, N, K, thr, flip, out, ld_out, stream)))
    assert one == (pack if pack[0] else [product[0], pack[1] + product[1]])

"""The launcher of the products on the host: which kernel a product takes, and what is refused (no GPU: every call here is
answered, refused or fails before a launch)."""
import ctypes as C
import os
import subprocess
import sys

import pytest

import paper_2503_06433_amd as ss

F32, BF16 = 0, 1
EPI_STORE, EPI_RESIDUAL, EPI_SWIGLU, EPI_STORE_F32, EPI_SWIGLU_HALVES = 0, 1, 2, 3, 4
INVALID_VALUE = 1
GENERIC, DIRECT, STREAM, TILE, STAGED = range(5)
WS = 128 << 20                                                # the layer calls' workspace


def _library():
    if not os.path.exists(ss.library_path()):
        from paper_2503_06433_amd.build import build
        build()
    return ss.library_path()


def plan(rows, n, k, epi=EPI_STORE, dt=BF16, ws=WS, cus=256):
    """(kernel, place of the tile in the list, ranges of K)"""
    f = C.CDLL(_library()).ssk_gemm_plan
    f.argtypes = [C.c_int] * 5 + [C.c_longlong, C.c_int, C.POINTER(C.c_int), C.POINTER(C.c_int)]
    pick, split = C.c_int(), C.c_int()
    return f(dt, rows, n, k, epi, ws, cus, pick, split), pick.value, split.value


def _symbol(prefix):
    out = subprocess.run(["nm", "-D", "--defined-only", _library()], capture_output=True, text=True, check=True).stdout
    return next(l.split()[2] for l in out.splitlines() if l.split()[2].startswith(prefix))


CALL = """
import ctypes as C, sys
f = getattr(C.CDLL(sys.argv[1]), sys.argv[2])
I, V = C.c_int, C.c_void_p
f.argtypes = [I, V, I, V, V, I, V, I, I, I, I, C.c_bool, V, V, C.c_size_t, I, V, C.c_float]
p = 4096                                                    # never followed: there is no device in this process
print(f(1, p, 1024, p, p, 1024, None, int(sys.argv[3]), 1024, 1024, int(sys.argv[4]), False, None, None, 0, 0, p if sys.argv[5] == "1" else None, -1.0))
"""


@pytest.mark.parametrize("rows", [65, 128, 333, 2000])
def test_fp32_output_refuses_a_row_factor(rows):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")

    def call(epi, factor):
        r = subprocess.run([sys.executable, "-c", CALL, _library(), _symbol("_ZN3ssk7gemm_nt"), str(rows), str(epi), factor],
                           capture_output=True, text=True, env=env, timeout=60)
        assert r.returncode == 0, r.stderr[-500:]
        return int(r.stdout.split()[-1])

    assert call(EPI_STORE_F32, "1") == INVALID_VALUE
    for epi, factor in ((EPI_STORE_F32, "0"), (EPI_STORE, "1")):      # taken: these get as far as the missing device
        assert call(epi, factor) not in (0, INVALID_VALUE)


# Both sides of the lines between the kernels, at products whose times on either side are in the comments of the rules.
@pytest.mark.parametrize("rows,n,k,epi,kernel,split", [
    # outputs of more three-tile blocks than compute units: few rows only up to 16
    (16, 13824, 5120, EPI_SWIGLU, DIRECT, 1), (17, 13824, 5120, EPI_SWIGLU, TILE, 1), (64, 27648, 5120, EPI_SWIGLU, TILE, 1),
    (64, 15360, 5120, EPI_STORE, TILE, 1), (64, 12288, 4096, EPI_STORE, DIRECT, 1), (64, 32000, 4096, EPI_STORE_F32, TILE, 1),
    # a vocabulary of more 128-wide tiles than compute units
    (64, 50256, 768, EPI_STORE_F32, STAGED, 1), (128, 50256, 1600, EPI_STORE_F32, STAGED, 1), (129, 50256, 768, EPI_STORE_F32, TILE, 1),
    (64, 50256, 4096, EPI_STORE_F32, TILE, 1), (128, 32000, 768, EPI_STORE_F32, TILE, 1),
    # an odd vocabulary
    (64, 20001, 4096, EPI_STORE_F32, DIRECT, 1), (48, 32001, 4096, EPI_STORE_F32, DIRECT, 1), (49, 32001, 4096, EPI_STORE_F32, STAGED, 2),
    (32, 32001, 1024, EPI_STORE_F32, DIRECT, 1), (33, 32001, 1024, EPI_STORE_F32, STAGED, 2), (17, 50257, 768, EPI_STORE_F32, STAGED, 1),
    (64, 13824, 200, EPI_SWIGLU_HALVES, DIRECT, 1),
    # long contractions of few rows
    (32, 5120, 13824, EPI_RESIDUAL, DIRECT, 1), (33, 5120, 13824, EPI_RESIDUAL, STAGED, 8), (64, 5120, 13824, EPI_RESIDUAL, STAGED, 8),
    (48, 8192, 28672, EPI_RESIDUAL, DIRECT, 1), (49, 8192, 28672, EPI_RESIDUAL, STAGED, 4), (64, 4096, 11008, EPI_RESIDUAL, DIRECT, 1),
    # ... and of up to 128
    (96, 5120, 13824, EPI_RESIDUAL, STAGED, 8), (128, 8192, 28672, EPI_RESIDUAL, STAGED, 4), (129, 8192, 28672, EPI_RESIDUAL, TILE, 1),
    (80, 4096, 11008, EPI_RESIDUAL, TILE, 1), (128, 8192, 28672, EPI_STORE_F32, TILE, 1),
    # the persistent kernel with K in ranges
    (777, 4096, 8192, EPI_STORE, STREAM, 4), (777, 4096, 8192, EPI_SWIGLU, STREAM, 4), (777, 4096, 8192, EPI_RESIDUAL, STREAM, 4),
    (270, 4096, 8192, EPI_STORE, STREAM, 8), (270, 4096, 8192, EPI_SWIGLU, STREAM, 8), (1000, 4096, 8192, EPI_STORE, TILE, 1),
    (512, 5120, 13824, EPI_RESIDUAL, STREAM, 4), (640, 4096, 11008, EPI_RESIDUAL, STREAM, 4), (384, 8192, 14336, EPI_RESIDUAL, STREAM, 4),
    (1024, 8192, 28672, EPI_RESIDUAL, STREAM, 2), (512, 6912, 5120, EPI_SWIGLU, TILE, 1),
])
def test_products_take_the_kernel_that_was_faster(rows, n, k, epi, kernel, split):
    got = plan(rows, n, k, epi)
    assert (got[0], got[2]) == (kernel, split)


@pytest.mark.parametrize("rows,n,k,epi,split", [
    (81, 1280, 8192, EPI_SWIGLU, 8), (141, 1096, 12288, EPI_RESIDUAL, 8), (333, 2088, 8192, EPI_STORE, 4), (120, 2112, 5120, EPI_SWIGLU, 8),
    (333, 4096, 11008, EPI_RESIDUAL, 4), (1000, 1280, 8192, EPI_STORE, 4), (864, 1280, 8192, EPI_STORE, 4), (170, 8192, 8192, EPI_RESIDUAL, 4),
    # unsplit: shorter contractions, fewer rows, heads
    (129, 5120, 5120, EPI_RESIDUAL, 1), (200, 3072, 4096, EPI_STORE, 1), (111, 5120, 5120, EPI_RESIDUAL, 1), (111, 8192, 8192, EPI_RESIDUAL, 1),
    (81, 1280, 8192, EPI_STORE_F32, 1),
])
def test_tiles_over_ranges_of_long_contractions(rows, n, k, epi, split):
    kernel, _, got = plan(rows, n, k, epi)
    assert (kernel, got) == (TILE, split)
    assert plan(rows, n, k, epi, ws=0)[2] == 1                    # nowhere to put the sums


@pytest.mark.parametrize("rows,n,k,epi,kernel,split", [
    (261, 2112, 12288, EPI_SWIGLU, TILE, 4), (97, 1096, 12800, EPI_RESIDUAL, STAGED, 8), (97, 1096, 12800, EPI_STORE, STAGED, 8),
    (601, 4160, 11008, EPI_RESIDUAL, STREAM, 4), (601, 4160, 11008, EPI_STORE, STREAM, 4), (700, 4112, 8192, EPI_RESIDUAL, STREAM, 4),
    (700, 4112, 8192, EPI_STORE, STREAM, 4),
])
def test_each_kernel_that_is_cut_has_a_product_whose_sums_are_tested(rows, n, k, epi, kernel, split):
    assert plan(rows, n, k, epi)[::2] == (kernel, split)


def stream_columns(rows, n, k, cus=256):
    f = C.CDLL(_library()).ssk_gemm_stream_columns
    f.argtypes = [C.c_int] * 4 + [C.POINTER(C.c_int)]
    return f(rows, n, k, cus, C.byref(C.c_int()))


@pytest.mark.parametrize("rows,n,k,columns", [
    (520, 22016, 4096, 21760), (864, 22016, 4096, 16384), (1400, 12288, 4096, 10752), (1800, 12288, 4096, 8192),
    (5000, 4096, 11008, 3072), (1400, 27648, 5120, 21760), (6400, 22016, 4096, 20736),
    # whole: a last round of more than a half or so, no last round, less than one round
    (1200, 22016, 4096, 22016), (5000, 15360, 5120, 15360), (4096, 12288, 4096, 12288), (864, 12288, 4096, 12288),
    # a contraction so short that a launch costs more than the round
    (520, 22016, 256, 22016),
])
def test_columns_of_the_whole_rounds(rows, n, k, columns):
    assert stream_columns(rows, n, k) == columns


@pytest.mark.parametrize("rows,cus", [(r, c) for r in (257, 640, 1111, 4123, 9000, 70000) for c in (8, 64, 256, 304)])
def test_a_cut_product_keeps_whole_tiles_and_whole_rounds(rows, cus):
    for n in (256, 1280, 4224, 12288, 22016, 57344):
        for k in (128, 4096, 28672):
            c, tiles_m = stream_columns(rows, n, k, cus), -(-rows // 256)
            assert c == n or (0 < c < n and c % 256 == 0 and tiles_m * c // 256 <= tiles_m * -(-n // 256) // cus * cus)


@pytest.mark.parametrize("dt,rows,hidden,vocab,inside", [
    (BF16, 8, 4096, 2048, True), (BF16, 8, 4096, 8192, True), (BF16, 8, 4096, 32000, False), (BF16, 1, 5120, 32000, False), (BF16, 8, 1024, 64000, True),
    (BF16, 9, 4096, 128256, True), (BF16, 16, 8192, 16000, True), (BF16, 16, 8192, 32000, False), (BF16, 32, 4096, 8192, True),
    (BF16, 32, 4096, 32000, False), (BF16, 48, 2048, 4096, True), (BF16, 48, 4096, 2048, False), (BF16, 64, 1024, 2048, True),
    (BF16, 64, 4096, 2048, False), (BF16, 65, 256, 512, False),
    (F32, 4, 256, 512, True), (F32, 16, 4096, 32000, True), (F32, 32, 1024, 16000, True), (F32, 17, 1024, 32000, False), (F32, 64, 256, 512, True),
    (F32, 64, 1024, 16000, False), (F32, 65, 256, 512, False),
])
def test_the_head_takes_its_norm_inside_where_that_saves_time(dt, rows, hidden, vocab, inside):
    f = C.CDLL(_library()).ssk_head_norms_itself
    f.restype = C.c_bool
    assert f(dt, rows, vocab, hidden) == inside


@pytest.mark.parametrize("dt,heads,kv_heads,d,seqs,pages,rotates", [
    # the plain kernel: few blocks of 64-wide heads only
    (F32, 4, 1, 64, 128, 400, True), (F32, 16, 16, 64, 32, 32, True), (F32, 16, 16, 64, 33, 3300, False), (F32, 16, 1, 64, 1024, 2048, False),
    (BF16, 16, 4, 64, 64, 64, True), (BF16, 16, 4, 64, 65, 6500, False), (F32, 8, 8, 128, 1, 1, False), (BF16, 32, 1, 128, 1, 9, False),
    (BF16, 32, 1, 128, 256, 5000, False),
    # the matrix-core kernel: all but many short sequences of ungrouped heads
    (BF16, 32, 32, 128, 1, 1, True), (BF16, 40, 40, 128, 255, 255, True), (BF16, 15, 15, 128, 256, 256, True), (BF16, 16, 16, 128, 256, 896, False), (BF16, 16, 16, 128, 256, 897, True),
    (BF16, 32, 32, 128, 512, 1792, False), (BF16, 32, 32, 128, 513, 514, True), (BF16, 32, 32, 128, 1024, 1024, False),
    (BF16, 64, 8, 128, 1024, 1024, True),
])
def test_where_decode_attention_rotates_by_itself(dt, heads, kv_heads, d, seqs, pages, rotates):
    f = C.CDLL(_library()).ssk_decode_rotates
    f.argtypes, f.restype = [C.c_int] * 5 + [C.c_longlong], C.c_bool
    assert f(dt, heads, kv_heads, d, seqs, pages) == rotates


@pytest.mark.parametrize("n,k", [(5120, 5120), (5120, 8192), (5120, 6912), (6912, 5120)])
def test_one_row_of_tiles_takes_64_x_64(n, k):
    assert plan(96, n, k, EPI_RESIDUAL)[:2] == plan(97, n, k, EPI_RESIDUAL)[:2] == (TILE, 1)


def test_fewer_compute_units_mean_fewer_tiles_for_the_persistent_kernel():
    assert plan(1024, 4096, 4096, cus=256)[0] == TILE and plan(1024, 4096, 4096, cus=64)[0] == STREAM


def test_the_parity_tests_reach_every_tile():
    """The cases of test_gpu_mid_rows.py take the tiles they are listed for: eighteen, with every epilogue of a layer."""
    import test_gpu_mid_rows as m
    assert sorted(m.GATE_UP_TILES) == sorted(m.DOWN_TILES) == list(range(18))
    for tile in range(18):
        T, hidden, ffn = m.GATE_UP_TILES[tile]
        assert plan(T, 2 * ffn, hidden, EPI_SWIGLU, ws=WS if T <= 2048 else 0) == (TILE, tile, 1)
        T, hidden, ffn = m.DOWN_TILES[tile]
        for epi in (EPI_RESIDUAL, EPI_STORE):
            assert plan(T, hidden, ffn, epi, ws=WS if T <= 2048 else 0) == (TILE, tile, 1)

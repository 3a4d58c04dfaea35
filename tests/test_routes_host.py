"""Host-side tests of csrc/routes.h: which calls a launcher keeps away from a kernel that cannot take them.  The header holds
plain host functions; a small shim of them is compiled with the system's C++ compiler, no GPU and no large tensor involved."""
import ctypes
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "routes.h"
extern "C" int folds(int n_seg1, int before, uintptr_t h0, uintptr_t h_final, int64_t bytes)
{ return mamba::ssd_folds(n_seg1, before, (const void *)h0, (const void *)h_final, bytes); }
extern "C" int few_fits(int64_t N, int64_t K) { return mamba::linear_few_fits(N, K); }
extern "C" int conv_step_fits(int64_t D, int64_t N) { return mamba::conv_step_fits(D, N); }
extern "C" int xproj_fits(int64_t D, int64_t N, int64_t dt_rank) { return mamba::step_xproj_fits(D, N, dt_rank); }
extern "C" int row_tiles(int64_t M, int64_t N) { return mamba::linear_few_row_tiles(M, N); }
extern "C" int tiles(int64_t M, int64_t N, int64_t K, int wide) { return mamba::linear_tiles(M, N, K, wide); }
extern "C" int ring(int64_t M, int64_t N, int64_t K, int vec) { return mamba::linear_ring(M, N, K, vec != 0); }
extern "C" int conv_tiles(int64_t M, int64_t D, int64_t K, int64_t taps) { return mamba::linear_conv_tiles(M, D, K, taps); }
extern "C" int wide256(int64_t M, int64_t N, int64_t K, int wide) { return mamba::linear_wide256(M, N, K, wide != 0); }
extern "C" int wide256x192(int64_t M, int64_t N, int64_t K, int vec) { return mamba::linear_wide256x192(M, N, K, vec != 0); }
extern "C" int64_t row_blocks(int64_t M, int64_t BM, int conv) { return mamba::row_blocks(M, BM, conv != 0); }
extern "C" int wide192(int64_t M, int64_t N, int64_t K, int wide) { return mamba::linear_wide192(M, N, K, wide, mamba::linear_tiles(M, N, K, wide)); }
extern "C" int route(int64_t M, int64_t n0, int64_t n1, int64_t n2, int64_t K)
{ const int64_t width[3] = {n0, n1, n2}; return mamba::linear_route(M, width, K); }
extern "C" int lanes_call(int64_t batch, int64_t L, int64_t D, int64_t N) { return mamba::scan_lanes_applies(batch, L, D, N); }
extern "C" int lanes_block(int64_t batch, int64_t L, int64_t D, int64_t N, int64_t dt_rank, int64_t chunks)
{ return mamba::scan_lanes_in_block(batch, L, D, N, dt_rank, chunks); }
extern "C" int lanes_low_dt(int64_t batch, int64_t L, int64_t D, int64_t dt_rank) { return mamba::scan_lanes_takes_low_dt(batch, L, D, dt_rank); }
extern "C" int lanes_channels(int64_t batch, int64_t L, int64_t D) { return mamba::lanes_channels(batch, L, D); }
extern "C" int lanes_tokens(int64_t batch, int64_t L, int64_t D, int bf16) { return mamba::lanes_tau(batch, L, D, bf16 != 0); }
extern "C" int xdt(int64_t M, int64_t d_inner, int64_t dt_rank, int64_t N, unsigned *groups)
{ return mamba::xdt_plan(M, d_inner, dt_rank, N, groups); }
"""

with open(os.path.join(ROOT, "paper_2506_01206_amd", "csrc", "routes.h")) as f:
    KERNELS = re.findall(r"\bk\w+", re.sub(r"//.*", "", re.search(r"enum LinearKernel \{(.*?)\};", f.read(), re.S).group(1)))


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(d / "shim.so"),
                           "-I" + os.path.join(ROOT, "paper_2506_01206_amd", "csrc"), str(d / "shim.cpp")])
    lib = ctypes.CDLL(str(d / "shim.so"))
    i32, i64, ptr = ctypes.c_int, ctypes.c_int64, ctypes.c_size_t
    lib.folds.argtypes = [i32, i32, ptr, ptr, i64]
    lib.few_fits.argtypes = [i64, i64]
    lib.conv_step_fits.argtypes = [i64, i64]
    lib.xproj_fits.argtypes = [i64, i64, i64]
    lib.row_tiles.argtypes = [i64, i64]
    lib.tiles.argtypes = [i64, i64, i64, i32]
    lib.wide192.argtypes = [i64, i64, i64, i32]
    lib.ring.argtypes = [i64, i64, i64, i32]
    lib.wide256.argtypes = [i64, i64, i64, i32]
    lib.wide256x192.argtypes = [i64, i64, i64, i32]
    lib.conv_tiles.argtypes = [i64] * 4
    lib.row_blocks.argtypes, lib.row_blocks.restype = [i64, i64, i32], i64
    lib.lanes_call.argtypes = [i64] * 4
    lib.lanes_block.argtypes = [i64] * 6
    lib.lanes_low_dt.argtypes = [i64] * 4
    lib.lanes_channels.argtypes = [i64] * 3
    lib.lanes_tokens.argtypes = [i64] * 3 + [i32]
    lib.route.argtypes = [i64] * 5
    lib.xdt.argtypes = [i64, i64, i64, i64, ctypes.POINTER(ctypes.c_uint)]
    return lib


def test_scalar_decay_segments_are_not_stitched_over_their_own_initial_state(routes):
    """Workgroups of the second pass read h0 while others write h_final: no fold where the two share a byte."""
    row = 24 * 64 * 128 * 4
    base, n = 1 << 40, 3 * row
    assert routes.folds(2, 1, base, base + n, n) and routes.folds(2, 1, base + n, base, n)     # side by side
    assert routes.folds(11, 10, base, 0, n) and routes.folds(11, 10, 0, base, n) and routes.folds(11, 10, 0, 0, n)
    assert not routes.folds(2, 1, base, base, n)                                              # in place
    for shift in (16, 64 * 128 * 4, row, 2 * row, n - 16):
        assert not routes.folds(2, 1, base, base + shift, n) and not routes.folds(2, 1, base + shift, base, n)
    assert not routes.folds(1, 0, base, 0, n) and not routes.folds(12, 11, base, 0, n)         # one segment; too many


def test_few_row_product_leaves_what_32_bits_do_not_count_to_others(routes):
    """It rounds k up to steps of 64 and launches 512 threads per 16 columns, both counted in 32 bits."""
    assert routes.few_fits(1, 8) and routes.few_fits(8191, 1 << 30) and routes.few_fits(1, (1 << 31) - 64)
    for K in ((1 << 31) - 56, (1 << 31) - 8, 1 << 31, (1 << 31) + 8, 1 << 32, 1 << 40):
        assert not routes.few_fits(1, K), K
    assert routes.few_fits(1 << 26, 768) and (((1 << 27) - 16) // 16) * 512 < 1 << 32
    assert routes.few_fits((1 << 27) - 16, 768) and not routes.few_fits(1 << 27, 768) and not routes.few_fits(1 << 31, 8)


@pytest.mark.parametrize("N", [4, 8, 16, 32])
def test_fused_layer_step_leaves_what_32_bits_do_not_count_to_others(routes, N):
    """Channels in 32 bits and a grid of fewer than 2^32 threads along x, one wavefront per 64 / (N / 4) channels times the
    pieces of a branch with many of them."""
    channels = 64 // (N // 4) * min(N // 4, 4)
    for D in (1, 1536, 1 << 30, (1 << 31) - 32, (1 << 31) - 24, 1 << 31, (1 << 32) - 64, (1 << 32) - 56, 1 << 32, 6 << 30):
        threads = -(-D // channels) * 64
        assert bool(routes.conv_step_fits(D, N)) == (D < 1 << 32 and threads < 1 << 32), D


@pytest.mark.parametrize("N", [4, 8, 16, 32])
@pytest.mark.parametrize("dt_rank", [8, 32, 48, 64, 128])
def test_draft_position_state_step_leaves_what_32_bit_offsets_do_not_reach_to_others(routes, N, dt_rank):
    """The kernel that adds up the x projection's partial sums counts a lane's bytes in 32 bits: every last place that it forms
    has to fit, and every block of which they all fit is still taken, up to the widest that the product ahead of it takes."""
    D_most = (1 << 26) - 16
    assert routes.few_fits(2 * D_most, 768)
    for D in (16, 1536, 5120, 1 << 24, (1 << 25) - 16, 1 << 25, (1 << 25) + 16, 44739232, 44739248, D_most):
        last = [16 * (D * N // 4 - 1), 2 * dt_rank * D - 8, 16 * (D // 16 * ((dt_rank + 2 * N) // 4) - 1), 4 * (D - 1)]
        assert bool(routes.xproj_fits(D, N, dt_rank)) == all(v < 1 << 32 for v in last), D
    assert bool(routes.xproj_fits((1 << 25) + 16, N, dt_rank)) == (N <= 16 and dt_rank <= 48)
    assert routes.xproj_fits(1 << 24, 32, 128) and not routes.xproj_fits((1 << 24) + 16, 32, 136)


def test_wide_blocks_of_few_rows_keep_the_two_projections_apart(routes):
    """x_proj and dt_proj in one kernel: from 768 rows up to 1536 channels, from 2700 beyond; only the sizes it is built for."""
    g = ctypes.c_uint()
    rows = lambda M, d_inner=1536, dt_rank=48, N=16: routes.xdt(M, d_inner, dt_rank, N, g)
    for d_inner, dt_rank in ((64, 32), (512, 32), (1024, 32), (1536, 48), (1536, 64)):
        assert rows(767, d_inner, dt_rank) == 0 and rows(768, d_inner, dt_rank) == 16 and g.value == 3
    for d_inner, dt_rank in ((1600, 48), (2048, 64), (3072, 48), (4096, 64), (5120, 64), (1 << 20, 64)):
        for M in (768, 1100, 2000, 2699):
            assert rows(M, d_inner, dt_rank) == 0, (M, d_inner)
        assert rows(2700, d_inner, dt_rank) == 16 and g.value == 1
    assert rows(1361) == 16 and g.value == 2 and rows(4096) == 16 and rows(4097) == 32 and rows(8193) == 64
    assert rows(8192, 64, 32) == 32 and rows(8193, dt_rank=64) != 64
    for kw in (dict(N=8), dict(N=32), dict(dt_rank=40), dict(dt_rank=96), dict(d_inner=1568), dict(d_inner=32), dict(d_inner=1 << 21)):
        assert rows(8000, **kw) == 0


def test_few_row_product_forms_no_more_row_tiles_than_there_are_rows(routes):
    """One round of workgroups where that is possible, and never twice the row tiles of 16 that the rows need."""
    assert [routes.row_tiles(M, 3072) for M in (1, 16, 17, 32, 33, 48, 64)] == [1, 1, 2, 2, 4, 4, 4]
    assert [routes.row_tiles(M, 1024) for M in (16, 17, 64)] == [1, 1, 1] and routes.row_tiles(64, 2048) == 2
    for N in (16, 3072, 4096, 4112, 6144, 8184, 10240, 1 << 20):
        for M in range(1, 65):
            tiles = routes.row_tiles(M, N)
            assert tiles in (1, 2, 4) and (tiles == 1 or 16 * tiles < 2 * 16 * -(-M // 16)), (M, N)


def test_tile_kernel_of_a_product(routes):
    """Which tile kernel a product gets where the rules asked before leave it: the ones measured faster in chains of blocks
    of other widths than 1536 channels, and never a kernel whose conditions it does not meet."""
    W256, W128, T128, T64x128, DEEP, T64 = (KERNELS.index(k) for k in ("kWide256", "kWide128", "kTiles128", "kTiles64x128", "kTiles64Deep", "kTiles64"))
    tiles = lambda M, N, K: routes.tiles(M, N, K, M >= 128 and N % 128 == 0 and K % 128 == 0)
    for kind, shapes in {
            W256: [(5003, 3072, 256), (10241, 1536, 128), (8192, 4096, 768), (2047, 8192, 512), (2500, 6144, 384), (1101, 8192, 1024),
                   (32768, 3072, 768), (1000, 10240, 2560), (4096, 10240, 2560), (3000, 4096, 1024), (6000, 2048, 4096)],
            W128: [(129, 32768, 128), (2177, 1152, 1024), (4001, 768, 1536), (3999, 1280, 128), (2048, 3072, 768), (8000, 768, 1536),
                   (32768, 768, 1536), (16000, 256, 512)],
            T128: [(1025, 8192, 512), (1001, 10240, 640), (8000, 3072, 768), (6000, 6144, 1536), (2000, 10240, 2560)],
            DEEP: [(200, 8192, 2048), (512, 4096, 1024), (2000, 1024, 2048), (1000, 2048, 4096)],
            T64: [(512, 6144, 128), (384, 8192, 384), (200, 10240, 2560)]}.items():
        for s in shapes:
            assert tiles(*s) == kind, s
    # not a multiple of 128: by the number of tiles alone
    assert [tiles(M, 4000, 128) for M in (5000, 1500, 300)] == [T128, T64x128, T64] and tiles(300, 1000, 1000) == DEEP
    for M in (128, 129, 255, 256, 257, 1000, 5000, 40000, 8388480):
        for N in (128, 256, 384, 1024, 1152, 8192, 12288):
            for K in (128, 384, 1024, 5120, 1 << 20):
                kind = tiles(M, N, K)
                assert kind in (W256, W128, T128, T64x128, DEEP, T64) and (kind != W256 or (M >= 256 and N % 256 == 0)), (M, N, K)


def test_192_row_tiles(routes):
    """The products that the parity tests name for them, those measured faster and slower, and never without their conditions."""
    takes = lambda M, N, K: bool(routes.wide192(M, N, K, M >= 128 and N % 128 == 0 and K % 128 == 0))
    for s in [(2977, 3072, 128), (8000, 3072, 256), (4993, 2048, 384), (5184, 2048, 512), (11905, 768, 1536), (12095, 768, 128), (3073, 6144, 128),
              (3000, 3072, 768), (8000, 3072, 768), (5000, 2048, 512), (12000, 768, 1536), (6000, 6144, 1536), (12000, 1536, 3072), (7000, 2560, 5120)]:
        assert takes(*s), s
    for s in [(16384, 3072, 768), (32768, 3072, 768), (8000, 4096, 1024), (1500, 3072, 768), (2000, 2560, 5120), (32768, 768, 1536), (191, 1 << 16, 128),
              (8000, 3000, 768), (8000, 3072, 760)]:
        assert not takes(*s), s


def test_one_round_of_tiles(routes):
    """The products that the parity test names for each tile, more than a round left alone, and never without the conditions."""
    none, t64, t64x128, t128 = (KERNELS.index(k) for k in ("kNoKernel", "kRing64", "kRing64x128", "kRing128"))
    # more 64 x 64 tiles than CUs: not with a long k and few rows
    for s in [(109, 10240, 8064), (87, 10240, 3584), (84, 9600, 7296), (166, 6656, 5632), (126, 9728, 5120), (85, 10240, 2816)]:
        assert routes.ring(*s, 1) == t64x128, s
    for s in [(126, 8192, 5120), (86, 8640, 2048), (85, 10240, 1984), (193, 5120, 5120), (593, 2048, 2688)]:
        assert routes.ring(*s, 1) == t64, s
    assert routes.ring(101, 8768, 8000, 1) == none
    for want, cases in ((t64, [(641, 1280, 256), (449, 2560, 1024), (704, 1856, 320), (64, 64, 1 << 28)]),
                        (t64x128, [(1025, 1536, 384), (1087, 1536, 448), (512, 3072, 768)]),
                        (t128, [(2049, 1152, 384), (2175, 1152, 1536), (4096, 768, 832)]),
                        (none, [(2048, 3072, 768), (1500, 3072, 768), (2048, 2048, 256), (63, 64, 256), (641, 1288, 256), (1025, 1600, 384),
                                (64, 64, 248), (64, 64, 264), (64, 64, (1 << 28) + 64), (1 << 20, 64, 256)])):
        for s in cases:
            assert routes.ring(*s, 1) == want, s
            assert routes.ring(*s, 0) == none, s


def test_conv_in_the_way_into_a_block(routes):
    """The tile that the parity test names for each product, the product and the conv apart where the rows that tiles share cost more
    than a launch, and never a tile that the shape does not divide into.  Every row has one block that stores it, and a tile of x the
    three rows before its own."""
    apart, r64, r64x128, r128, w128, w192, w256 = range(7)
    for kind, shapes in {r64: [(64, 1536, 768), (100, 1536, 768), (64, 64, 256), (189, 128, 256), (333, 1536, 768), (600, 512, 256), (64, 1 << 20, 256)],
                         r64x128: [(200, 4096, 2048), (100, 5120, 2560)], r128: [(1000, 1024, 256), (2003, 512, 256), (1000, 1536, 768)],
                         w128: [(1254, 1536, 256), (1264, 1536, 256), (2048, 1536, 768)],
                         w192: [(1281, 1536, 384), (8000, 1536, 768)],
                         w256: [(4031, 2048, 384), (4048, 2048, 384), (4000, 4096, 2048), (10000, 1536, 768), (16384, 3072, 1536), (32768, 1536, 768)],
                         # a long k that the few-row kernels share among wavefronts
                         apart: [(70, 256, 2496), (65, 128, 2112), (133, 128, 2112), (86, 128, 2112), (67, 192, 1600), (116, 512, 2048), (258, 128, 1664),
                                 (182, 64, 2432), (66, 448, 1536), (112, 128, 1536), (63, 1536, 768), (333, 1536, 192), (333, 1536, 800), (333, 1500, 768), (512, 4096, 2048), (2048, 4096, 2048),
                                 (1 << 24, 128, 256), (333, (1 << 20) + 64, 768)]}.items():
        for s in shapes:
            got = routes.conv_tiles(*s, 4)
            assert got == kind or (kind == r64 and s[1] == 1 << 20 and got in (apart, r64)), (s, got)
            assert routes.conv_tiles(*s, 3) == apart, s
    size = {r64: (64, 64), r64x128: (64, 128), r128: (128, 128), w128: (128, 128), w192: (192, 128), w256: (256, 256)}
    for D in (64, 128, 192, 320, 512, 1088, 1536, 4096):
        for K in (256, 320, 768, 2048):
            for M in (64, 65, 127, 128, 191, 192, 255, 256, 500, 1000, 3000, 20000, 1 << 23):
                kind = routes.conv_tiles(M, D, K, 4)
                if kind != apart:
                    bm, bn = size[kind]
                    assert M >= bm and D % bn == 0 and (kind < w128 or K % 128 == 0), (M, D, K)
    for bm in (64, 128, 192, 256):
        for M in (bm, bm + 1, bm + 3, 2 * bm - 4, 2 * bm - 3, 2 * bm - 2, 10 * bm, 10 * bm - 27, 10 * bm - 26):
            stored = 0
            for r in range(routes.row_blocks(M, bm, 1)):
                first = 0 if r == 0 else bm + (r - 1) * (bm - 3)
                m0 = min(first - 3 if r else 0, M - bm)
                assert first == stored and m0 >= 0 and (r == 0 or first - m0 >= 3), (M, bm, r)
                stored = m0 + bm
            assert stored == M and routes.row_blocks(M, bm, 0) == -(-M // bm)


def test_256_x_192_tiles_by_rounds(routes):
    """Products measured faster and slower on 256 x 192 tiles, those that the parity tests name for other tiles, and never without the conditions."""
    for s in [(16384, 1536, 768), (32768, 768, 1536), (16384, 768, 1536), (4096, 3072, 768), (32768, 1152, 2304), (16384, 1536, 3072), (16384, 576, 1152)]:
        assert routes.wide256x192(*s, 1) and not routes.wide256x192(*s, 0), s
    # widths that 128 does not divide: any number of rounds; others: whole ones
    for s in [(1856, 4800, 6016), (2429, 4800, 7552), (3615, 2880, 4352), (4993, 7296, 4096), (1240, 9600, 5888), (21699, 1152, 2048)]:
        assert routes.wide256x192(*s, 1), s
    for s in [(5578, 1536, 6400), (2221, 4224, 6016), (7419, 1152, 6528), (25274, 768, 7040), (2787, 3072, 3456), (1790, 5376, 4224),
              (1730, 5376, 2560), (1166, 6912, 2944), (1277, 7296, 2944), (1016, 8832, 1920), (1765, 6144, 3072),
              (8000, 768, 1536), (6000, 768, 768), (24000, 768, 768), (8000, 3072, 768), (32768, 3072, 768), (32768, 6144, 1536), (10000, 1536, 3072), (6000, 1536, 3072), (16384, 1152, 2304),
              (999, 768, 768), (16384, 1600, 768), (16384, 1536, 832), (16384, 1536, (1 << 28) + 128),
              (8000, 3072, 256), (11905, 768, 1536), (12095, 768, 128), (4097, 3072, 128), (16385, 768, 256), (2977, 3072, 128), (5003, 3072, 384)]:
        assert not routes.wide256x192(*s, 1), s


def test_256_tiles_by_rounds(routes):
    """Products measured faster and slower on 256 x 256 tiles, those that the parity tests name for other tiles, and never without the
    conditions."""
    takes = lambda M, N, K: bool(routes.wide256(M, N, K, M >= 128 and N % 128 == 0 and K % 128 == 0))
    for s in [(16384, 768, 1536), (10000, 3072, 768), (16384, 3072, 768), (32768, 3072, 768), (5000, 3072, 768), (5000, 6144, 1536), (10000, 2560, 5120)]:
        assert takes(*s), s
    for s in [(8000, 768, 1536), (12000, 3072, 768), (8000, 3072, 768), (8000, 512, 1024), (999, 10240, 2560), (16384, 896, 1536), (16384, 768, 1600),
              (2977, 3072, 128), (4993, 2048, 384), (11905, 768, 1536), (12095, 768, 128), (3073, 6144, 128), (1025, 8192, 512), (1001, 10240, 640),
              (2177, 1152, 1024), (4001, 768, 1536), (129, 32768, 128)]:
        assert not takes(*s), s


# The kernel that each product of the GPU parity tests is there for: rows, columns, k.  (Those of test_linear_few_every_split_of_k, every k
# on ten shapes, are left to the rules that its docstring names.)
PARITY = {
    "kFew16x8": [(1, 1, 8), (5, 80, 48), (130, 200, 72), (129, 129, 1032), (12, 80, 1536), (32, 768, 1536), (33, 100, 520), (64, 50, 1544),
                 (3, 1000, 72), (65, 96, 512), (13, 80, 1024), (333, 80, 2056)],
    "kFew16x16": [(1, 4096, 8), (17, 2050, 40), (257, 250, 1544)],
    "kFew16x16Stream": [(12, 8200, 136), (1, 50280, 768), (16, 50280, 768)],
    "kFew32x16": [(1000, 80, 1536), (64, 1536, 48), (18, 3072, 768), (19, 4090, 768), (100, 800, 520), (100, 790, 1032)],
    "kFew32x32": [(384, 768, 1536), (65, 4000, 512), (255, 999, 1288), (2700, 80, 1536), (330, 761, 1096), (641, 700, 1024), (50, 5000, 264),
                  (64, 4500, 776)],
    "kFew64x32": [(129, 2600, 4104)],
    "kRing64": [(257, 3072, 768), (641, 1280, 256), (449, 2560, 1024), (704, 1856, 320)],
    "kRing64x128": [(1025, 1536, 384), (1087, 1536, 448), (512, 3072, 768)],
    "kRing128": [(1024, 3072, 768), (4096, 768, 1536), (384, 8192, 384), (2049, 1152, 384), (2175, 1152, 1536), (4096, 768, 832),
                 (2177, 1152, 1024), (4001, 768, 1536)],
    "kWide256x192": [(3713, 3264, 128), (3840, 3264, 256), (5761, 2112, 384), (1921, 6144, 384), (7000, 1728, 128)],
    "kWide256": [(4097, 3072, 128), (16385, 768, 256), (7936, 2048, 512), (5003, 3072, 384), (2047, 8192, 128), (16384, 2048, 256),
                 (8192, 4096, 512), (5003, 3072, 256), (10241, 1536, 128), (8192, 4096, 768), (2047, 8192, 512), (2500, 6144, 384)],
    "kWide192": [(2977, 3072, 128), (4993, 2048, 384), (5184, 2048, 512), (11905, 768, 1536), (12095, 768, 128), (3073, 6144, 128),
                 (8000, 3072, 256, 1504), (16384, 1152, 384), (16384, 1152, 640), (1101, 8192, 1024), (1001, 10240, 640), (1025, 8192, 512)],
    "kWide128Eight": [(8000, 768, 1536), (5505, 768, 1536), (5888, 768, 1024), (2177, 2304, 1024)],
    "kWide128": [(3968, 1280, 384), (4097, 1280, 384), (4223, 1280, 512), (3969, 1280, 640), (129, 32768, 128), (3999, 1280, 128)],
    "kTiles128": [(8000, 3072, 256, 1500), (8190, 4100, 136), (8192, 4096, 40), (8300, 4000, 32), (4096, 4096, 64), (4100, 4000, 128),
                  (4096, 4104, 192), (4090, 4096, 320), (5000, 3400, 448)],
    "kTiles64x128": [(1472, 4000, 320), (1500, 4000, 128), (1501, 4001, 200)],
    "kTiles64Deep": [(704, 1000, 1000), (641, 1000, 1000), (1030, 1200, 520), (450, 3000, 1288)],
    "kTiles64": [(512, 6144, 128), (2688, 1152, 256)],
    "kTiles64Stream": [(64, 9000, 64)],
}


def test_every_product_of_the_parity_tests_reaches_the_kernel_it_is_there_for(routes):
    """The whole choice, in the order in which its rules are asked: no kernel without a parity test, no product that slips to another one,
    and for the tiles that move their last row block back one that is full, one that is not, outputs split and a residual in place, and
    more slabs than are requested before the first product."""
    import test_gpu_parity as gpu
    widths = lambda N, splits: (list(splits or (N,)) + [0, 0])[:3]
    kernel = lambda M, N, K, splits=None: KERNELS[routes.route(M, *widths(N, splits), K)]
    cases = {}                                                     # shape (and first output, where one shape comes twice) -> its splits
    for name in dir(gpu):
        marks = [k.args for k in getattr(getattr(gpu, name), "pytestmark", ()) if k.name == "parametrize"]
        if name.startswith("test_linear_") and len(marks) == 1 and marks[0][0] == "M,N,K,splits":
            for M, N, K, splits in marks[0][1]:
                listed = [(M, N, K, splits[0])] if splits and any((M, N, K, splits[0]) in l for l in PARITY.values()) else [(M, N, K)]
                cases.setdefault(listed[0], []).append(splits)
    assert sorted(cases) == sorted(shape for shapes in PARITY.values() for shape in shapes)
    assert set(PARITY) | {"kNoKernel"} == set(KERNELS)
    rows = dict(kRing64=64, kRing64x128=64, kRing128=128, kWide256x192=256, kWide256=256, kWide192=192, kWide128Eight=128, kWide128=128)
    for want, shapes in PARITY.items():
        for shape in shapes:
            for splits in cases[shape]:
                assert kernel(*shape[:3], splits) == want, (shape, splits)
        if want in rows:
            assert {shape[0] % rows[want] == 0 for shape in shapes} == {True, False}, want
            assert {splits is None for shape in shapes for splits in cases[shape]} == {True, False}, want
            assert any(K >= 384 and M % rows[want] and None in cases[(M, N, K)] for M, N, K in (s for s in shapes if len(s) == 3)), want
    # the launches that have to agree, and the sampled rows
    assert [kernel(*s) for s in ((8192, 4096, 768), (16384, 1152, 1536), (4096, 768, 1536))] == ["kWide256", "kWide128", "kRing128"]
    assert kernel(32768, 3072, 768, (1536, 1536)) == "kWide256" and kernel(32768, 768, 1536) == "kWide256x192"


def test_short_contexts_of_a_block_keep_the_single_launch_where_the_lanes_scan_takes_several_rounds(routes):
    """Up to 16 tokens the two passes are one launch: blocks measured faster and slower on the lanes kernel than on that one."""
    takes = lambda b, L, D, R=48, chunks=1: bool(routes.lanes_block(b, L, D, 16, R, chunks))
    for s in [(1, 4, 256), (2, 4, 256), (1, 6, 768), (1, 16, 256), (1, 16, 1536), (1, 8, 1536), (2, 15, 1024), (12, 16, 256), (4, 13, 256), (1, 16, 2048),
              (2, 12, 256), (1, 15, 1024, 96)]:
        assert takes(*s), s
    for s in [(1, 4, 1536), (3, 4, 1536), (3, 16, 1536), (6, 8, 768), (12, 8, 256), (12, 4, 256), (1, 8, 4096), (1, 16, 4096), (2, 16, 1536), (3, 9, 768),
              (2, 5, 2048), (3, 5, 1024), (1, 5, 2560), (1, 7, 3072), (14, 9, 256, 64), (6, 16, 768), (1, 16, 2560, 80), (9, 10, 256), (17, 8, 64),
              (1, 6, 2048), (1, 4, 768, 96), (1, 3, 64), (8, 6, 1536), (1, 9, 5120)]:
        assert not takes(*s), s
    # more tokens are three launches: the other line
    for s in [(1, 17, 1536), (1, 40, 1536), (2, 17, 1024), (3, 20, 1536), (1, 24, 2048)]:
        assert takes(*s, 48, 2), s
    assert not takes(3, 25, 2560, 48, 2) and not takes(1, 40, 1537, 48, 3) and not routes.lanes_block(1, 40, 1536, 8, 48, 3)
    assert routes.lanes_low_dt(1, 512, 1536, 64) and not routes.lanes_low_dt(1, 513, 1536, 64) and not routes.lanes_low_dt(1, 40, 1536, 72)


def test_lanes_scan_counts_its_places_in_32_bits(routes):
    """The kernel addresses the rows of a super-step, up to 512, by 32-bit element offsets, of layers as wide as its lines let through."""
    widest = 0
    for D in [2 * i for i in range(3, 5000)] + [1 << k for k in range(14, 31)]:
        for L in (4, 16, 17, 33, 64, 300, 512, 1000, 4000, 5050, 32000000 // D, 1 << 20):
            for chunks in (1, 3):
                if routes.lanes_call(1, L, D, 16) or routes.lanes_block(1, L, D, 16, 48, chunks):
                    widest = max(widest, D)
    assert 4600 <= widest <= 4608 and 512 * widest < 1 << 32
    # tokens to a lane: what a call's super-steps come to
    assert [routes.lanes_tokens(1, L, 1536, 1) for L in (256, 257, 384, 385, 512, 700, 1100)] == [4, 6, 6, 8, 8, 6, 6]
    assert routes.lanes_tokens(1, 1100, 512, 1) == 4 and routes.lanes_tokens(1, 700, 1536, 0) == 6 and routes.lanes_tokens(6, 2251, 488, 0) == 8


def test_blocks_take_the_lanes_scan_where_its_last_round_is_full(routes):
    """Blocks near the line between the lanes scan and the two passes, measured faster and slower."""
    takes = lambda b, L, D: bool(routes.lanes_block(b, L, D, 16, 48, 5))
    for s in [(1, 10500, 1536), (1, 16000, 1536), (1, 20000, 1536), (2, 4000, 1536), (2, 8000, 1536), (3, 3000, 1536), (1, 8000, 1024), (1, 9000, 3072),
              (1, 3000, 2048), (1, 40, 1536), (2, 40, 1536), (3, 1000, 1024), (1, 2041, 256), (1, 4065, 768), (2, 4101, 384), (1, 17, 4096)]:
        assert takes(*s), s
    for s in [(2, 9084, 640), (4, 8311, 320), (1, 6653, 1280), (2, 521, 1792), (3, 10189, 448), (2, 1164, 2048), (1, 1577, 2368), (1, 14920, 1408),
              (2, 8701, 704), (1, 6769, 2816), (2, 14536, 704), (1, 32768, 1536), (4, 8000, 1536), (1, 10000, 768), (8, 500, 1536), (1, 6000, 4096),
              (4, 40, 1536), (2, 1500, 2048), (8, 2000, 1536), (1, 6000, 512)]:
        assert not takes(*s), s


def test_blocks_of_the_parity_tests_reach_the_kernels_they_are_there_for(routes):
    """Every tile that forms the conv, on products whose launch apart sums in the same order and in another; every number of channels and
    tokens of a scan that takes the dt projection along, and blocks on both sides of its lines."""
    import test_gpu_parity as gpu
    cases = lambda f: next(k.args[1] for k in f.pytestmark if k.name == "parametrize")
    tiles = set()
    for B, L, dm, D in cases(gpu.test_block_conv_in_the_way_in):
        tiles.add(routes.conv_tiles(B * L, D, dm, 4))
        few = KERNELS[routes.route(B * L, D, D, 0, dm)].startswith("kFew")
        assert few == gpu.few_outputs(B * L, D), (B, L, dm, D)
    assert tiles == set(range(1, 7))                               # never apart
    low, apart = set(), 0
    for B, L, dm, D, R in cases(gpu.test_block_dt_projection_in_the_scan):
        lanes = routes.lanes_call(B, L, D, 16) or routes.lanes_block(B, L, D, 16, R, 1 if L <= 16 else 2)
        if lanes and routes.lanes_low_dt(B, L, D, R):
            low.add((routes.lanes_channels(B, L, D), routes.lanes_tokens(B, L, D, 1)))
        else:
            apart += 1
    assert low == {(2, 4), (4, 4), (4, 6), (4, 8), (6, 4), (6, 6), (6, 8)} and apart >= 4

"""The rules by which the library chooses among its kernels, compiled for the host: which side of each measured line a call
falls on, over the sizes on both sides of it."""
import ctypes
import os
import subprocess
import types

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_06941_amd", "csrc")


def _compile(tmp_path_factory, name, code):
    d = tmp_path_factory.mktemp(name)
    src, lib = d / (name + ".cpp"), d / (name + ".so")
    src.write_text(code)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-pthread", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    return ctypes.CDLL(str(lib))


@pytest.fixture(scope="module")
def sgd(tmp_path_factory):
    L = _compile(tmp_path_factory, "sgd_rule", '''#include "sgd_rule.h"
extern "C" int pay(uint64_t ratings, uint32_t B, uint64_t chain, int F, uint32_t cus) { return sgd_rounds_pay(ratings, B, chain, F, cus); }
''')
    L.pay.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint64, ctypes.c_int, ctypes.c_uint32]
    return lambda ratings, B, chain, F, cus: bool(L.pay(ratings, B, int(chain * B), F, cus))


# (ratings, blocks, mean over the strata of their largest cell, factors, compute units, ms one after the other, ms in rounds)
MEASURED = [
    (16_253, 1024, 2.5, 64, 256, 2.45, 4.01), (125_091, 1024, 4.5, 16, 256, 2.68, 3.69), (1_043_634, 1024, 6.6, 64, 256, 4.18, 4.77),
    (3_108_417, 1024, 14.5, 64, 256, 6.79, 5.75), (2_079_384, 1024, 10.4, 16, 256, 5.42, 4.56), (3_108_417, 1024, 14.5, 16, 256, 6.77, 4.85),
    (16_084_561, 512, 131.9, 64, 256, 25.3, 8.46), (16_084_561, 512, 131.9, 64, 32, 29.7, 22.0), (16_084_561, 512, 131.9, 64, 16, 34.8, 38.9),
    (16_084_561, 512, 131.9, 64, 8, 56.4, 72.5), (16_084_561, 512, 131.9, 16, 16, 27.6, 12.3), (1_801_150, 1024, 14.2, 64, 32, 7.32, 22.3),
    (1_801_150, 1024, 14.2, 16, 32, 6.42, 12.0), (1_801_150, 256, 61.3, 64, 32, 5.97, 3.28), (1_801_150, 256, 61.3, 64, 8, 7.67, 8.93),
    (1_801_150, 128, 170.8, 64, 8, 8.67, 6.97), (255_238, 64, 90.5, 64, 256, 1.94, 0.594), (255_238, 64, 90.5, 16, 16, 1.91, 0.492),
    (128_491_641, 1024, 272.0, 64, 64, 125.2, 79.7), (128_491_641, 1024, 272.0, 32, 32, 128.7, 67.2), (16_084_561, 512, 131.9, 64, 24, 31.1, 27.9),
    (1_801_150, 1024, 14.2, 32, 32, 6.98, 17.7), (16_084_561, 512, 131.9, 32, 8, 35.5, 32.8), (1_801_150, 256, 61.3, 32, 16, 6.20, 3.68),
    (293, 16, 3.4, 16, 256, 0.047, 0.053), (1139, 16, 10.3, 64, 256, 0.077, 0.064), (39, 2, 10.5, 64, 256, 0.0097, 0.0079),
]


def test_sgd_takes_the_faster_side_of_every_measured_size(sgd):
    for ratings, B, chain, F, cus, in_a_row, rounds in MEASURED:
        assert sgd(ratings, B, chain, F, cus) == (rounds < in_a_row), (ratings, B, F, cus)


def test_sgd_blocks_the_library_makes_are_worked_on_in_rounds(sgd):
    for ratings in (40, 500, 13_920, 132_749, 922_110, 16_084_561, 1 << 27):
        B = 1024
        while B > 1 and ratings // (B * B) < 32:
            B //= 2
        mean = ratings / B / B
        for F in (16, 32, 64):
            for cus in (64, 128, 256):
                if mean <= 256:
                    assert sgd(ratings, B, 1.2 * mean, F, cus), (ratings, F, cus)
    assert not sgd(257, 1, 257, 16, 256)                        # beyond 256 ratings a cell on average
    assert not sgd(0, 4, 0, 16, 256) and not sgd(0, 1, 0, 64, 256)


@pytest.fixture(scope="module")
def cells(tmp_path_factory):
    L = _compile(tmp_path_factory, "sgd_cells", '''#include "sgd_rule.h"
extern "C" int eight(uint32_t n, uint32_t cus) { return sgd_eight_cells_a_unit(n, cus); }
extern "C" int ahead(uint64_t ratings, uint32_t B, uint32_t n, uint32_t cus) { return sgd_reads_ahead(ratings, B, n, cus); }
''')
    L.ahead.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint32]
    return types.SimpleNamespace(eight=lambda n, cus: bool(L.eight(n, cus)), ahead=lambda ratings, B, cus, n=0: bool(L.ahead(ratings, B, n or B, cus)))


# (blocks, ratings a cell, compute units, ms of an iteration with the next stratum's programs read ahead, without)
AHEAD_MEASURED = [
    (256, 31, 32, 1.953, 1.658), (512, 7.7, 64, 3.627, 2.438), (512, 7.7, 32, 5.233, 3.507), (512, 7.7, 128, 2.458, 2.310), (1024, 15.3, 128, 9.347, 7.031),
    (1024, 1.9, 256, 5.839, 4.999), (256, 245, 32, 6.744, 5.834), (512, 61, 24, 27.99, 25.73), (512, 61, 32, 21.79, 20.52), (128, 31, 24, 0.965, 0.897),
    (128, 8.4, 256, 0.495, 0.438), (128, 16.8, 128, 0.529, 0.502), (384, 12.6, 256, 1.738, 1.651), (256, 7.8, 256, 1.106, 1.087), (512, 16.7, 128, 3.924, 3.749),
    (128, 33.5, 32, 0.741, 0.726), (384, 25.1, 96, 3.119, 3.048), (512, 33, 96, 5.085, 4.765),
    (512, 61, 256, 4.659, 5.262), (512, 49, 192, 6.169, 6.450), (256, 245, 256, 4.614, 4.905), (1024, 33, 256, 8.437, 9.373), (1024, 49, 256, 11.30, 12.38),
    (512, 25, 256, 2.927, 3.253), (512, 33, 128, 3.562, 3.774), (384, 25.1, 128, 2.052, 2.131), (128, 25.2, 256, 0.554, 0.563), (256, 16.6, 256, 1.125, 1.169),
    (256, 33, 96, 1.467, 1.546), (128, 123, 64, 1.196, 1.250), (128, 66, 96, 0.759, 0.807),
]


def test_programs_are_read_ahead_where_that_was_measured_to_be_faster(cells):
    for B, mean, cus, ahead, without in AHEAD_MEASURED:
        assert cells.ahead(int(mean * B * B), B, cus) == (ahead < without), (B, mean, cus)
    assert not cells.ahead(60 * 127 * 127, 127, 256) and not cells.ahead(0, 128, 256) and not cells.ahead(1 << 30, 1024, 1)
    # parts of strata: 512 blocks of 61 and 49, 256 of 31 and 8 ratings a cell
    assert cells.ahead(61 << 18, 512, 256, 52) and cells.ahead(61 << 18, 512, 64, 100) and not cells.ahead(61 << 18, 512, 64) and not cells.ahead(49 << 18, 512, 256, 20)
    assert cells.ahead(31 << 16, 256, 64, 52) and not cells.ahead(31 << 16, 256, 256, 3) and not cells.ahead(8 << 16, 256, 256, 52)


# (cells of a launch, compute units): eight workgroups a unit where the launch has that many, and never together with reading ahead
@pytest.mark.parametrize("n,cus,want", [(1, 1, False), (7, 1, False), (8, 1, True), (56, 8, False), (57, 8, True), (64, 256, False), (512, 64, True), (512, 74, False), (1024, 146, True), (1024, 256, False)])
def test_sgd_cells_that_share_a_unit(cells, n, cus, want):
    assert cells.eight(n, cus) == want
    assert not (want and any(cells.ahead(mean << 20, 1024, cus, n) for mean in (2, 60, 1000)))


@pytest.fixture(scope="module")
def pr(tmp_path_factory):
    L = _compile(tmp_path_factory, "pr_rules", '''#include "pr_rules.h"
extern "C" int runs(uint32_t src, int64_t V, uint32_t cus, int hands_out) { return scatter_in_runs(src, V, cus, hands_out != 0); }
extern "C" int g_alone(uint32_t rows, uint32_t Qe, uint64_t total, uint32_t cus) { return gather_alone(rows, Qe, total, cus); }
extern "C" uint64_t g_least(uint32_t rows, uint64_t heaviest) { return least_gather_weight(rows, heaviest); }
extern "C" uint64_t least(uint64_t all) { return least_scatter_weight(all); }
extern "C" int s_alone(uint32_t src, uint64_t all, uint32_t cus) { return scatter_alone(src, all, cus); }
''')
    L.runs.argtypes = [ctypes.c_uint32, ctypes.c_int64, ctypes.c_uint32, ctypes.c_int]
    L.g_alone.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint32]
    L.g_least.argtypes, L.g_least.restype = [ctypes.c_uint32, ctypes.c_uint64], ctypes.c_uint64
    L.least.argtypes, L.least.restype = [ctypes.c_uint64], ctypes.c_uint64
    L.s_alone.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint32]
    return L


# (sources a partition, vertices, compute units, more tiles than workgroups, us an iteration with groups of eight, of four)
SCATTER_MEASURED = [
    (16384, 1 << 23, 64, 1, 1640, 1442), (16384, 1_000_003, 256, 0, 30.4, 31.4), (16384, 3_000_000, 128, 0, 123.0, 125.9),
    (32768, 1 << 24, 64, 1, 1815, 1968), (32768, 1 << 24, 64, 0, 326, 337), (32768, 1 << 25, 64, 0, 414, 439), (32768, 1 << 25, 64, 1, 932, 987),
    (32768, 1 << 24, 256, 0, 367, 349), (32768, 1 << 24, 256, 1, 816, 752), (32768, 1 << 24, 128, 1, 1142, 1105), (32768, 1 << 24, 128, 0, 534, 519),
    (32768, 3_000_000, 64, 0, 177, 187), (32768, 3_000_000, 256, 0, 83.0, 85.7), (32768, 1_000_003, 64, 0, 46.4, 48.6),
]


def test_scatter_groups_are_the_faster_ones_of_every_measured_size(pr):
    for src, V, cus, hands_out, eight, four in SCATTER_MEASURED:
        assert bool(pr.runs(src, V, cus, hands_out)) == (four < eight), (src, V, cus, hands_out)


# (thousands of messages and values a compute unit, units, us an iteration with two workgroups a unit, with one)
SCATTER_ALONE = [(9, 16, 18.1, 16.8), (22, 16, 27.5, 27.0), (53, 16, 64.8, 67.0), (84, 16, 40.0, 41.0), (9, 32, 18.6, 17.4), (22, 32, 24.8, 23.8),
                 (72, 32, 116.7, 123.0), (13, 64, 21.2, 19.6), (25, 64, 23.6, 22.0), (44, 64, 69.8, 76.2), (72, 64, 35.6, 37.0), (13, 128, 25.1, 23.2),
                 (27, 128, 39.4, 38.0), (58, 128, 47.8, 57.5), (98, 128, 48.0, 50.0), (17, 256, 33.5, 32.1), (29, 256, 39.6, 37.5), (49, 256, 41.8, 40.4),
                 (72, 256, 55.5, 63.0)]


def test_scatter_workgroups_a_unit_are_the_faster_number(pr):
    for share, cus, two, one in SCATTER_ALONE:
        assert bool(pr.s_alone(16384, share * 1000 * cus, cus)) == (one < two), (share, cus)
    assert pr.s_alone(32768, 1 << 40, 16)                       # the large kernel fits once


# (thousands of weight a compute unit, ranges with edges, units, us an iteration with two workgroups a unit, with one)
GATHER_ALONE = [(65, 2, 16, 22.2, 19.6), (130, 8, 16, 26.9, 28.8), (256, 8, 16, 37.6, 42.9), (33, 2, 32, 23.4, 18.6), (65, 8, 32, 24.8, 21.3),
                (130, 13, 32, 28.6, 29.3), (65, 13, 64, 26.8, 21.8), (137, 32, 64, 35.6, 39.4), (68, 32, 128, 28.4, 23.2), (164, 64, 128, 39.1, 38.4),
                (80, 64, 256, 34.9, 30.8), (130, 49, 256, 43.5, 37.0), (330, 64, 64, 50.5, 58.0), (260, 49, 128, 47.8, 53.4)]


def test_gather_workgroups_a_unit_are_the_faster_number(pr):
    for share, Qe, cus, two, one in GATHER_ALONE:
        assert bool(pr.g_alone(8192, Qe, share * 1000 * cus, cus)) == (one < two), (share, cus)
    assert pr.g_alone(16384, 1000, 1 << 40, 16)                 # the large kernel fits once
    assert not pr.g_alone(8192, 9, 1000, 16)                    # fewer than two units a range


def test_least_gather_piece(pr):
    for rows, least in ((8192, 49152), (16384, 65536)):
        assert pr.g_least(rows, 0) == pr.g_least(rows, 2_800_000) == least and pr.g_least(rows, 1 << 24) == 29 * 4096


def test_least_scatter_tile(pr):
    assert pr.least(0) == 1 and pr.least(1) == 1
    for all_ in (300, 8200, 10_000, 16_384):
        assert pr.least(all_) == all_                           # one tile
    assert pr.least(16_385) == pr.least(26_000) == 4096         # several
    assert pr.least(1 << 26) == 6 * 8192


@pytest.fixture(scope="module")
def gemm(tmp_path_factory):
    L = _compile(tmp_path_factory, "gemm_tiles", '''#include "gemm_tiles.h"
extern "C" int choose(int M, int N, int K, int cus) { return gemm_choose(M, N, K, cus); }
extern "C" int tiles(void) { return kGemmTiles; }
''')
    return L


# (compute units of the stream, (M, N, K), us with every tile, operands not in a cache)
GEMM_MEASURED = [
    (32, (256, 15616, 1216), [59.1, 92.6, 89.1, 132.1, 193.7, 226.1, 73.4]), (32, (512, 11008, 64), [24.9, 28.8, 21.5, 25.1, 37.4, 104.5, 15.7]),
    (32, (256, 16384, 16384), [567.3, 912.0, 1034.4, 1638.0, 2518.4, 2432.0, 858.0]), (32, (1280, 3840, 192), [30.4, 30.1, 24.6, 30.2, 43.1, 98.0, 22.1]),
    (64, (256, 15616, 1216), [31.7, 48.4, 47.5, 68.2, 100.4, 117.1, 38.2]), (64, (512, 11008, 64), [17.4, 15.9, 12.7, 14.9, 20.5, 54.8, 9.6]),
    (64, (2048, 2048, 128), [10.4, 11.6, 9.4, 11.0, 15.8, 41.5, 8.3]), (64, (256, 16384, 16384), [301.8, 468.3, 530.9, 824.1, 1281.0, 1214.4, 434.1]),
    (64, (512, 15104, 1024), [50.7, 73.1, 70.1, 106.6, 159.0, 185.1, 61.7]), (64, (1792, 4096, 640), [35.4, 46.6, 39.7, 51.3, 77.9, 111.7, 41.4]),
    (128, (256, 15616, 1216), [31.7, 26.6, 26.6, 37.2, 51.9, 61.2, 28.8]), (128, (512, 11008, 64), [10.2, 11.5, 8.8, 9.2, 11.9, 28.8, 7.3]),
    (128, (256, 16384, 16384), [300.6, 248.6, 280.6, 424.9, 646.5, 636.8, 335.7]), (128, (512, 15104, 1024), [28.3, 39.1, 39.7, 57.9, 85.9, 94.5, 34.0]),
    (256, (256, 15616, 1216), [31.7, 26.6, 19.4, 21.7, 28.2, 32.5, 28.7]), (256, (2048, 2048, 128), [10.4, 7.1, 5.5, 5.1, 6.2, 12.3, 6.3]),
    (256, (256, 16384, 16384), [318.9, 249.8, 204.2, 229.6, 331.6, 332.0, 342.9]), (256, (1792, 4096, 640), [20.7, 16.1, 15.1, 19.5, 25.5, 34.1, 17.8]),
]


def test_gemm_tiles_are_the_fast_ones_of_every_measured_size(gemm):
    assert gemm.tiles() == 7
    for cus, shape, us in GEMM_MEASURED:
        assert us[gemm.choose(*shape, cus)] <= 1.1 * min(us), (cus, shape)


def test_gemm_rows_beyond_a_32_bit_offset_take_the_kernel_with_64_bit_addresses(gemm):
    for cus in (16, 256):
        for M, N in ((256, 256), (256, 512)):                   # (A and B may be one buffer: 2^29 values of K fit the memory)
            for K in (306_783_424, 1 << 29, 2_147_483_584):
                assert 7 * 2 * K + 112 >= 1 << 32 and gemm.choose(M, N, K, cus) == gemm.tiles() - 1
            assert gemm.choose(M, N, (1 << 27) + 64, cus) == gemm.tiles() - 1
            assert 0 <= gemm.choose(M, N, 1 << 27, cus) < gemm.tiles() - 1 and 7 * 2 * (1 << 27) + 112 < 1 << 31

"""The rules that choose between the forms of a kernel (csrc/agc_dispatch.h), compiled on their own with the host
compiler: on either side of the lines, at shapes where both forms were timed.  CPU only."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "agc_dispatch.h"
extern "C" int parts(int64_t d, int n, int k, int nnz, int band, int norm, int bucket)
{
    return agc::use_parts(d, n, k, nnz, band, norm != 0, bucket != 0);
}
extern "C" int decode_per_cu(unsigned lds_bytes) { return agc::decode_per_cu(lds_bytes); }
extern "C" int64_t decode_groups(int64_t tiles, int chunks, int per_cu) { return agc::decode_groups(tiles, chunks, per_cu); }
extern "C" int decode_is_direct(int n, int64_t d) { return agc::decode_is_direct(n, d); }
extern "C" int decode_coords(int64_t d, int two, int many_scales, int sum_bits)
{
    return agc::decode_coords(d, two != 0, many_scales != 0, sum_bits);
}
extern "C" int ls_fold(int64_t n_rows, int64_t rows_per_part, int n_feat) { return agc::ls_fold(n_rows, rows_per_part, n_feat); }
extern "C" int ls_reduce_few(int wg_per_part) { return agc::ls_reduce_few(wg_per_part); }
extern "C" unsigned first_group(int64_t d, unsigned groups) { return agc::first_group(d, groups); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("dispatch")
    (tmp / "driver.cpp").write_text(DRIVER)
    cxx = shutil.which("g++") or shutil.which("c++")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared",
                    "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "paper_2605_15890_amd", "csrc"), str(tmp / "driver.cpp"),
                    "-o", str(tmp / "librules.so")], check=True)
    lib = ctypes.CDLL(str(tmp / "librules.so"))
    lib.parts.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 6
    lib.decode_per_cu.argtypes = [ctypes.c_uint]
    lib.decode_groups.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    lib.decode_groups.restype = ctypes.c_int64
    lib.decode_is_direct.argtypes = [ctypes.c_int, ctypes.c_int64]
    lib.decode_coords.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 3
    lib.ls_fold.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.ls_reduce_few.argtypes = [ctypes.c_int]
    lib.first_group.argtypes = [ctypes.c_int64, ctypes.c_uint]
    lib.first_group.restype = ctypes.c_uint
    return lib


@pytest.mark.parametrize("shared,d,n,k,nnz,band,norm,bucket", [
    # cyclic band: whole vectors of 2^19 coordinates took 0.62 to 0.87 of the time in the long form
    (0, 524288, 16, 16, 48, 3, 0, 0), (0, 524288, 64, 64, 192, 3, 1, 0), (0, 524288, 32, 32, 256, 8, 0, 1),
    (0, 393216, 128, 128, 384, 3, 0, 0), (0, 262144, 32, 32, 96, 3, 1, 0),
    (1, 262144, 32, 32, 96, 3, 0, 0), (1, 196608, 32, 32, 96, 3, 1, 0),
    # a band that ends inside a block: as one of whole blocks (64 x 500000 Euclidean 100 us in parts, 69 in the long form)
    (0, 500000, 64, 64, 192, 3, 1, 0), (0, 500000, 64, 64, 192, 3, 0, 1), (0, 327681, 64, 64, 192, 3, 0, 0),
    (1, 262143, 64, 64, 192, 3, 0, 0), (0, 262145, 64, 64, 192, 3, 0, 0), (1, 196607, 64, 64, 192, 3, 1, 0),
    (0, 196609, 64, 64, 192, 3, 1, 0), (1, 196607, 5, 5, 10, 2, 0, 1), (0, 196609, 5, 5, 10, 2, 0, 1),
    (1, 65536, 48, 48, 144, 3, 0, 0), (1, 4096, 4, 4, 8, 2, 0, 0), (0, 262144, 4, 4, 8, 2, 0, 0),
    # one or two workers share nothing
    (0, 200000, 1, 1, 1, 1, 0, 0), (0, 262144, 2, 2, 4, 2, 0, 0), (0, 4096, 2, 2, 4, 2, 1, 0),
    # window driver: three partitions a worker in runs of up to eight
    (0, 262144, 12, 36, 80, -8, 0, 0), (0, 65536, 8, 24, 50, -8, 1, 0), (1, 4096, 24, 72, 95, -8, 0, 0),
    (1, 65536, 48, 48, 96, -4, 0, 0), (0, 400000, 50, 50, 100, -4, 0, 0), (1, 250001, 48, 48, 96, -4, 1, 0),
    # gather driver
    (1, 200000, 24, 24, 96, 0, 0, 0), (1, 900000, 24, 24, 192, 0, 0, 0), (0, 1048576, 48, 48, 96, 0, 0, 0),
    (0, 786432, 12, 12, 48, 0, 0, 0), (1, 500000, 60, 60, 480, 0, 1, 0)])
def test_workers_are_shared_where_that_was_measured_to_be_faster(rules, shared, d, n, k, nnz, band, norm, bucket):
    assert rules.parts(d, n, k, nnz, band, norm, bucket) == shared


@pytest.mark.parametrize("band", [-8, -4, -2, 0, 1, 8])
def test_sharing_rule_at_the_ends_of_its_ranges(rules, band):
    """No overflow (the driver is built with the sanitizer), and long vectors always take the long form."""
    for n in (1, 3, 4, 255, 256):
        for k in (1, n, 65536):
            for nnz in (0, k, 2 ** 24):
                for norm, bucket in ((0, 0), (1, 0), (0, 1), (1, 1)):
                    assert rules.parts(2 ** 33, n, k, nnz, band, norm, bucket) == 0
                    assert rules.parts(256 * 4096 + 1, n, k, nnz, band, norm, bucket) == 0
                    assert rules.parts(1, n, k, nnz, band, norm, bucket) == (n >= 3)


@pytest.mark.parametrize("d,early", [(1, 0), (1_000_000, 0), (1024 * 1024, 0), (1024 * 1024 - 1, 0), (1024 * 1024 + 1, 64),
                                     (5_400_003, 64), (11_700_224, 0), (25_600_000, 0), (2 ** 33 - 1, 64)])
def test_the_block_that_the_vector_ends_in_starts_early(rules, d, early):
    """Only where the vector ends inside a block and the chip does not hold all groups at once (256 workers x
    1 000 000: 5 % slower in any other order)."""
    groups = -(-(-(-d // 256)) // 4)
    assert rules.first_group(d, groups) == (groups - early if early else 0)


def test_decode_launches_what_a_compute_unit_holds(rules):
    """160 KB of LDS: six workgroups with one scale per vector, five with bucket-wise scales and with layers, four
    with layers and two tracks."""
    assert [rules.decode_per_cu(b) for b in (24624, 28976, 28720, 32816)] == [6, 5, 5, 4]


@pytest.mark.parametrize("tiles,chunks,per_cu,groups", [
    (1, 1, 6, 1), (1319, 9, 6, 1319), (1319, 2, 5, 1280), (6250, 2, 6, 1536), (6250, 3, 5, 1280), (6250, 4, 6, 6250),
    (6250, 20, 5, 6250), (2637, 20, 6, 1536), (2857, 20, 6, 2857), (2560, 20, 5, 2560), (2 ** 21, 1, 4, 1024)])
def test_decode_walks_over_the_tiles_where_a_tile_is_little_work(rules, tiles, chunks, per_cu, groups):
    assert rules.decode_groups(tiles, chunks, per_cu) == groups


@pytest.mark.parametrize("n,d,direct", [(0, 1, 1), (1, 4096, 1), (2, 25_600_000, 1), (3, 25_600_000, 0), (4, 2 ** 25 - 1, 0),
                                        (4, 2 ** 25, 1), (5, 2 ** 33, 0)])
def test_decode_of_a_few_workers_takes_no_chunks(rules, n, d, direct):
    assert rules.decode_is_direct(n, d) == direct


@pytest.mark.parametrize("d,two,many_scales,sum_bits,coords", [
    (2 ** 21, 0, 0, 192, 8), (5 * 2 ** 20 - 1, 0, 0, 192, 8), (5 * 2 ** 20, 0, 0, 192, 16), (5_400_000, 0, 0, 40, 8),
    (25_600_000, 0, 0, 32, 8), (25_600_000, 0, 0, 41, 16), (15 * 2 ** 18 - 1, 0, 1, 192, 8), (15 * 2 ** 18, 0, 1, 192, 16),
    (25_600_000, 1, 0, 307, 8), (25_600_000, 1, 1, 307, 8)])
def test_decode_takes_sixteen_coordinates_per_lane_on_long_vectors(rules, d, two, many_scales, sum_bits, coords):
    assert rules.decode_coords(d, two, many_scales, sum_bits) == coords


@pytest.mark.parametrize("k,rows,n_feat,fold", [
    (1, 4096, 128, 1), (4, 16, 128, 1), (32, 16, 1024, 1), (128, 32, 128, 1), (128, 48, 1024, 1), (128, 48, 128, 1),
    (128, 64, 128, 2), (128, 96, 256, 2), (128, 128, 128, 4), (16, 512, 128, 16), (16, 512, 256, 8), (16, 512, 384, 4),
    (16, 512, 512, 4), (16, 512, 640, 2), (16, 512, 1024, 2), (16, 512, 1152, 1), (32, 32768, 4096, 1), (1, 16384, 128, 16)])
def test_least_squares_folds_no_wider_than_a_partition_fills(rules, k, rows, n_feat, fold):
    assert rules.ls_fold(k * rows, rows, n_feat) == fold


def test_least_squares_sums_few_parts_by_one_thread(rules):
    assert [rules.ls_reduce_few(p) for p in (1, 16, 17, 512)] == [1, 1, 0, 0]

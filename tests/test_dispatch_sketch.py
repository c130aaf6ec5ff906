"""The rule that decides between one read of G and two (csrc/agc_dispatch.h), compiled on its own with the host compiler:
on either side of its line, at shapes where both forms were timed, and at the ends of its ranges.  CPU only."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "agc_dispatch.h"
extern "C" int one_read(int64_t d, int n, int k, double levels, int gather, int parts)
{
    return agc::use_sketch(d, n, k, levels, gather != 0, parts != 0, agc::sketch_cap(n));
}
extern "C" int fits(int n, int k, int64_t d, size_t free_bytes, size_t total_bytes)
{
    return agc::sketch_fits(n, k, d, free_bytes, total_bytes);
}
extern "C" int64_t bytes(int n, int64_t d) { return agc::sketch_bytes(n, d); }
extern "C" int64_t block(int64_t nblocks, int samples, uint64_t seed, uint64_t step, int64_t e)
{
    return agc::sample_block(agc::sample_runs(nblocks, samples, seed, step), e);
}
extern "C" int count(int64_t nblocks) { return agc::sample_count(nblocks); }
extern "C" int cap(int n) { return agc::sketch_cap(n); }
extern "C" int one_read_max(int64_t d, int n, int k, double levels) { return agc::use_sketch_max(d, n, k, levels); }
extern "C" int max_cap(int n, int k) { return agc::sketch_max_cap(n, k); }
extern "C" unsigned max_limit(int k, int samples) { return agc::sketch_max_limit(k, samples); }
extern "C" unsigned read_cost() { return agc::kReadCost; }
extern "C" int64_t max_bytes(int n, int k, int64_t d) { return agc::sketch_bytes(n, d, agc::sketch_max_cap(n, k)); }
extern "C" int max_fits(int n, int k, int64_t d, size_t free_bytes, size_t total_bytes)
{
    return agc::sketch_fits(n, k, d, free_bytes, total_bytes, agc::sketch_max_cap(n, k));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("sketch")
    (tmp / "driver.cpp").write_text(DRIVER)
    cxx = shutil.which("g++") or shutil.which("c++")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared",
                    "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "paper_2605_15890_amd", "csrc"), str(tmp / "driver.cpp"),
                    "-o", str(tmp / "librules.so")], check=True)
    lib = ctypes.CDLL(str(tmp / "librules.so"))
    lib.one_read.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_double, ctypes.c_int, ctypes.c_int]
    lib.fits.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_size_t, ctypes.c_size_t]
    lib.bytes.argtypes, lib.bytes.restype = [ctypes.c_int, ctypes.c_int64], ctypes.c_int64
    lib.one_read_max.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_double]
    lib.max_bytes.argtypes, lib.max_bytes.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_int64], ctypes.c_int64
    lib.max_fits.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_size_t, ctypes.c_size_t]
    lib.max_limit.restype = lib.read_cost.restype = ctypes.c_uint
    lib.count.argtypes = [ctypes.c_int64]
    lib.block.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int64]
    lib.block.restype = ctypes.c_int64
    return lib


@pytest.mark.parametrize("one,d,n,k,bits", [
    (1, 25_600_000, 64, 64, 3), (1, 11_700_000, 32, 32, 4), (1, 5_400_003, 50, 50, 6), (1, 5_400_001, 10, 30, 3),
    (1, 1_000_001, 64, 64, 3), (1, 3_000_000, 256, 256, 2), (1, 12_000_000, 64, 64, 6),
    (0, 25_600_000, 4, 4, 8), (0, 5_400_000, 64, 64, 8), (0, 4_000_000, 8, 8, 3), (0, 500_000, 32, 32, 3),
    (0, 2_000_000, 16, 16, 6), (0, 65536, 128, 128, 3), (0, 1_000_001, 128, 128, 6)])
def test_one_read_where_that_was_measured_to_be_faster(rules, one, d, n, k, bits):
    assert rules.one_read(d, n, k, float(n * (2 ** (bits - 1) - 1)), 0, 0) == one
    assert rules.one_read(d, n, k, float(n * (2 ** (bits - 1) - 1)), 1, 1) == 0


@pytest.mark.parametrize("one,d,n,k,levels,gather", [
    # sixty layers of very different magnitude: these took the second pass for up to a seventh of the groups, and longer than two reads
    (0, 700_353, 59, 59, 857, 0), (0, 965_376, 59, 59, 1217, 0), (0, 1_271_552, 58, 58, 1038, 0), (0, 1_294_221, 60, 60, 1184, 0),
    (0, 359_951, 48, 123, 896, 1), (0, 583_808, 31, 74, 623, 1), (0, 886_016, 44, 73, 914, 1), (0, 1_647_104, 14, 35, 1018, 1),
    # and these did not, or gained more than that pass takes
    (1, 1_050_112, 41, 41, 150, 0), (1, 4_071_000, 31, 31, 330, 0), (1, 2_586_889, 45, 45, 480, 0), (1, 5_400_003, 50, 50, 4078, 0),
    (1, 25_600_000, 64, 64, 8128, 0), (1, 4_924_838, 34, 78, 1060, 1), (1, 541_184, 45, 127, 190, 1),
    # few workers: signs and tables by coordinates outweigh the rows
    (0, 19_554_560, 6, 6, 96, 0), (0, 25_600_000, 5, 5, 40, 0)])
def test_one_read_takes_the_second_pass_into_account(rules, one, d, n, k, levels, gather):
    assert rules.one_read(d, n, k, float(levels), gather, 0) == one


def test_ends_of_the_ranges(rules):
    """No overflow (the driver is built with the sanitizer), room for a whole number of 16-byte pieces in 64 KB of LDS."""
    for n in range(1, 257):
        cap = rules.cap(n)
        assert cap >= 32 and cap % 2 == 0 and cap <= 32 * n
        lds = 32 * n + 4096 * -(-n // 32) + 32 * cap
        assert lds <= 64 * 1024
        assert 128 * 1280 // (-(-lds // 1280) * 1280) >= (4 if n <= 96 else 3 if n <= 160 else 2)   # of a compute unit's LDS
        for d in (1, 2 ** 33):
            for k in (1, 65536):
                for level in (1, 32767):
                    one = rules.one_read(d, n, k, float(n * level), 0, 0)
                    assert not (d == 1 and one)


def test_a_program_that_fills_the_card_keeps_its_memory(rules):
    """A context may be made before the gradients: G counts whether it is there or not."""
    total = 288 * 10 ** 9
    need = rules.bytes(64, 25_600_000)
    assert need == 100_000 * (2048 + 8 * rules.cap(64))
    assert rules.fits(64, 64, 25_600_000, total, total) and rules.fits(64, 64, 25_600_000, 8 * need, total)
    assert not rules.fits(64, 64, 25_600_000, 8 * need - 8, total)
    assert rules.fits(64, 64, 480_000_000, total, total) and not rules.fits(64, 64, 1_000_000_000, total, total)
    for n, k, d in ((1, 1, 2 ** 33), (256, 65536, 2 ** 33), (256, 4, 2 ** 33)):
        assert not rules.fits(n, k, d, total, total)
    assert not rules.fits(1, 1, 1, 0, 0)


@pytest.mark.parametrize("one,d,n,k,levels", [
    (1, 25_600_000, 64, 64, 192), (1, 27_000_000, 40, 40, 160), (1, 90_000_000, 12, 12, 36), (1, 36_000_000, 10, 30, 40),
    (1, 25_600_000, 64, 64, 1024), (0, 25_600_000, 64, 64, 1025),                        # wide codes
    (1, 1 << 24, 64, 64, 192), (0, (1 << 24) - 1, 64, 64, 192), (0, 12_800_000, 64, 64, 192),   # less than 4 GB
    (1, 20480 * 256, 128, 205, 384), (0, 20480 * 256 - 1, 128, 256, 384),                # too short
    (0, 8_500_000, 129, 129, 387), (0, 98_000_000, 11, 11, 33), (0, 2 ** 33, 1, 1, 1), (1, 2 ** 33, 128, 65536, 128)])
def test_one_read_of_the_largest_magnitude(rules, one, d, n, k, levels):
    assert rules.one_read_max(d, n, k, float(levels)) == one


@pytest.mark.parametrize("k,cost,one", [  # of steps in both forms
    (64, 0.13, 1), (64, 0.31, 1), (64, 0.43, 1), (64, 1.0, 0), (40, 0.28, 1), (24, 0.28, 1), (12, 0.08, 1), (12, 0.17, 0), (12, 0.22, 0),
    (16, 0.25, 1), (16, 0.43, 0), (16, 0.6, 0), (30, 0.02, 1)])
def test_what_the_sampled_blocks_may_cost(rules, k, cost, one):
    for samples in (163, 512):
        assert (int(cost * rules.read_cost() * samples) <= rules.max_limit(k, samples)) == one


def test_ends_of_the_ranges_of_the_largest_magnitude(rules):
    """Records leave the ring of 512 in halves of it, and their array holds the sample's sums, four bytes a worker and block."""
    for k in (1, 2, 7, 8, 9, 11, 12, 13, 64, 65535, 65536):
        assert rules.max_limit(k, 1) <= rules.read_cost() // 2 and rules.max_limit(k, 512) < 2 ** 15
        assert (rules.max_limit(k, 512) == 0) == (k <= 8)
        for n in range(1, 257):
            cap = rules.max_cap(n, k)
            assert cap >= 256 and cap % 256 == 0 and cap - 256 < min(32 * k, 128 * n) <= cap and 8 * cap >= 4 * n
            assert cap <= 256 * n
    need = rules.max_bytes(64, 64, 25_600_000)
    assert need == 100_000 * (2048 + 8 * 2048)
    total = 288 * 10 ** 9
    assert rules.max_fits(64, 64, 25_600_000, 8 * need, total) and not rules.max_fits(64, 64, 25_600_000, 8 * need - 8, total)
    assert not rules.max_fits(256, 65536, 2 ** 33, total, total) and not rules.max_fits(1, 1, 1, 0, 0)


@pytest.mark.parametrize("nblocks,samples", [(1, 1), (63, 1), (64, 2), (4096, 128), (10_547, 329), (32768, 512), (100_000, 512),
                                             (2 ** 25, 512)])
def test_samples_spread_over_the_vector_and_over_the_columns_of_matrices(rules, nblocks, samples):
    """One block of each of equal runs, other ones with every seed and step; with rows of 16 to 64 blocks all columns are met
    (for each of them the number of samples in 40 steps is a sum of nearly independent draws: eight standard deviations)."""
    assert rules.count(nblocks) == samples and samples <= -(-nblocks // 4)   # rows of the scratch
    draws = [[rules.block(nblocks, samples, 2 ** 64 - 1 - t % 3, t, e) for e in range(samples)] for t in range(40)]
    for blocks in draws:
        at = 0
        for e, b in enumerate(blocks):
            length = nblocks // samples + (e < nblocks % samples)
            assert at <= b < at + length
            at += length
        assert at == nblocks
    if samples >= 64:
        assert len({tuple(b) for b in draws}) == 40
        for width in (16, 32, 64):
            count = [0] * width
            for blocks in draws:
                for b in blocks:
                    count[b % width] += 1
            mean = 40 * samples / width
            assert all(abs(c - mean) < 8 * mean ** 0.5 for c in count)

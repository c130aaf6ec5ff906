"""Which codes have their rows of G streamed once (csrc/agc_stream.h), compiled on its own with the host compiler, and the order of
their entries: a model of the driver forms every worker's row from them.  CPU only."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from gpu_util import cyclic_csr, monotone_csr, random_csr
from test_gpu_long_runs import CODES, _runs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <string.h>
#include "agc_stream.h"
extern "C" int records(int n, int k, const int32_t* row_ptr, const int32_t* col, const float* val, agc::StreamRec* out)
{
    const std::vector<agc::StreamRec> r = agc::stream_records(n, k, row_ptr, col, val);
    if (!r.empty()) memcpy(out, r.data(), r.size() * sizeof r[0]);
    return (int)r.size();
}
extern "C" int slots() { return agc::kStreamSlots; }
"""
REC = np.dtype([("col", np.int32), ("val", np.float32), ("slot", np.int32), ("last", np.int32)])


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("stream")
    (tmp / "driver.cpp").write_text(DRIVER)
    cxx = shutil.which("g++") or shutil.which("c++")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared",
                    "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "paper_2605_15890_amd", "csrc"), str(tmp / "driver.cpp"),
                    "-o", str(tmp / "libstream.so")], check=True)
    return ctypes.CDLL(str(tmp / "libstream.so"))


def _records(lib, csr, k):
    row_ptr, col, val = csr
    out = np.zeros(len(col) + 1, REC)
    count = lib.records(len(row_ptr) - 1, k, *(a.ctypes.data_as(ctypes.c_void_p) for a in (row_ptr, col, val, out)))
    return out[:count]


def _formed(recs, k, slots):
    """What encode_stream does with them: the terms of every worker, in order."""
    workers, open_, at = [], [[] for _ in range(slots)], 0
    for j in range(k):
        while recs[at]["col"] == j:
            r = recs[at]
            open_[r["slot"]].append((j, float(r["val"])))
            if r["last"]:
                workers.append(open_.pop(0))
                open_.append([])
            at += 1
    assert at == len(recs) - 1 and not any(open_)   # the sentinel is left, and nobody is open
    return workers


def _check(lib, csr, k):
    recs = _records(lib, csr, k)
    assert len(recs) == len(csr[1]) + 1
    want = [[(int(c), float(v)) for c, v in zip(csr[1][a:b], csr[2][a:b])] for a, b in zip(csr[0], csr[0][1:])]
    assert _formed(recs, k, lib.slots()) == want


@pytest.mark.parametrize("name", sorted(CODES))
def test_codes_of_the_parity_tests(lib, name):
    runs, k = CODES[name]
    csr = _runs(np.random.default_rng(len(name)), runs)
    if name in ("three_open", "gaps", "two_rows_shared"):
        assert len(_records(lib, csr, k)) == 0
    else:
        _check(lib, csr, k)


def test_rows_that_nobody_holds_are_not_streamed(lib):
    """Before the first run, between two, after the last, and none."""
    rng = np.random.default_rng(1)
    for runs, k, streamed in (([(0, 12), (12, 12)], 24, True), ([(0, 12), (12, 12)], 25, False), ([(1, 12), (13, 12)], 25, False),
                              ([(0, 12), (13, 12)], 25, False), ([(10 * i, 10) for i in range(10)], 100, True),
                              ([(11 * i, 10) for i in range(10)], 110, False), ([(0, 20), (100, 20)], 120, False)):
        csr = _runs(rng, runs)
        assert (len(_records(lib, csr, k)) > 0) == streamed, (runs, k)
        if streamed:
            _check(lib, csr, k)


def test_random_codes(lib):
    """Runs that share up to three columns with the one before, some of them a single column; and codes that are not runs."""
    rng = np.random.default_rng(2)
    taken = 0
    for _ in range(400):
        n, lo, hi, runs = int(rng.integers(1, 20)), 0, 0, []
        for _ in range(n):
            lo = max(lo, hi - int(rng.integers(0, 4))) if runs else 0
            hi = max(hi, lo + int(rng.integers(1, 12)))
            runs.append((lo, hi - lo))
        csr = _runs(rng, runs)
        covered = np.zeros((n, hi), int)
        for i, (a, length) in enumerate(runs):
            covered[i, a:a + length] = 1
        if covered.sum(0).max() <= lib.slots():
            _check(lib, csr, hi)
        if len(_records(lib, csr, hi)):
            _check(lib, csr, hi)
            taken += 1
    assert taken > 50
    for csr, k in ((cyclic_csr(rng, 9, 3), 9), (random_csr(rng, 6, 30, 9), 30), (monotone_csr(rng, 8, 30, 1), 30)):
        recs = _records(lib, csr, k)
        if len(recs):
            _check(lib, csr, k)

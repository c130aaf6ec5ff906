"""Codes whose rows are long runs of columns, few of them open at a time: rows of G are streamed once.  Runs longer than any
window, workers of one column between them, overlaps of one row and of two, fewer rows than are
requested ahead, zeros of both signs; every kind of scale and both forms of the worker side.  Codes that have too many workers
open or columns that nobody holds take the general driver (test_stream_records.py asserts which do).  Bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import compare_with_oracle, to_device

pytestmark = pytest.mark.gpu


def _runs(rng, runs):
    """CSR of the given (first, length) of every worker."""
    row_ptr = np.concatenate([[0], np.cumsum([length for _, length in runs])]).astype(np.int32)
    col = np.concatenate([np.arange(lo, lo + length) for lo, length in runs]).astype(np.int32)
    return row_ptr, col, rng.uniform(-1.0, 1.0, len(col)).astype(np.float32)


CODES = {  # runs, columns
    "one_row_shared": ([(0, 11), (10, 9), (18, 12)], 30),
    "short_between": ([(0, 12), (11, 1), (11, 1), (11, 1), (11, 10), (20, 1), (20, 3)], 23),
    "two_rows_shared": ([(0, 10), (8, 12), (18, 2), (18, 9)], 27),   # three open at columns 18 and 19: the general driver
    "two_rows_of_two": ([(0, 10), (8, 12), (18, 9), (25, 2), (26, 1)], 27),
    "three_open": ([(0, 12), (5, 12), (9, 12)], 21),   # the general driver
    "gaps": ([(3, 9), (14, 1), (20, 17)], 41),         # the general driver: columns without a holder
    "one_worker": ([(0, 9)], 9),
    "whole_and_last": ([(0, 33), (32, 1), (32, 1)], 33),
}


def _G(rng, k, d):
    G = rng.standard_normal((k, d)).astype(np.float32)
    G[:, ::7] = 0.0
    G[:, 3::11] = -0.0
    return G


@pytest.mark.parametrize("name", sorted(CODES))
@pytest.mark.parametrize("mode", [api.AGC_SCALE_MAXABS, api.AGC_SCALE_L2])
@pytest.mark.parametrize("d", [1, 300, 5 * 1024 + 77])
@pytest.mark.parametrize("form", ["two_reads", "one_read", "bucket", "many_bits"])
def test_long_runs(name, mode, d, form):
    import torch
    rng = np.random.default_rng([d, mode, len(name)])
    runs, k = CODES[name]
    n = len(runs)
    csr = _runs(rng, runs)
    bits = rng.integers(2, 9, n).astype(np.uint8) if form != "many_bits" else np.full(n, 16, np.uint8)
    w, mask = rng.uniform(0.2, 3.0, n).astype(np.float32), (rng.random(n) < 0.7).astype(np.uint8)
    G = _G(rng, k, d)
    ctx = api.Context(n, k, d, scale_mode=mode, bucket=256 if form == "bucket" else 0)
    ctx.agc_set_code(*csr)
    assert ctx.agc_code_path() == 0
    ctx.agc_debug_force_long()
    if form == "one_read":
        ctx.agc_debug_sketch(1) if mode == api.AGC_SCALE_L2 else ctx.agc_debug_sketch_max(1)
    codes, scales, ghat = ctx.alloc_outputs(bits)
    ctx.agc_step(to_device(G), bits, w, mask, 5, 6, codes, scales, ghat)
    torch.cuda.synchronize()
    out = [c.cpu().numpy() for c in codes], scales.cpu().numpy(), ghat.cpu().numpy()
    ctx.close()
    if form == "bucket":
        o = O.step_bucket(G, O.Csr(*csr, k), bits, w, mask, 5, 6, mode)
        assert all(np.array_equal(a, b) for a, b in zip(out[0], o[0]))
        assert np.array_equal(out[1].view(np.uint32), o[1].view(np.uint32))
        assert np.array_equal(out[2].view(np.uint32), o[2].view(np.uint32))
    else:
        compare_with_oracle(G, k, *csr, bits, w, mask, 5, 6, mode, out, tag=(name, form))


@pytest.mark.parametrize("mode", [api.AGC_SCALE_MAXABS, api.AGC_SCALE_L2])
def test_forty_workers_in_several_fills(mode):
    """More codes than one fill of the staging area holds, rows non-temporal and kept."""
    import torch
    rng = np.random.default_rng(3)
    runs = [(i // 4 * 10, 1) if i % 4 else (max(0, i // 4 * 10 - 10), 11 if i else 1) for i in range(40)]
    k, n, d = 91, 40, (1 << 20) + 77   # 4 bytes x 91 x 1 M: above what the memory-side cache holds
    csr = _runs(rng, runs)
    bits, w, mask = np.full(n, 13, np.uint8), np.ones(n, np.float32), (rng.random(n) < 0.7).astype(np.uint8)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    for length in (d, 40000):
        G = api.padded_rows(k, length)
        G.normal_(generator=gen)
        outs = []
        for generic in (False, True):
            ctx = api.Context(n, k, length, scale_mode=mode, force_generic=generic)
            ctx.agc_set_code(*csr)
            ctx.agc_debug_force_long()
            codes, scales, ghat = ctx.alloc_outputs(bits)
            ctx.agc_step(G, bits, w, mask, 5, 6, codes, scales, ghat)
            torch.cuda.synchronize()
            outs.append([c.cpu().numpy() for c in codes] + [scales.cpu().numpy().view(np.uint32), ghat.cpu().numpy().view(np.uint32)])
            ctx.close()
        assert all(np.array_equal(a, b) for a, b in zip(*outs))


def _both_drivers(csr, k, G, bits, w, mask, layers=None):
    """Codes, scales and estimate of the streaming driver and of the general one, and the form that the first took."""
    import torch
    outs, last = [], None
    for generic in (False, True):
        ctx = api.Context(len(bits), k, G.shape[1], force_generic=generic)
        ctx.agc_set_code(*csr)
        if layers is not None:
            ctx.agc_set_layers(np.array(layers, np.int64))
        elif generic:
            ctx.agc_debug_sketch_max(2)
        codes, scales, ghat = ctx.alloc_outputs(bits)
        ctx.agc_step(G, bits, w, mask, 5, 6, codes, scales, ghat)
        torch.cuda.synchronize()
        last = last or ctx.agc_debug_sketch_last()
        outs.append([*codes, scales.view(torch.int32), ghat.view(torch.int32)])
        ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    return last


@pytest.mark.parametrize("d", [20480 * 256, 20481 * 256 + 77, 20482 * 256 - 3])
@pytest.mark.parametrize("layers", [False, True])
def test_two_blocks_a_wave(d, layers):
    """From 20480 blocks a wave of the scale pass takes two: whole pairs, a single block and a piece of one at the end, and layers that
    end between the two blocks of a pair.  Against the general driver, which takes one."""
    import torch
    rng = np.random.default_rng([d, layers])
    runs, k = CODES["two_rows_of_two"]
    csr, n = _runs(rng, runs), len(runs)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    G = api.padded_rows(k, d)
    G.normal_(generator=gen)
    G[:, 5::1001] = -0.0
    w, mask = rng.uniform(0.2, 3.0, n).astype(np.float32), np.ones(n, np.uint8)
    last = _both_drivers(csr, k, G, np.full(n, 5, np.uint8), w, mask, [256 * 7, 256 * 8, 256 * 1025, d] if layers else None)
    assert not last["one_read"]


@pytest.mark.parametrize("law", ["heavy", "alike"])
def test_one_read_of_long_runs_by_the_rule(law):
    """A length that the rule takes: the sketch of the streaming driver, and, where the sample refuses it, the scale pass that
    depends on that, two blocks a wave."""
    import torch
    rng = np.random.default_rng(8)
    runs, k = CODES["one_row_shared"]
    csr, n, d = _runs(rng, runs), len(runs), (1 << 30) // 30 + 77
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    G = api.padded_rows(k, d)
    for j in range(k):
        G[j].normal_(generator=gen)
        if law == "heavy":
            G[j].pow_(7)
    last = _both_drivers(csr, k, G, np.full(n, 5, np.uint8), np.ones(n, np.float32), np.ones(n, np.uint8))
    assert last["one_read"] and last["bound_failed"] == (law == "alike")

"""Decode at the edges of its tiles and chunks: 256 * 8 or 256 * 16 coordinates per tile (one track and more
than 40 bits in all: from 5 * 2^20 coordinates on, 15 * 2^18 with bucket- and layer-wise scales), chunks of 48 or 24
stream units filled by whole workers, more tiles than resident workgroups, and a stream that ends inside a
unit; and without chunks (one or two workers, four from 2^25 coordinates on).  The streams are random bytes
(every bit pattern is a code); both tracks must equal the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

pytestmark = pytest.mark.gpu


def _check(n, d, bits, kind, two, seed, arrived=0.8):
    import torch
    rng = np.random.default_rng(seed)
    bits = np.asarray(bits, dtype=np.uint8)
    ctx = api.Context(n, n, d, allow_1bit=True, bucket=256 if kind == "bucket" else 0)
    per = 1
    if kind == "bucket":
        per = (d + 255) // 256
    elif kind == "layers":
        cut = max(256, d // 3 // 256 * 256)
        ends = np.array([e for e in (cut, 2 * cut) if e < d] + [d], dtype=np.int64)
        ctx.agc_set_layers(ends)
        per = len(ends)
    streams = [rng.integers(0, 256, api.agc_code_bytes(d, int(b)), dtype=np.uint8) for b in bits]
    scales = rng.uniform(0.5, 2.0, (n, per)).astype(np.float32)
    scales[0, 0] = 1e-41     # a weight that cannot be halved exactly
    w, v = rng.uniform(-2, 2, (2, n)).astype(np.float32)
    mask = (rng.random(n) < arrived).astype(np.uint8)
    mask[0] = 1
    codes = [torch.from_numpy(s).cuda() for s in streams]
    sc = torch.from_numpy(scales).cuda()
    got = [torch.full((d,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    if two:
        ctx.agc_decode2(codes, sc, bits, w, v, mask, got[0], got[1])
    else:
        ctx.agc_decode(codes, sc, bits, w, mask, got[0])
    torch.cuda.synchronize()
    for x, weights in zip(got[:1 + two], (w, v)):
        if kind == "bucket":
            want = O.decode_bucket(streams, scales, bits, weights, mask, d, 0, d)
        elif kind == "layers":
            want = O.decode_layers(streams, scales, bits, weights, mask, d, ends)
        else:
            want = O.decode(streams, scales[:, 0].copy(), bits, weights, mask, d, 0, d)
        assert np.array_equal(want.view(np.uint32), x.cpu().numpy().view(np.uint32)), (n, d, kind, two)
    ctx.close()


@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("kind", ["vector", "bucket", "layers"])
@pytest.mark.parametrize("d", [1, 127, 129, 2047, 2049, 4095, 4097, 40001])
def test_every_width_at_tile_edges(d, kind, two):
    _check(17, d, [2] + list(range(1, 17)), kind, two, d)


@pytest.mark.parametrize("kind", ["vector", "bucket"])
@pytest.mark.parametrize("d", [(1 << 21) - 1, 1 << 21, (1 << 21) + 129, 6_400_003])
def test_both_tilings_and_more_tiles_than_workgroups(d, kind):
    _check(5, d, [2, 3, 5, 7, 2], kind, False, d)


def test_two_tracks_with_more_tiles_than_workgroups():
    _check(3, 3_300_001, [2, 3, 6], "vector", True, 4)


@pytest.mark.parametrize("n,width", [(256, 16), (256, 2), (130, 9), (64, 12), (65, 7)])
def test_chunks_of_many_workers(n, width):
    _check(n, 3001, [width] * n, "vector", False, n + width)
    _check(n, 3001, [width] * n, "bucket", True, n + width)


@pytest.mark.parametrize("kind,two,d", [("vector", False, 3_300_001), ("vector", False, 6_400_003), ("bucket", False, 2_700_001),
                                        ("bucket", False, 5_400_001), ("layers", False, 2_700_001), ("layers", False, 5_400_001),
                                        ("vector", True, 3_300_001), ("bucket", True, 2_700_001), ("layers", True, 2_200_001)])
@pytest.mark.parametrize("chunks", [1, 2, 3])
def test_several_chunks_and_several_tiles_per_workgroup(kind, two, d, chunks):
    """An odd and an even number of chunks: the two buffers keep or change their parts from tile to tile.  Chunks
    of 24 units are filled exactly, those of 48 end in seven unused ones."""
    bits = [8, 7, 7] if chunks == 1 else ([11, 13] if not two and d > 5_000_000 else [16, 11, 12, 2]) * chunks
    _check(len(bits), d, bits, kind, two, d + chunks, arrived=1.0)


@pytest.mark.parametrize("kind,two,d", [("vector", False, 11_100_001), ("vector", True, 5_600_001), ("bucket", False, 9_300_001),
                                        ("layers", True, 3_700_001)])
def test_one_workgroup_per_tile(kind, two, d):
    """Four chunks and more to a tile, and at least 1.75 tiles to a resident workgroup."""
    _check(16, d, [12, 13] * 8, kind, two, d, arrived=1.0)


@pytest.mark.parametrize("line", [15 << 18, 5 << 20])
@pytest.mark.parametrize("kind", ["vector", "bucket", "layers"])
def test_both_sides_of_the_lines_between_the_tilings(kind, line):
    for d in (line - 1, line, line + 129):
        _check(6, d, [9, 8, 7, 2, 9, 8], kind, False, d, arrived=1.0)
    _check(6, line, [9, 8, 7, 2, 9, 5], kind, False, line, arrived=1.0)   # 40 bits


@pytest.mark.parametrize("kind", ["vector", "bucket", "layers"])
@pytest.mark.parametrize("d", [1, 31, 32, 33, 255, 257, 8191, 8193, 40001])
def test_a_few_workers_without_chunks(kind, d):
    for b in range(1, 17):
        _check(2, d, [b, 17 - b], kind, False, 100 * d + b, arrived=1.0)
        _check(1, d, [b], kind, False, 100 * d + b, arrived=1.0)


@pytest.mark.parametrize("kind", ["vector", "layers"])
def test_four_workers_on_a_very_long_vector_without_chunks(kind):
    for d in ((1 << 25) - 1, (1 << 25) + 5):
        _check(4, d, [2, 1, 5, 3], kind, False, d, arrived=1.0)


@pytest.mark.parametrize("n", [65, 256])
def test_decode_of_many_workers_recorded_in_a_hip_graph(n):
    """More than 64 workers: the arguments of the prologue are larger than 4 KB.  Every replay, with eager
    decodes of another arrival pattern between them, gives the eager result; likewise without a context."""
    import torch
    rng = np.random.default_rng(n)
    d = 70_001
    bits = rng.integers(1, 9, n).astype(np.uint8)
    ctx = api.Context(n, n, d, allow_1bit=True)
    codes = [torch.from_numpy(rng.integers(0, 256, api.agc_code_bytes(d, int(b)), dtype=np.uint8)).cuda() for b in bits]
    scales = torch.from_numpy(rng.uniform(0.5, 2.0, n).astype(np.float32)).cuda()
    w, v = rng.uniform(-2, 2, (2, n)).astype(np.float32)
    everyone, some = np.ones(n, np.uint8), (rng.random(n) < 0.5).astype(np.uint8)
    out = [torch.empty(d, dtype=torch.float32, device="cuda") for _ in range(3)]

    def decode(mask):
        ctx.agc_decode2(codes, scales, bits, w, v, mask, out[0], out[1])
        api.agc_decode_noalloc(n, d, 0, codes, scales, bits, w, mask, out[2])

    decode(everyone)
    torch.cuda.synchronize()
    want = [t.clone() for t in out]
    streams = [c.cpu().numpy() for c in codes]
    ref = O.decode(streams, scales.cpu().numpy(), bits, w, everyone, d, 0, d)
    assert np.array_equal(ref.view(np.uint32), want[0].cpu().numpy().view(np.uint32))
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        decode(everyone)
    for replay in range(3):
        decode(some)
        torch.cuda.synchronize()
        for t in out:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, expected in zip(out, want):
            assert torch.equal(got.view(torch.int32), expected.view(torch.int32)), replay
    del graph
    ctx.close()

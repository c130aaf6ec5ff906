"""Decode at the edges of its tiles and chunks: 256 * 8 or 256 * 16 coordinates per tile (one track from
2^21 coordinates on), chunks of 48 or 24 stream units filled by whole workers, more
tiles than resident workgroups, and a stream that ends inside a unit.  The streams are random bytes (every
bit pattern is a code); both tracks must equal the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

pytestmark = pytest.mark.gpu


def _check(n, d, bits, kind, two, seed):
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
    mask = (rng.random(n) < 0.8).astype(np.uint8)
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

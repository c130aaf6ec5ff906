"""Short vectors, where the waves of a workgroup share the workers of one block, on both sides of the lines to
the long form (four blocks per workgroup, every wave walks over all workers): all drivers, scale kinds, ragged
last blocks and segments, fused and two-pass steps, and widths that sum to more than the one fill of a short
vector's staging area holds (1024 bits; the scale pass is then still shared, the quantize pass is not).  Codes,
scales and estimates equal the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr, to_device
from test_gpu_random_shapes import _case

pytestmark = pytest.mark.gpu

LINE = 1024 * 256


def _step(c):
    import torch
    n, k, d = c["n"], c["k"], c["d"]
    ctx = api.Context(n, k, d, scale_mode=c["scale_mode"], allow_1bit=True, bucket=c["bucket"], unfused_step=c["unfused"])
    ctx.agc_set_code(*c["code"])
    codes, scales, ghat = ctx.alloc_outputs(c["bits"])
    for t in codes:
        t.fill_(0x5A)
    ghat.fill_(float("nan"))
    G = to_device(c["G"])
    for _ in range(2):   # the second pass finds what the first left behind
        ctx.agc_step(G, c["bits"], c["w"], c["mask"], c["seed"], c["step"], codes, scales, ghat)
    torch.cuda.synchronize()
    step = O.step_bucket if c["bucket"] else O.step
    o_streams, o_scales, o_ghat = step(c["G"], O.Csr(*c["code"], k), c["bits"], c["w"], c["mask"], c["seed"], c["step"],
                                       c["scale_mode"])
    tag = {kk: vv for kk, vv in c.items() if kk not in ("G", "code")}
    assert np.array_equal(scales.cpu().numpy().view(np.uint32), o_scales.view(np.uint32)), tag
    for i in range(n):
        assert np.array_equal(codes[i].cpu().numpy(), o_streams[i]), (tag, i)
    assert np.array_equal(ghat.cpu().numpy().view(np.uint32), o_ghat.view(np.uint32)), tag
    ctx.close()


@pytest.mark.parametrize("d", [LINE - 3, LINE, LINE + 1, LINE + 1285])
@pytest.mark.parametrize("seed", range(12))
def test_both_sides_of_the_line(seed, d):
    c = _case(7000 + seed)
    rng = np.random.default_rng(seed)
    c["d"] = d
    c["G"] = (rng.standard_normal((c["k"], d)) * 1e-2).astype(np.float32)
    _step(c)


@pytest.mark.parametrize("code,blocks", [("cyclic", 2048), ("general", 3072)])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_the_lines_of_sixteen_workers(code, blocks, over):
    """Vectors that end inside a block: a band up to 2048 blocks, and partitions with four holders up to 3072."""
    rng = np.random.default_rng(blocks + over)
    n = k = 17
    if code == "cyclic":
        csr = cyclic_csr(rng, n, 4)
    else:
        csr = (np.arange(n + 1, dtype=np.int32) * 5, np.concatenate([rng.choice(k, 5, replace=False) for _ in range(n)]).astype(np.int32),
               rng.standard_normal(5 * n).astype(np.float32))
    d = 256 * blocks - 2 + 3 * over
    for scale_mode, bucket in ((0, 0), (1, 0), (1, 256)):
        _step(dict(n=n, k=k, d=d, code=csr, bits=rng.integers(1, 9, n).astype(np.uint8),
                   w=rng.uniform(0.2, 3.0, n).astype(np.float32), mask=(rng.random(n) < 0.7).astype(np.uint8),
                   G=rng.standard_normal((k, d)).astype(np.float32), scale_mode=scale_mode, bucket=bucket,
                   unfused=False, seed=5, step=3))


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 9, 63, 64, 65, 255, 256])
@pytest.mark.parametrize("code", ["cyclic", "interval", "general"])
def test_every_split_of_the_workers(code, n):
    """The last parts of the workers are short or empty.  255 and 256 workers at up to 4 bits stay below 1024 bits;
    at up to 16 they need more than one fill and the quantize pass keeps the long form's kernels."""
    rng = np.random.default_rng(n)
    k = n if code == "cyclic" else max(1, n // 2 + 3)
    csr = (cyclic_csr(rng, n, min(n, 5)) if code == "cyclic"
           else monotone_csr(rng, n, k, 4) if code == "interval" else random_csr(rng, n, k, 4))
    for scale_mode, bucket, unfused, most in ((0, 0, False, 4), (1, 0, True, 4), (1, 256, False, 16), (0, 256, False, 16),
                                              (0, 0, True, 16), (1, 0, False, 16)):
        if n < 255 and most == 4:
            most = 16
        d = int(rng.choice([1, 255, 700, 1025, 2000]))
        _step(dict(n=n, k=k, d=d, code=csr, bits=rng.integers(1, most + 1, n).astype(np.uint8),
                   w=rng.uniform(0.2, 3.0, n).astype(np.float32), mask=(rng.random(n) < 0.7).astype(np.uint8),
                   G=rng.standard_normal((k, d)).astype(np.float32), scale_mode=scale_mode, bucket=bucket,
                   unfused=unfused, seed=int(rng.integers(0, 2 ** 62)), step=3))

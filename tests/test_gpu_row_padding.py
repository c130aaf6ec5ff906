"""What lies behind the end of G's rows (the rest of the last float4, the padding up to the row stride) counts
nowhere: the block that the vector ends in reads it with the other lanes and drops it.  NaN, infinities and the largest
finite values there, every driver, both forms of the two passes, all kinds of scale; results equal the oracle's bit for bit,
which never sees the padding."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 255, 257, 1021, 1026, 2303])
@pytest.mark.parametrize("kind", ["cyclic", "interval", "general"])
@pytest.mark.parametrize("long_form", [False, True])
def test_padding_counts_nowhere(kind, d, long_form):
    import torch
    rng = np.random.default_rng([d, len(kind)])
    n = k = 11
    csr = (cyclic_csr(rng, n, 4) if kind == "cyclic" else monotone_csr(rng, n, k, 4) if kind == "interval"
           else random_csr(rng, n, k, 4, allow_empty=False))
    G_host = rng.standard_normal((k, d)).astype(np.float32)
    stride = (d + 3) // 4 * 4 + 8
    buf = torch.empty((k, stride), dtype=torch.float32, device="cuda")
    bits = rng.integers(1, 13, n).astype(np.uint8)
    w = rng.uniform(0.2, 3.0, n).astype(np.float32)
    mask = (rng.random(n) < 0.7).astype(np.uint8)
    for scale_mode, bucket in ((0, 0), (1, 0), (0, 256), (1, 256)):
        step = O.step_bucket if bucket else O.step
        o_streams, o_scales, o_ghat = step(G_host, O.Csr(*csr, k), bits, w, mask, 11, 4, scale_mode)
        for filler in (float("nan"), float("inf"), -3.4e38):
            buf.fill_(filler)
            buf[:, :d].copy_(torch.from_numpy(G_host))
            ctx = api.Context(n, k, d, scale_mode=scale_mode, allow_1bit=True, bucket=bucket)
            ctx.agc_set_code(*csr)
            ctx.agc_debug_force_long(long_form)
            codes, scales, ghat = ctx.alloc_outputs(bits)
            ctx.agc_step(buf[:, :d], bits, w, mask, 11, 4, codes, scales, ghat)
            torch.cuda.synchronize()
            tag = (scale_mode, bucket, filler)
            assert np.array_equal(scales.cpu().numpy().view(np.uint32), o_scales.view(np.uint32)), tag
            for i in range(n):
                assert np.array_equal(codes[i].cpu().numpy(), o_streams[i]), (tag, i)
            assert np.array_equal(ghat.cpu().numpy().view(np.uint32), o_ghat.view(np.uint32)), tag
            ctx.close()

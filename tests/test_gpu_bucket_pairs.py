"""Bucket-wise scales are found for two workers at a time where the driver knows a worker's parity (cyclic band, general
codes), and for one at a time in the windows: even and odd numbers of workers, runs of workers of every length among the
waves of short vectors, one-bit workers and several fills of the staging area between the two of a pair, blocks and groups
that end inside the vector.  Bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr
from test_gpu_short_vectors import _step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 7, 16, 33, 64, 129])
@pytest.mark.parametrize("kind", ["cyclic", "interval", "general"])
@pytest.mark.parametrize("long_form", [False, True])
def test_pairs_of_workers(kind, n, long_form, monkeypatch):
    if long_form:
        create = api.Context.__init__

        def create_long(self, *args, **kwargs):
            create(self, *args, **kwargs)
            self.agc_debug_force_long(True)

        monkeypatch.setattr(api.Context, "__init__", create_long)
    rng = np.random.default_rng([n, len(kind)])
    k = n if kind == "cyclic" else n + 2
    csr = (cyclic_csr(rng, n, min(n, 3)) if kind == "cyclic" else monotone_csr(rng, n, k, 4) if kind == "interval"
           else random_csr(rng, n, k, 4))
    for scale_mode in (api.AGC_SCALE_L2, api.AGC_SCALE_MAXABS):
        for most, d in ((4, 1024), (16, 1500)):
            G = rng.standard_normal((k, d)).astype(np.float32)
            G[:, 256:512] = 0.0   # a bucket whose scale is 0
            _step(dict(n=n, k=k, d=d, code=csr, bits=rng.integers(1, most + 1, n).astype(np.uint8),
                       w=rng.uniform(0.2, 3.0, n).astype(np.float32), mask=(rng.random(n) < 0.7).astype(np.uint8), G=G,
                       scale_mode=scale_mode, bucket=256, unfused=False, seed=13, step=6))

"""The kernels of long vectors at small sizes.  Short vectors take kernels of their own, so the suites that walk
over every driver, band width, ragged length, option and layer boundary are run here once more with the
testing hook that keeps a context on the long form (agc_debug_force_long); what they compare with the
oracle stays as it is in their own files."""
import numpy as np
import pytest

from oracle import agc_oracle as O
from paper_2605_15890_amd import api

from gpu_util import cyclic_csr, monotone_csr, random_csr
from test_gpu_bucket import test_generic_code_and_wide_band, test_ragged_sizes  # noqa: F401
from test_gpu_layers import (test_layerwise_decode_and_two_track_decode_match_oracle,  # noqa: F401
                             test_layerwise_euclidean_step_matches_oracle,
                             test_layerwise_scales_with_the_maximum_number_of_layers_and_workers,
                             test_layerwise_step_matches_oracle)
from test_gpu_parity import (test_degenerate_inputs, test_every_band_width,  # noqa: F401
                             test_fused_step_equals_two_pass_step, test_general_codes, test_maximum_worker_count,
                             test_monotone_interval_codes_take_the_window_path, test_ragged_sizes_cyclic_and_generic,
                             test_step_recorded_in_a_hip_graph_replays_the_eager_result)
from test_gpu_random_shapes import test_random_case  # noqa: F401
from test_gpu_short_vectors import _step

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def long_form(monkeypatch):
    create = api.Context.__init__

    def create_long(self, *args, **kwargs):
        create(self, *args, **kwargs)
        self.agc_debug_force_long(True)

    monkeypatch.setattr(api.Context, "__init__", create_long)


@pytest.mark.parametrize("kind", ["cyclic", "interval", "general"])
@pytest.mark.parametrize("most", [8, 16])
def test_the_block_that_the_vector_ends_in_starts_early(kind, most):
    """More groups of blocks than the chip holds at once and a ragged end: the workgroups start 64 groups before
    the end and wrap around, with one fill of the staging area (24 workers of up to 8 bits) and with two."""
    rng = np.random.default_rng(most)
    n, k, d = 24, 24, 1024 * 1024 + 77
    csr = cyclic_csr(rng, n, 5) if kind == "cyclic" else monotone_csr(rng, n, k, 6) if kind == "interval" else random_csr(rng, n, k, 4)
    bits = rng.integers(most - 1, most + 1, n).astype(np.uint8)
    assert (int(bits.sum()) > 319) == (most == 16)
    for scale_mode in (api.AGC_SCALE_L2, api.AGC_SCALE_MAXABS):
        _step(dict(n=n, k=k, d=d, code=csr, bits=bits, w=rng.uniform(0.2, 3.0, n).astype(np.float32),
                   mask=(rng.random(n) < 0.7).astype(np.uint8), G=rng.standard_normal((k, d)).astype(np.float32),
                   scale_mode=scale_mode, bucket=0, unfused=False, seed=7, step=2))

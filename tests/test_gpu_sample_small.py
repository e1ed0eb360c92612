"""Bitstrings of states of one chunk (up to 2^12 amplitudes), where the sampler reads the chunk as it is up to
2^11 and through LDS above: every size, states with most of their mass missing, and the last index."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import assert_valid_samples, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", range(1, 14))
def test_against_the_definition(n, prec):
    rng = np.random.default_rng(40 + n)
    ctx = rsv.rsv_ctx_create(0)
    dim, shots = 1 << n, 3000
    sparse = np.zeros(dim, dtype=complex)
    sparse[rng.choice(dim, min(dim, 5), replace=False)] = rng.normal(size=min(dim, 5)) + 0.2
    last = np.zeros(dim, dtype=complex)
    last[-1] = 1.0
    for k, psi in enumerate((wl.random_state(n, rng), 3.0 * sparse, last)):
        d = to_dev(psi, prec)
        got = rsv.rsv_sample_device(ctx, n, d, 100 + k, shots, prec)
        assert_valid_samples(got, to_host(d), 100 + k, shots - 2)
        if k == 2:
            assert (np.asarray(got) == dim - 1).all()
    rsv.rsv_ctx_destroy(ctx)

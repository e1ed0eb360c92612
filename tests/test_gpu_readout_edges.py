"""Outputs of a device state where the kernels change shape: around one chunk of 2^12 (and, for
the correlators from 20 atoms, 2^14) amplitudes, and where the sampler's search takes one, two
and three rounds.  Oracle: FP64 numpy sums of |psi|^2.  Every value is a sum of at most 2^14
thread-local and 2^10 second-stage terms added in chains of fewer than 300, so it lies within
600 eps of the total of the reference (whose pairwise sums are closer than that)."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import assert_valid_samples, to_dev

pytestmark = pytest.mark.gpu
BOUND = 600 * np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    c = rsv.rsv_ctx_create(0)
    yield c
    rsv.rsv_ctx_destroy(c)


def bit_sums(p, n):
    """<n_i n_j> numerators by the halves of the index."""
    a = n // 2
    m = p.reshape(1 << a, -1)
    bh = ((np.arange(1 << a)[:, None] >> (a - 1 - np.arange(a))) & 1).astype(float)
    bl = ((np.arange(1 << (n - a))[:, None] >> (n - a - 1 - np.arange(n - a))) & 1).astype(float)
    hl = bh.T @ m @ bl
    return np.block([[bh.T @ (m.sum(1)[:, None] * bh), hl], [hl.T, bl.T @ (m.sum(0)[:, None] * bl)]])


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", [7, 8, 11, 12, 13, 14, 19, 20, 21, 23])
def test_sums_and_samples(ctx, n, prec):
    psi = wl.random_state(n, np.random.default_rng(n))
    psi[: 1 << (n - 2)] = 0  # whole chunks without mass
    d = to_dev(psi, prec)
    held = d.cpu().numpy().astype(np.complex128)
    p = held.real ** 2 + held.imag ** 2
    tot = p.sum()
    want = bit_sums(p, n) / tot
    np.testing.assert_allclose(rsv.rsv_correlations_device(ctx, n, d, prec), want, rtol=0, atol=BOUND)
    np.testing.assert_allclose(rsv.rsv_occupations_device(ctx, n, d, prec), np.diag(want), rtol=0,
                               atol=BOUND)
    shots = 400
    got = rsv.rsv_sample_device(ctx, n, d, 17, shots, prec)
    assert_valid_samples(got, held, 17, shots - 2)


def test_sampler_on_one_basis_state_in_the_last_block(ctx):
    for n in (12, 21, 22):  # 1, 512 and 1024 blocks
        psi = np.zeros(1 << n, dtype=np.complex128)
        psi[-1] = 1.0
        got = rsv.rsv_sample_device(ctx, n, to_dev(psi, "c128"), 3, 64)
        assert np.all(got == (1 << n) - 1)

"""Density matrices whose sums of squares say nothing about their symmetry take the general Arnoldi
process: infinite elements (the call fails and leaves the matrix as it was), and matrices so small
that the squared difference from their adjoint underflows."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
N = 10


@pytest.fixture(scope="module")
def handles():
    ctx = rsv.rsv_ctx_create(0)
    reg = {p: rsv.rsv_register_create(ctx, wl.chain(N, 6.0), wl.C6_RB, p) for p in ("c128", "c64")}
    om, de, _ = wl.sweep_pulses(50, 100, 9.0, 9.0)
    yield reg, rsv.PulseArrays(om, de)
    for r in reg.values():
        rsv.rsv_register_destroy(r)
    rsv.rsv_ctx_destroy(ctx)


def matrix(rng):
    a = rng.normal(size=(1 << N, 1 << N)) + 1j * rng.normal(size=(1 << N, 1 << N))
    return a / np.linalg.norm(a)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_an_infinite_element_leaves_the_matrix_alone(handles, prec):
    reg, pulses = handles
    rho = matrix(np.random.default_rng(1))
    rho[3, 700] = np.inf
    d = to_dev(rho.reshape(-1), prec)
    before = d.clone()
    with pytest.raises(rsv.RsvError) as e:
        rsv.rsv_lindblad_evolve_device(reg[prec], pulses, rsv.evolve_opts(10, 1e-6, 20, n_steps=1), (0.5, 0.5), d)
    assert e.value.code == rsv.RSV_ENUMERIC
    assert np.array_equal(to_host(d), to_host(before), equal_nan=True)


def test_a_tiny_matrix_keeps_its_skew_part(handles):
    """A skew-Hermitian part of 1e-9 at a scale of 2^-506 (5e-153), where its squares vanish: the
    result is that of the unscaled matrix up to the tolerance, 1e-12 of the norm in both (the squares
    of the elements, about 2e-311, keep 12 digits each and their sum more)."""
    reg, pulses = handles
    a = matrix(np.random.default_rng(2))
    rho = (a + a.conj().T) / 2 + 1e-9 * (a - a.conj().T) / 2
    scale = 2.0 ** -506

    def evolved(x, tol):
        d = to_dev(x.reshape(-1), "c128")
        rsv.rsv_lindblad_evolve_device(reg["c128"], pulses, rsv.evolve_opts(10, tol, 40, n_steps=1), (0.5, 0.5), d)
        return to_host(d)

    want = evolved(rho, 1e-12)
    got = evolved(rho * scale, 1e-12 * scale) / scale
    assert np.linalg.norm(got - want) <= 2e-12

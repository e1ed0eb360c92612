"""The iterations that Arnoldi exponentials queue against those their steps need, where vectors need second
Gram-Schmidt passes: what is queued behind such a vector is computed again, so after the first step
the queue ends with it.  Strong dissipation (every vector), the gradients' block operator (the
second one), and sub-steps.  And a window of steps against one call per step, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = rsv.rsv_ctx_create(0)
    yield c
    rsv.rsv_ctx_destroy(c)


def sweep(n):
    w = wl.random27(0, n, "c128")
    return w.xyz, rsv.PulseArrays(w.omega, w.delta)


@pytest.mark.parametrize("n,rates", [(4, (30.0, 60.0)), (8, (50.0, 50.0)), (10, (50.0, 50.0)), (10, (0.5, 1.0))])
def test_lindblad_windows(ctx, n, rates):
    first, steps = 100, 5
    xyz, pulses = sweep(n)
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, "c128")
    psi = torch.from_numpy(wl.random_state(n, np.random.default_rng(n))).cuda()
    a = torch.outer(psi, psi.conj()).reshape(-1).contiguous()
    b = a.clone()

    def evolve(x, k, count):
        return rsv.rsv_lindblad_evolve_device(reg, pulses, rsv.evolve_opts(10, 1e-9, 48, 12, k, count), rates, x)

    dims = [int(evolve(a, first + k, 1).krylov_max) for k in range(steps)]
    st = evolve(b, first, steps)
    assert st.substeps == 0 and st.krylov_max == max(dims)
    # the first step knows nothing; after it, at most one more than needed per step
    assert sum(dims) <= st.krylov_iters <= sum(dims) + dims[0] + steps - 1
    assert np.array_equal(to_host(a), to_host(b))
    rsv.rsv_register_destroy(reg)


@pytest.mark.parametrize("n,kmax", [(16, 48), (18, 40), (16, 20)])
def test_gradient_windows(ctx, n, kmax):
    """A step's five exponentials (forward, recomputed, adjoint, two of the block operator) take at most
    krylov_max iterations for each of their parts, and one more where the dimension falls."""
    xyz, pulses = sweep(n)
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, "c128")
    psi0 = wl.random_state(n, np.random.default_rng(n))
    weights = np.random.default_rng(1).uniform(-1, 1, n)

    def stats(steps):
        return rsv.rsv_gradient_occupations(reg, pulses, rsv.evolve_opts(10, 1e-9, kmax, 12, 100, steps), weights, psi0)[3]

    short, long = stats(2), stats(5)
    parts = 3 * 5 + long.substeps - short.substeps
    assert long.krylov_iters - short.krylov_iters <= parts * (long.krylov_max + 1)
    assert (long.substeps > 0) == (kmax == 20)
    rsv.rsv_register_destroy(reg)

"""Which route a small register's call takes, by what only one of them does.  Three atoms 1.9 um apart (U =
1.15e5 rad/us): a step's exponential is far beyond the device's series, which would have to sub-step;
the host driver's eigenvectors resolve it in the eight dimensions there are."""
import numpy as np
import pytest

from oracle import evolve, observables
from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def test_a_wide_spectrum_takes_the_host_driver():
    n, steps, dt = 3, 2, 10
    t = np.arange(steps * dt + 1)
    w = wl.Workload("wide", wl.chain(n, 1.9), wl.C6_RB, 9.0 + 0.1 * t, -6.0 + 0.2 * t, None, steps * dt, dt,
                    tol=1e-9, kmax=20)
    psi0 = wl.random_state(n, np.random.default_rng(3))
    ctx = rsv.rsv_ctx_create(0)
    reg = rsv.rsv_register_create(ctx, w.xyz, w.c6, "c128")
    d = to_dev(psi0, "c128")
    st = rsv.rsv_evolve_device(reg, rsv.PulseArrays(w.omega, w.delta), rsv.evolve_opts(dt, w.tol, w.kmax), d)
    assert st.substeps == 0 and st.krylov_max <= w.kmax
    ref = evolve.evolve_workload(w, psi0=psi0, method="dense")
    assert observables.fidelity_loss(ref, to_host(d)) <= 1e-10
    rsv.rsv_register_destroy(reg)
    rsv.rsv_ctx_destroy(ctx)

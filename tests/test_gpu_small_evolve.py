"""Registers of one workgroup, evolved on the device in one call: every thread layout (one wave
to 1024 threads, one to eight amplitudes each), both drives, launches that continue each other,
recorded occupations, and the register too strongly interacting for the device's series, which
takes the host driver.  Oracle: exponentials per step; the bars are the workload specification's
(infidelity 1e-10 / 1e-6; occupations 1e-8 / 1e-5, the square root of what an infidelity at the
bar allows is larger still)."""
import numpy as np
import pytest

from oracle import evolve, observables
from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
INFID = {"c128": 1e-10, "c64": 1e-6}
OCC = {"c128": 1e-8, "c64": 1e-5}


@pytest.fixture(scope="module")
def ctx():
    c = rsv.rsv_ctx_create(0)
    yield c
    rsv.rsv_ctx_destroy(c)


def workload(n, site, steps, prec, dt=10):
    rng = np.random.default_rng(100 + n)
    t = steps * dt
    s = np.arange(t + 1) / max(t, 1)
    om, de, ph = 9.0 * np.sin(np.pi * (0.1 + 0.8 * s)), -6.0 + 14.0 * s, None
    if site:
        om, de = np.outer(rng.uniform(0.5, 1.5, n), om), np.outer(rng.uniform(0.5, 1.5, n), de)
        ph = np.outer(rng.uniform(-1, 1, n), s + 0.3)
    return wl.Workload(f"small{n}", wl.random_register(n, 22.0, 4.5, rng), wl.C6_RB, om, de, ph, t,
                       dt, tol=1e-10 if prec == "c128" else 1e-7, kmax=40, precision=prec)


def run(ctx, w, prec, psi, first=0, steps=-1, every=0):
    reg = rsv.rsv_register_create(ctx, w.xyz, w.c6, prec)
    pulses = rsv.PulseArrays(w.omega, w.delta, w.phi)
    opts = rsv.evolve_opts(w.dt_ns, w.tol, w.kmax, 12, first, steps)
    d = to_dev(psi, prec)
    if every:
        st, occ = rsv.rsv_evolve_device_observed(reg, pulses, opts, d, every)
    else:
        st, occ = rsv.rsv_evolve_device(reg, pulses, opts, d), None
    rsv.rsv_register_destroy(reg)
    return to_host(d), occ, st.as_dict()


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,site,steps", [(1, False, 5), (2, True, 90), (5, False, 225), (6, True, 12),
                                          (7, False, 9), (8, True, 20), (9, False, 12), (10, True, 16),
                                          (11, True, 14), (12, False, 4), (12, True, 13), (13, True, 12)])
def test_against_the_oracle(ctx, prec, n, site, steps):
    w = workload(n, site, steps, prec, dt=5 if steps > 100 else 10)
    psi0 = wl.random_state(n, np.random.default_rng(n)) * 1.5  # any norm is carried
    every = max(1, steps // 3)
    psi, occ, st = run(ctx, w, prec, psi0, every=every)
    method = "dense" if n <= 8 else "lanczos"
    ref, rows = psi0.copy(), []
    for k in range(steps):
        ref = evolve.evolve_workload(w, steps=1, first_step=k, psi0=ref, method=method)
        if (k + 1) % every == 0:
            rows.append(observables.occupations(ref))
    assert observables.fidelity_loss(ref, psi) <= INFID[prec]
    assert abs(st["norm_final"] - 1.5) <= (1e-10 if prec == "c128" else 1e-5)
    np.testing.assert_allclose(occ, np.array(rows), rtol=0, atol=OCC[prec])
    assert st["steps"] == steps and st["krylov_iters"] >= steps and st["krylov_max"] <= w.kmax
    # split at a step boundary: the same state bit for bit, and without recording
    cut = steps // 2
    if cut:
        a, _, _ = run(ctx, w, prec, psi0, steps=cut)
        b, _, _ = run(ctx, w, prec, a, first=cut)
        assert np.array_equal(b, psi)


def test_strong_interactions_take_the_host_driver(ctx):
    """Six atoms 1.9 um apart: tau times the spectrum's bound is far beyond the device's series."""
    w = workload(6, False, 2, "c128")
    w.xyz = wl.chain(6, 1.9)
    psi0 = wl.random_state(6, np.random.default_rng(3))
    psi, _, st = run(ctx, w, "c128", psi0)
    ref = evolve.evolve_workload(w, psi0=psi0, method="dense")
    assert observables.fidelity_loss(ref, psi) <= 1e-10


def test_failures_leave_the_state_alone(ctx):
    w = workload(9, False, 30, "c128")
    psi0 = wl.random_state(9, np.random.default_rng(3))
    for bad, code in ((np.zeros_like(psi0), rsv.RSV_ENUMERIC), (np.full_like(psi0, np.nan), rsv.RSV_ENUMERIC)):
        with pytest.raises(rsv.RsvError) as e:
            run(ctx, w, "c128", bad)
        assert e.value.code == code
    reg = rsv.rsv_register_create(ctx, w.xyz, w.c6, "c128")
    d = to_dev(psi0, "c128")
    with pytest.raises(rsv.RsvError) as e:
        rsv.rsv_evolve_device(reg, rsv.PulseArrays(w.omega, w.delta), rsv.evolve_opts(10, 1e-10, 3, 0), d)
    assert e.value.code == rsv.RSV_ENOTCONV
    assert np.array_equal(to_host(d), psi0)
    rsv.rsv_register_destroy(reg)

"""Full re-orthogonalisation where the inner products' grid changes (2^9 amplitudes, 1024 workgroups from
2^18 to 2^21, 2048 from 2^22 on): one step with it against one without.  Each is within the
tolerance of the exact step; complex64 adds its storage rounding over about 30 vectors."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", [1, 9, 17, 18, 19, 21, 22])
def test_one_step_with_and_without(n, prec):
    rng = np.random.default_rng(n)
    om, de, _ = wl.sweep_pulses(50, 100, 12.0, 9.0)
    tol = 1e-10 if prec == "c128" else 1e-6
    ctx = rsv.rsv_ctx_create(0)
    reg = rsv.rsv_register_create(ctx, wl.random_register(n, 32.0, 5.0, rng), wl.C6_RB, prec)
    pulses = rsv.PulseArrays(om, de)
    psi0 = np.zeros(1 << n, dtype=complex)
    psi0[: min(1 << n, 64)] = wl.random_state(min(n, 6), rng)
    out = []
    for reorth in (0, 1):
        d = to_dev(psi0, prec)
        rsv.rsv_evolve_device(reg, pulses, rsv.evolve_opts(5, tol, 60, 12, 10, 1, reorth), d)
        out.append(to_host(d))
    assert np.linalg.norm(out[0] - out[1]) <= 2 * tol + (30 * 6e-8 if prec == "c64" else 1e-13)
    rsv.rsv_register_destroy(reg)
    rsv.rsv_ctx_destroy(ctx)

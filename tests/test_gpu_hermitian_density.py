"""Hermitian density matrices of 10 atoms and more, whose Arnoldi process reads one triangle: against
the general process on i times the same matrix (the Liouvillian is linear, and i rho is not
Hermitian), and the tiled Liouvillian at its smallest sizes with both forms of the drive."""
import numpy as np
import pytest

from oracle import lindblad, model
from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.test_gpu_lindblad import ctx, dev, host, pulses, random_rho  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,per_site,rates", [(9, False, (0.8, 0.3)), (10, False, (0.8, 0.3)),
                                              (10, True, (0.0, 0.6)), (11, True, (0.7, 0.0))])
def test_evolution_equals_the_general_process(ctx, n, per_site, rates, prec):  # noqa: F811
    rng = np.random.default_rng(200 + n)
    xyz = wl.random_register(n, 18.0, 4.5, rng)
    om, de, ph = pulses(n, 100, rng, per_site)
    rho = random_rho(n, rng)  # a a^+ from a library product: Hermitian up to rounding
    tol = 1e-11 if prec == "c128" else 1e-7
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, prec)
    pl = rsv.PulseArrays(om, de, ph)

    def run(start, *ranges):
        x = dev(start, prec)
        for first, steps in ranges:
            rsv.rsv_lindblad_evolve_device(reg, pl, rsv.evolve_opts(10, tol, 40, 12, first, steps), rates, x)
        return host(x, n)

    got = run(rho, (2, 3))
    general = run(1j * rho, (2, 3)) / 1j
    split = run(rho, (2, 1), (3, 2))
    rsv.rsv_register_destroy(reg)
    # each of the two runs is within tol |rho| a step; complex64 adds its rounding, 3 steps of
    # about 25 vectors at 6e-8 each
    bound = 2 * 3 * tol * 10 + (3 * 25 * 6e-8 if prec == "c64" else 1e-13)
    assert np.linalg.norm(got - general) <= bound * np.linalg.norm(rho)
    if n >= 10:
        assert np.array_equal(got, got.conj().T)
    assert np.array_equal(got, split)


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,per_site", [(10, False), (10, True), (11, False), (13, False)])
def test_tiled_liouvillian(ctx, n, per_site, prec):  # noqa: F811
    import torch
    rng = np.random.default_rng(300 + n)
    xyz = wl.random_register(n, 20.0, 4.0, rng)
    om, de, ph = pulses(n, 100, rng, per_site)
    d, rates = 1 << n, (0.9, 0.35)
    g = torch.Generator(device="cuda:0").manual_seed(n)
    x = torch.randn(d * d, dtype=torch.complex128 if prec == "c128" else torch.complex64,
                    device="cuda:0", generator=g)
    y = torch.empty_like(x)
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, prec)
    rsv.rsv_lindblad_apply(reg, rsv.PulseArrays(om, de, ph), 4, 10, rates, x, y)
    rho, out = host(x, n), host(y, n)
    rsv.rsv_register_destroy(reg)
    u = model.interaction_matrix(xyz, wl.C6_RB)
    pars = model.step_parameters(n, om, de, ph, 10, 4)
    pts = [(0, 0), (d - 1, d - 1), (0, d - 1), (d - 1, 0), (31, 32), (32, 31), (63, 0)]
    pts += [(int(a), int(b)) for a, b in rng.integers(0, d, (150, 2))]
    # 2 n + 2 terms, each rounded at the size of the largest diagonal entry times |rho|
    largest = np.abs(np.triu(u, 1)).sum() + n * 30.0
    eps = 2.3e-16 if prec == "c128" else 1.2e-7
    for r, c in pts:
        want = lindblad.liouvillian_element(r, c, rho, u, *pars, *rates)
        scale = np.abs(rho[r, :]).max() + np.abs(rho[:, c]).max()
        assert abs(out[r, c] - want) <= (2 * n + 2) * 4 * eps * largest * scale, (r, c, out[r, c], want)

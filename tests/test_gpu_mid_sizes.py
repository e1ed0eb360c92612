"""Sizes between one workgroup's registers and those that fill the chip with full tiles: the plans
of small tiles (13 to 20 atoms), iterations with and without sums in the forming pass, and the
gradients' block operator on both sides of its largest register."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.test_gpu_gradient import ctx, gpu_grad  # noqa: F401

pytestmark = pytest.mark.gpu


def taylor_steps(reg, pl, psi, first, steps, dt, parts):
    """exp(-i H_k dt) psi by the Taylor series of `parts` equal sub-steps, on H psi in complex128."""
    import torch
    h = torch.empty_like(psi)
    tau = dt * 1e-3 / parts
    for k in range(first, first + steps):
        for _ in range(parts):
            term, out = psi.clone(), psi.clone()
            for i in range(1, 60):
                rsv.rsv_apply_hamiltonian(reg, pl, k, dt, term, h)
                term = h * (-1j * tau / i)
                out += term
                if float(term.norm()) < 1e-17:
                    break
            psi = out
    return psi


@pytest.mark.parametrize("drive", ["global", "phase", "site"])
@pytest.mark.parametrize("n", [13, 14, 15, 16, 17, 18, 19, 20, 21, 23])
def test_evolution_against_taylor_series(ctx, n, drive):  # noqa: F811
    import torch
    rng = np.random.default_rng(500 + n)
    t_ns, dt, steps = 100, 10, 2
    xyz = wl.random_register(n, 12.0 * np.sqrt(n), 6.0, rng)
    om, de = wl.pwl([0, 50, 100], [3, 12, 4], t_ns), wl.pwl([0, 100], [-9, 7], t_ns)
    ph = None if drive == "global" else np.linspace(-0.5, 0.7, t_ns + 1)
    if drive == "site":
        om, de = np.outer(rng.uniform(0.5, 1.5, n), om), np.outer(rng.uniform(0.5, 1.5, n), de)
        ph = np.outer(rng.uniform(-1, 1, n), np.linspace(0, 1, t_ns + 1))
    pl = rsv.PulseArrays(om, de, ph)
    psi0 = torch.from_numpy(wl.random_state(n, rng)).to("cuda:0")
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, "c128")
    # |H| tau: drive and detuning of all atoms, and the pairs' energies
    u = wl.C6_RB / np.linalg.norm(xyz[:, None] - xyz[None] + 1e9 * np.eye(n)[..., None], axis=-1) ** 6
    parts = int(np.ceil((n * 30.0 + np.triu(u, 1).sum()) * dt * 1e-3 / 2.0))
    ref = taylor_steps(reg, pl, psi0.clone(), 4, steps, dt, parts)
    for prec, tol, bound in (("c128", 1e-11, 1e-9), ("c64", 1e-7, 1e-5)):
        r = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, prec)
        psi = psi0.to(torch.complex64 if prec == "c64" else torch.complex128).clone()
        rsv.rsv_evolve_device(r, pl, rsv.evolve_opts(dt, tol, 30, 12, 4, steps), psi)
        err = float((psi.to(torch.complex128) - ref).norm())
        assert err <= bound, (prec, err)
        e = rsv.rsv_energy_device(r, pl, 6, dt, psi)
        wide = psi.to(torch.complex128)
        h = torch.empty_like(wide)
        rsv.rsv_apply_hamiltonian(reg, pl, 6, dt, wide, h)
        want = float((wide.conj() * h).sum().real) / float(wide.norm()) ** 2
        scale = n * 30.0 + np.triu(u, 1).sum()
        assert abs(e - want) <= (1e-13 if prec == "c128" else 1e-6) * scale, (prec, e, want)
        rsv.rsv_register_destroy(r)
    rsv.rsv_register_destroy(reg)


@pytest.mark.parametrize("n", [10, 13, 17, 18, 19])
def test_gradient_of_two_distant_groups(ctx, n):  # noqa: F811
    """Two groups too far apart to interact: cost and gradients are the sums of the groups' own
    (registers of at most 10 atoms, which are compared with the oracle elsewhere)."""
    rng = np.random.default_rng(600 + n)
    t_ns, dt = 40, 10
    k = n // 2
    a = wl.random_register(k, 18.0, 5.5, rng)
    b = wl.random_register(n - k, 18.0, 5.5, rng)
    far = b + np.array([1e4] + [0.0] * (b.shape[1] - 1))
    om, de = wl.pwl([0, 40], [6, 13], t_ns), wl.pwl([0, 40], [-5, 11], t_ns)
    ph = np.linspace(-0.4, 0.8, t_ns + 1)
    w = rng.uniform(-1, 1, n)
    c, g_om, g_de, _ = gpu_grad(ctx, np.vstack([a, far]), wl.C6_RB, om, de, ph, dt, w, "c128")
    ca, a_om, a_de, _ = gpu_grad(ctx, a, wl.C6_RB, om, de, ph, dt, w[:k], "c128")
    cb, b_om, b_de, _ = gpu_grad(ctx, b, wl.C6_RB, om, de, ph, dt, w[k:], "c128")
    scale = max(np.abs(a_om + b_om).max(), np.abs(a_de + b_de).max())
    assert abs(c - ca - cb) <= 2e-10
    assert np.abs(g_om - a_om - b_om).max() <= 2e-8 * scale
    assert np.abs(g_de - a_de - b_de).max() <= 2e-8 * scale

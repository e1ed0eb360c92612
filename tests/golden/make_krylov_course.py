"""Writes tests/golden/krylov_course.npz: the Lanczos coefficients of consecutive time steps and
the smallest dimension that meets the tolerance in each, for replays of the rule that decides when a
growing Krylov space is tested and how many iterations are queued before that.

The three-term recurrence in complex128 on the oracle's H psi, to kmax vectors whatever the
tolerance; a step not resolved by them advances by the longest part that is (the first dyadic
fraction, then ten bisections) and goes on from there, as the library does.  Per run:
  name              the series it belongs to (runs of one series are consecutive)
  run               0 for a step's first run, 1, 2, .. for the parts that follow
  norm, tau, tol    |psi|, the part of the step still to do (us), the tolerance
  kmax, need        the dimension limit, and the smallest dimension that meets tol (0: none)
  alpha, beta       alpha_0.., beta_0.. (kmax of each, padded with zeros)

python tests/golden/make_krylov_course.py   (about ten minutes)
"""
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
sys.path.insert(0, ROOT)

from oracle import model  # noqa: E402
from paper_2510_09813_amd import workloads as wl  # noqa: E402


def exponential(al, be, tau):
    """exp(-i tau T) e_1 from the eigenvectors of T."""
    lam, q = np.linalg.eigh(np.diag(al) + np.diag(be, 1) + np.diag(be, -1))
    return q @ (np.exp(-1j * tau * lam) * q[0])


def series(name, w, psi, first, steps, rows):
    u = model.interaction_matrix(w.xyz, w.c6)
    psi = psi.astype(np.complex128)
    for k in range(first, first + steps):
        om, de, ph = model.step_parameters(w.n_atoms, w.omega, w.delta, w.phi, w.dt_ns, k)
        left, run = w.dt_ns * 1e-3, 0
        while left > 0.0:
            nrm = float(np.linalg.norm(psi))
            basis, al, be = [psi / nrm], [], []
            for j in range(w.kmax):
                z = model.apply_hamiltonian(basis[j], u, om, de, ph)
                al.append(float(np.vdot(basis[j], z).real))
                z = z - al[j] * basis[j] - (be[j - 1] * basis[j - 1] if j else 0.0)
                be.append(float(np.linalg.norm(z)))
                basis.append(z / be[j])

            def estimate(m, t):
                return be[m - 1] * abs(exponential(al[:m], be[:m - 1], t)[-1]) * nrm

            need = next((m for m in range(1, w.kmax + 1) if estimate(m, left) <= w.tol), 0)
            part, m = left, need or w.kmax
            if not need:
                d = next(d for d in range(1, 13) if estimate(m, np.ldexp(left, -d)) <= w.tol)
                part, bad = np.ldexp(left, -d), np.ldexp(left, 1 - d)
                for _ in range(10):
                    mid = 0.5 * (part + bad)
                    part, bad = (mid, bad) if estimate(m, mid) <= w.tol else (part, mid)
            rows.append((name, run, nrm, left, w.tol, w.kmax, need, al, be))
            y = exponential(al[:m], be[:m - 1], part)
            psi = nrm * sum(c * v for c, v in zip(y, basis))
            left, run = 0.0 if part == left else left - part, run + 1
    print(name, [r[6] for r in rows if r[0] == name], flush=True)


def product_state(n, rng):
    psi = np.ones(1, dtype=complex)
    for _ in range(n):
        p, ph = rng.uniform(0.02, 0.15), rng.uniform(-np.pi, np.pi)
        psi = np.kron(psi, [np.sqrt(1 - p), np.sqrt(p) * np.exp(1j * ph)])
    return psi


def main():
    rows = []
    ground = np.zeros(1 << 21)
    ground[0] = 1.0
    # the random-register sweep from its start: interactions set the width of the spectrum
    series("sweep21", wl.random27(0, 21, "c64"), ground, 0, 10, rows)
    # windows of a sweep: fast convergence, from far above the tolerance and from near it
    for n, dt, kmax, tol in ((13, 5, 30, 1e-10), (15, 10, 48, 1e-7)):
        rng = np.random.default_rng(n)
        om, de, t = wl.sweep_pulses(500, 3000, *rng.uniform(wl.TWO_PI, 3 * wl.TWO_PI, 2))
        w = wl.Workload("", wl.random_register(n, 30.0, 5.0, rng), wl.C6_RB, om, de, None, t, dt, tol, kmax)
        series(f"window{n}", w, product_state(n, rng), 100, 5, rows)
    # a lattice whose steps take more than kmax vectors
    w = wl.square20()
    w.xyz = wl.square_lattice(4, 4, 6.0)
    series("square16", w, product_state(16, np.random.default_rng(5)), 100, 3, rows)
    pad = max(len(r[7]) for r in rows)
    np.savez_compressed(
        os.path.join(HERE, "krylov_course.npz"),
        name=np.array([r[0] for r in rows]), run=np.array([r[1] for r in rows]),
        norm=np.array([r[2] for r in rows]), tau=np.array([r[3] for r in rows]),
        tol=np.array([r[4] for r in rows]), kmax=np.array([r[5] for r in rows]),
        need=np.array([r[6] for r in rows]),
        alpha=np.array([np.pad(r[7], (0, pad - len(r[7]))) for r in rows]),
        beta=np.array([np.pad(r[8], (0, pad - len(r[8]))) for r in rows]))


if __name__ == "__main__":
    main()

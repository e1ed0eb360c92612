"""Host logic of the sweeps' plans (CPU only), for both kinds of input: every bit is flipped exactly
once by the low pass, its extension or a high pass, every high tile lies inside the index with its
run below its high bits, and both kinds share the low tile (one set of diagonal tables serves
them).  And the Chebyshev form of the tridiagonal exponential against scipy: at most 256 terms of
rounding eps on a unit vector, 1e-13."""
import ctypes as C

import numpy as np
import pytest
import scipy.linalg

from paper_2510_09813_amd import rsv
from tests.test_tile_plan import TilePlan


def plan(prec, n, stored):
    f = rsv.lib()._ZN3rsv10sweep_planEiib  # rsv::sweep_plan(int, int, bool), host code
    f.restype, f.argtypes = TilePlan, [C.c_int, C.c_int, C.c_bool]
    return f(prec, n, stored)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("stored", [False, True])
def test_plans_partition_the_bits(prec, stored):
    for n in range(1, 31):
        p = plan(prec, n, stored)
        assert p.n == n and p.lo_bits == plan(prec, n, not stored).lo_bits
        covered = []
        for i in range(p.n_hi_passes):
            r, a, g = p.run_bits[i], p.tile_a[i], p.hi_bits - p.run_bits[i]
            assert 3 <= r <= 6 and r <= a and a + g <= n and a <= p.flip_lo[i] < p.flip_hi[i] <= a + g
            assert 8 <= p.hi_bits <= 13 and p.hi_bits <= n
            covered += list(range(p.flip_lo[i], p.flip_hi[i]))
        if p.lo_ext:
            covered += list(range(p.lo_ext_bit, p.lo_ext_bit + p.lo_ext))
        assert 0 <= p.lo_ext <= 7 and sorted(covered) == list(range(p.lo_bits, n))
        # only a stored input's neighbours can be read in place of a high pass
        assert p.n_hi_passes > 0 or p.lo_bits == n or stored


@pytest.mark.parametrize("m", [1, 2, 5, 28, 64])
@pytest.mark.parametrize("width", [1e-3, 1.0, 20.0, 120.0, 900.0])
def test_tridiagonal_series(m, width):
    f = rsv.lib()._ZN3rsv19tridiag_expm_seriesEiPKdS1_dPdS2_S2_
    rng = np.random.default_rng(m)
    al, be = rng.uniform(-1, 1, m) * width, rng.uniform(0.1, 0.7, max(m - 1, 1)) * width
    t = np.diag(al) + np.diag(be[: m - 1], 1) + np.diag(be[: m - 1], -1)
    vp = lambda x: x.ctypes.data_as(C.c_void_p)
    for tau in (1.0, -0.6):
        yr, yi, work = np.zeros(m), np.zeros(m), np.zeros(2 * m * m + 2 * m)
        assert f(m, vp(al), vp(be), C.c_double(tau), vp(yr), vp(yi), vp(work)) == 0
        ref = scipy.linalg.expm(-1j * tau * t)[:, 0]
        # (scipy's own error grows with the norm it squares away)
        np.testing.assert_allclose(yr + 1j * yi, ref, rtol=0, atol=1e-13 * max(1.0, width))

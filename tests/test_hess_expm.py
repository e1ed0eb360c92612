"""First column of the exponential of an upper Hessenberg matrix (host, CPU only), on both of its
routes: the Chebyshev series (nearly skew-Hermitian matrices) and the Pade approximant, against
scipy.  Tolerance: the series sums K <= 600 terms of size at most e^2 with rounding eps each, the
norm of the column being at most 1 here: 600 e^2 eps = 1e-12 (K of the widest case)."""
import ctypes as C

import numpy as np
import pytest
import scipy.linalg

from paper_2510_09813_amd import rsv


def hess_expm_e1(a, ld, tau):
    # rsv::hess_expm_e1(int, const std::complex<double>*, int, double, std::complex<double>*)
    f = rsv.lib()._ZN3rsv12hess_expm_e1EiPKSt7complexIdEidPS1_
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_void_p, C.c_int, C.c_double, C.c_void_p]
    y = np.zeros(a.shape[0], dtype=complex)
    full = np.zeros((a.shape[0], ld), dtype=complex)
    full[:, : a.shape[0]] = a
    assert f(a.shape[0], full.ctypes.data, ld, tau, y.ctypes.data) == 0
    return y


@pytest.mark.parametrize("m", [1, 2, 3, 12, 28, 63])
@pytest.mark.parametrize("half_width", [1e-3, 1.0, 30.0, 250.0])
@pytest.mark.parametrize("loss", [0.0, 0.02, 5.0])
def test_against_scipy(m, half_width, loss):
    rng = np.random.default_rng(m)
    b = rng.uniform(0.3, 1, m - 1) * half_width
    a = np.diag(1j * rng.normal(size=m) * half_width) + np.diag(b, -1) - np.diag(b, 1)
    a = a - loss * np.diag(rng.uniform(0, 1, m)) + 1e-3 * loss * np.triu(rng.normal(size=(m, m)))
    for tau in (1.0, 0.3):
        ref = scipy.linalg.expm(tau * a)[:, 0]
        np.testing.assert_allclose(hess_expm_e1(a, m + 2, tau), ref, rtol=0, atol=1e-12)

"""The series forms of the host exponentials under the address and undefined-behaviour sanitizers
(tests/cpp/host_series_test.cpp), and the rule that sends a small register's call to the device's
series (packed_resolves): its bound on the number of terms, and the Bessel tail behind it.  CPU only; the
driver needs g++ and the HIP headers (the sources include them for their declarations)."""
import ctypes as C
import os
import shutil
import subprocess

import pytest
import scipy.special

from paper_2510_09813_amd import rsv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_09813_amd", "csrc")
DRIVER = os.path.join(ROOT, "tests", "cpp", "host_series_test.cpp")
HIP_INC = "/opt/rocm/include"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INC, "hip")),
                    reason="g++ or the HIP headers not available")
def test_series_under_sanitizers(tmp_path):
    flags = ["-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer"]
    inc = ["-D__HIP_PLATFORM_AMD__", f"-I{HIP_INC}", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]
    exe = tmp_path / "host_series_test"
    subprocess.run(["g++", *flags, *inc, DRIVER, os.path.join(CSRC, "tridiag.cpp"),
                    os.path.join(CSRC, "dense_expm.cpp"), "-o", str(exe)], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
    assert "host_series ok" in r.stdout


def test_which_steps_the_device_series_resolves():
    f = rsv.lib()._ZN3rsv15packed_resolvesEdd
    f.restype, f.argtypes = C.c_bool, [C.c_double, C.c_double]
    # the device sums at most 512 terms; T's Gershgorin half-width is at most three times the
    # spectrum's, and a + 8 a^(1/3) + 20 terms leave a tail below 1e-15
    lo, hi = 0.0, 1e6
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if f(1.0, mid) else (lo, mid)
    a = 3.0 * lo
    assert abs(a + 8.0 * a ** (1 / 3) + 20.0 - 510.0) < 1e-6
    assert abs(scipy.special.jv(510, a)) < 1e-15
    for tau in (0.005, 0.01, 1.0):  # the product decides
        assert f(tau, lo * (1 - 1e-9) / tau) and not f(tau, lo * (1 + 1e-9) / tau)
    assert f(0.01, 0.0) and not f(0.01, float("inf"))

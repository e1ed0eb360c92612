"""The rule that says when a growing Krylov space is tested and how many iterations are queued
before that (csrc/krylov_course.h), replayed on stored coefficients of consecutive time steps
(tests/golden/make_krylov_course.py) under the address and undefined-behaviour sanitizers.

The dimension must be the smallest that meets the tolerance, however the iterations were queued.  Of
costly vectors no iteration beyond it is queued once a step before says what to expect (a step's
dimension falls by at most one against the step before in these series), of cheap ones at most
one per run on average.  CPU only; needs g++ and the HIP headers."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_09813_amd", "csrc")
HIP_INC = "/opt/rocm/include"


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INC, "hip")):
        pytest.skip("g++ or the HIP headers not available")
    tmp = tmp_path_factory.mktemp("course")
    d = np.load(os.path.join(ROOT, "tests", "golden", "krylov_course.npz"))
    names = list(dict.fromkeys(d["name"].tolist()))
    with open(tmp / "runs.txt", "w") as f:
        f.write(f"{len(d['run'])}\n")
        for i in range(len(d["run"])):
            k = int(d["kmax"][i])
            f.write(f"{names.index(d['name'][i])} {d['run'][i]} {float(d['norm'][i])!r} {float(d['tau'][i])!r} "
                    f"{float(d['tol'][i])!r} {k} {d['need'][i]}\n")
            f.write(" ".join(repr(float(x)) for x in (*d["alpha"][i, :k], *d["beta"][i, :k])) + "\n")
    exe = tmp / "krylov_course_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
                    "-D__HIP_PLATFORM_AMD__", f"-I{HIP_INC}", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
                    os.path.join(ROOT, "tests", "cpp", "krylov_course_test.cpp"), os.path.join(CSRC, "tridiag.cpp"),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    r = subprocess.run([str(exe), str(tmp / "runs.txt")], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and "replay ok" in r.stdout, r.stdout[-500:] + r.stderr[-3000:]
    rows = np.array([[int(x) for x in line.split()] for line in r.stdout.splitlines()[:-1]])
    return d, names, rows


def test_dimensions_do_not_depend_on_the_queue(replay):
    d, _, rows = replay
    want = np.where(d["need"] > 0, d["need"], d["kmax"])
    for p in range(6):
        np.testing.assert_array_equal(rows[:, 3 + 2 * p], want)


@pytest.mark.parametrize("series", ["sweep21", "window13", "window15", "square16"])
def test_queued_iterations(replay, series):
    d, names, rows = replay
    rows = rows[rows[:, 0] == names.index(series)]
    dim, costly, cheap = rows[:, 3], rows[:, 4], rows[:, 10]
    assert len(rows) >= 5
    np.testing.assert_array_equal(costly, dim)
    assert (cheap >= dim).all() and cheap.sum() <= dim.sum() + len(rows)

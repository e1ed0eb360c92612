"""Windows of several steps that converge inside kmax: the iterations queued against the dimensions
the steps needed, and a window against the same steps one call each (which know no previous step),
bit for bit.  The registers are the random-register sweep's: vectors of 16 MiB and more queue
nothing beyond what a step needs while dimensions rise; smaller ones at most one iteration per step
on average."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import empty_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,spare", [(16, "c128", 1), (17, "c64", 1), (20, "c128", 0), (21, "c64", 0),
                                          (22, "c64", 0)])
def test_iterations_of_a_window(n, prec, spare):
    first, steps = 5, 8
    w = wl.random27(0, n, prec)
    ctx = rsv.rsv_ctx_create(0)
    reg = rsv.rsv_register_create(ctx, w.xyz, w.c6, prec)
    pulses = rsv.PulseArrays(w.omega, w.delta)

    def evolve(psi, k, count):
        return rsv.rsv_evolve_device(reg, pulses, rsv.evolve_opts(w.dt_ns, w.tol, w.kmax, 12, k, count), psi)

    a = empty_dev(n, prec)
    a.zero_()
    a[0] = 1
    evolve(a, 0, first)
    b = a.clone()
    one = [evolve(a, first + k, 1) for k in range(steps)]
    dims = [int(s.krylov_max) for s in one]
    st = evolve(b, first, steps)
    assert st.substeps == 0 and st.krylov_max == max(dims) < w.kmax
    fall = sum(max(0, x - y - 1) for x, y in zip(dims, dims[1:]))  # more than a hint allows for
    assert sum(dims) <= st.krylov_iters <= sum(dims) + fall + spare * steps
    assert np.array_equal(to_host(a), to_host(b))
    rsv.rsv_register_destroy(reg)
    rsv.rsv_ctx_destroy(ctx)

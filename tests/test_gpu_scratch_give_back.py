"""Device scratch of finished calls is kept within its bound, and rsv_ctx_trim gives it back to the
device; registers, their workspaces and results are not kept."""
import time

import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import empty_dev, to_dev

pytestmark = pytest.mark.gpu


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def soon(condition):
    """The driver may count freed memory a little later than hipFree returns."""
    for _ in range(100):
        if condition():
            return True
        time.sleep(0.05)
    return False


def test_trim_returns_call_scratch_only():
    import torch
    om, de, _ = wl.sweep_pulses(50, 100, 9.0, 9.0)
    pulses = rsv.PulseArrays(om, de)
    n, kmax = 10, 14
    rho = torch.zeros(4 ** n, dtype=torch.complex128, device="cuda:0")
    rho[0] = 1.0
    psi = empty_dev(22, "c128")
    psi.zero_()
    psi[0] = 1.0
    small = to_dev(wl.random_state(14, np.random.default_rng(1)), "c128")
    ctx = rsv.rsv_ctx_create(0)
    try:
        assert rsv.rsv_ctx_trim(ctx) == 0
        reg = rsv.rsv_register_create(ctx, wl.chain(n, 6.0), wl.C6_RB, "c128")
        rsv.rsv_lindblad_evolve_device(reg, pulses, rsv.evolve_opts(10, 1e-8, kmax, n_steps=1), (0.5, 0.5), rho)
        held = rsv.rsv_ctx_bytes_in_use(ctx)
        before = free_bytes()
        arnoldi = (kmax + 1) * 16 * 4 ** n  # 240 MiB
        kept = rsv.rsv_ctx_trim(ctx)
        assert arnoldi <= kept <= arnoldi + (64 << 20)
        assert soon(lambda: free_bytes() - before >= arnoldi)
        assert rsv.rsv_ctx_trim(ctx) == 0 and rsv.rsv_ctx_bytes_in_use(ctx) == held
        # a workspace of 1 GiB goes back with its register
        before = free_bytes()
        reg2 = rsv.rsv_register_create(ctx, wl.random_register(22, 30.0, 5.0, np.random.default_rng(2)), wl.C6_RB, "c128")
        rsv.rsv_evolve_device(reg2, pulses, rsv.evolve_opts(10, 1e-6, 13, n_steps=1), psi)
        assert soon(lambda: before - free_bytes() >= 1 << 30)
        rsv.rsv_register_destroy(reg2)
        assert soon(lambda: before - free_bytes() < 1 << 28)
        assert rsv.rsv_ctx_trim(ctx) == 0
        occ = rsv.rsv_occupations_device(ctx, 14, small)
        assert rsv.rsv_ctx_trim(ctx) > 0
        np.testing.assert_array_equal(rsv.rsv_occupations_device(ctx, 14, small), occ)
        rsv.rsv_register_destroy(reg)
        assert rsv.rsv_ctx_bytes_in_use(ctx) == 0
    finally:
        rsv.rsv_ctx_destroy(ctx)

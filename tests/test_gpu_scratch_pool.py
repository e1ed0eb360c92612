"""Device scratch kept between calls: what a context holds back neither counts as in use nor
against its budget, makes way for requests that need the room, and is safe on another stream."""
import numpy as np
import pytest

from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu


def test_kept_blocks_leave_the_budget_to_later_calls():
    import torch
    n, kmax = 6, 20
    om, de, _ = wl.sweep_pulses(50, 100, 9.0, 9.0)
    pulses, opts = rsv.PulseArrays(om, de), rsv.evolve_opts(10, 1e-10, kmax, n_steps=1)
    xyz = wl.chain(n, 6.0)
    # room for the 4^6-element Arnoldi space and the register, and little more
    arnoldi = (kmax + 3) * 16 * 4 ** n
    ctx = rsv.rsv_ctx_create(0, arnoldi + (1 << 20))
    try:
        reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, "c128")
        rho = torch.zeros(4 ** n, dtype=torch.complex128, device="cuda:0")
        rho[0] = 1.0
        rsv.rsv_lindblad_evolve_device(reg, pulses, opts, (0.5, 0.5), rho)
        held = rsv.rsv_ctx_bytes_in_use(ctx)
        psi = to_dev(wl.random_state(n, np.random.default_rng(1)), "c128")
        for _ in range(3):  # other sizes of scratch, then the large block again
            occ = rsv.rsv_occupations_device(ctx, n, psi)
            cor = rsv.rsv_correlations_device(ctx, n, psi)
            assert rsv.rsv_ctx_bytes_in_use(ctx) == held
            rsv.rsv_lindblad_evolve_device(reg, pulses, opts, (0.5, 0.5), rho)
            assert rsv.rsv_ctx_bytes_in_use(ctx) == held
        np.testing.assert_allclose(np.diag(cor), occ, rtol=1e-13)
        # a second register whose workspace fits only once the kept block is gone
        reg2 = rsv.rsv_register_create(ctx, wl.chain(11, 6.0), wl.C6_RB, "c128")
        d = to_dev(wl.random_state(11, np.random.default_rng(2)), "c128")
        rsv.rsv_evolve_device(reg2, pulses, opts, d)
        rsv.rsv_register_destroy(reg2)
        assert rsv.rsv_ctx_bytes_in_use(ctx) == held
        rsv.rsv_register_destroy(reg)
        assert rsv.rsv_ctx_bytes_in_use(ctx) == 0
    finally:
        rsv.rsv_ctx_destroy(ctx)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_scratch_moves_between_streams(prec):
    import torch
    ctx = rsv.rsv_ctx_create(0)
    try:
        n = 14
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        states = [to_dev(wl.random_state(n, np.random.default_rng(s)), prec) for s in (3, 4)]
        torch.cuda.synchronize()
        want = [(rsv.rsv_occupations_device(ctx, n, x, prec), rsv.rsv_sample_device(ctx, n, x, 5, 200, prec))
                for x in states]
        for k in range(6):
            x, st = states[k % 2], streams[(k // 2) % 2]
            np.testing.assert_array_equal(
                rsv.rsv_occupations_device(ctx, n, x, prec, stream=st.cuda_stream), want[k % 2][0])
            np.testing.assert_array_equal(
                rsv.rsv_sample_device(ctx, n, x, 5, 200, prec, stream=st.cuda_stream), want[k % 2][1])
    finally:
        rsv.rsv_ctx_destroy(ctx)

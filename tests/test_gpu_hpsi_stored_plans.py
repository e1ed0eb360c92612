"""H|psi> of 13 to 20 atoms, where every size has a plan of its own for a stored input (low tiles of 9
to 12 bits with 4 to 7 bits read beyond them, or one high pass), in both precisions and with every
form of the drive, against the oracle.  Tolerances as in test_gpu_hpsi."""
import pytest

from oracle import model
from paper_2510_09813_amd import rsv
from paper_2510_09813_amd import workloads as wl
from tests.gpu_util import empty_dev, rel_err, to_dev, to_host
from tests.test_gpu_hpsi import TOL, _pulses, _register, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", range(13, 21))
def test_every_size_and_drive(ctx, n, prec):  # noqa: F811
    xyz, rng = _register(n, 900 + n)
    reg = rsv.rsv_register_create(ctx, xyz, wl.C6_RB, prec)
    u = model.interaction_matrix(xyz, wl.C6_RB)
    d_in = to_dev(wl.random_state(n, rng), prec)
    psi, d_out = to_host(d_in), empty_dev(n, prec)
    for per_site, phase in ((False, False), (False, True), (True, True)):
        om, de, ph = _pulses(n, rng, per_site, phase)
        rsv.rsv_apply_hamiltonian(reg, rsv.PulseArrays(om, de, ph), 1, 5, d_in, d_out)
        ref = model.apply_hamiltonian(psi, u, *model.step_parameters(n, om, de, ph, 5, 1))
        assert rel_err(to_host(d_out), ref) < TOL[prec], (n, per_site, phase)
    rsv.rsv_register_destroy(reg)

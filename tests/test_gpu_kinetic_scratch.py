"""fr_kinetic_energy evaluates its residual into a Runge-Kutta register. No scheme carries anything in
the registers from one step to the next, so diagnostics between steps must leave the run unchanged
bit for bit, and a call before any step must agree with one after."""
import numpy as np
import pytest

from paper_2308_06605_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["lsrk45", "rk4", "ssprk104"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_diagnostics_between_steps(scheme, prec):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    m = I.box_mesh((3, 5, 4), q=2, curve_amp=0.04)
    kw = dict(prec="fp32", ref_rho=1.0, ref_p=1.0 / (1.4 * 0.01)) if prec == "fp32" else {}
    states, energies = [], []
    for diagnose in (True, False):
        g = fr.FRMesh(m, 3, mu=1e-3, flux="roe", **kw)
        X = g.sol_coords()
        U = I.state_from_coords(X, I.tgv_state) + I.random_smooth_perturbation(X, seed=2, amp=0.01)
        g.set_state(U)
        for _ in range(3):
            if diagnose:
                energies.append(g.kinetic_energy())
            g.rk_step(1e-3, scheme, 2)
        states.append(g.get_state())
        g.set_state(U)
        energies.append(g.kinetic_energy())
        g.close()
    assert np.array_equal(states[0], states[1])
    assert energies[0] == energies[3] == energies[4]

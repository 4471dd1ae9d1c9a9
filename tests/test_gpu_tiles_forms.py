"""Every tile choice against the default by size, bit for bit, in the forms whose other tests run the
default alone: p = 1 and 4 in both precisions, the inviscid equations, an eddy viscosity, walls, the
local DG flux. Meshes of 75 elements: the default takes half blocks and one-wave face blocks for
them, large meshes the others; ragged last blocks, residuals and fused runs of several steps."""
import numpy as np
import pytest

from paper_2308_06605_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,prec,form", [
    (0, "fp64", "br2"), (1, "fp64", "br2"), (4, "fp64", "br2"), (0, "fp32", "br2"), (1, "fp32", "br2"), (4, "fp32", "br2"),
    (1, "fp64", "euler"), (3, "fp64", "euler"), (2, "fp32", "euler"), (4, "fp32", "euler"),
    (1, "fp64", "eddy"), (3, "fp64", "eddy"), (4, "fp64", "eddy"), (3, "fp64", "ldgeddy"),
    (2, "fp64", "walls"), (3, "fp64", "walls"), (4, "fp64", "walls"), (2, "fp32", "walls"), (3, "fp32", "walls"),
    (4, "fp32", "walls"), (1, "fp64", "ldg"), (2, "fp64", "ldg"), (4, "fp64", "ldg")])
def test_every_choice_bitwise(p, prec, form):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    p0 = 1.0 / (1.4 * 0.01)
    kw = dict(mu=0.0 if form == "euler" else 1e-2, flux="roe")
    if prec == "fp32":
        kw.update(prec="fp32", ref_rho=1.0, ref_p=p0)
    if "ldg" in form:
        kw.update(viscous="ldg", ldg_tau=0.2)
    if form == "walls":
        m = I.box_mesh((3, 5, 5), q=1, periodic=(True, False, True))
        kw.update(bc_tag=I.boundary_tags(m), wall_T=p0)
    else:
        m = I.box_mesh((3, 5, 5), q=max(1, min(p, 2)), curve_amp=0.04)
    g = fr.FRMesh(m, p, **kw)
    X = g.sol_coords()
    U = I.state_from_coords(X, I.tgv_state) + I.random_smooth_perturbation(X, seed=p, amp=0.01)
    if "eddy" in form:
        g.set_eddy_viscosity(np.random.default_rng(p).uniform(0, 0.01, m.n_elem))

    def results():
        g.set_state(U)
        R = g.residual()
        g.rk_step(1e-4, "lsrk45", 3)
        return R, g.get_state()

    R0, S0 = results()
    assert np.isfinite(S0).all() and not np.array_equal(S0, U)
    for epb in (0, 1):
        for fbs in (0, 1, 2):
            g.set_tiles(epb, fbs)
            R, S = results()
            assert np.array_equal(R, R0) and np.array_equal(S, S0), (epb, fbs)
    g.close()

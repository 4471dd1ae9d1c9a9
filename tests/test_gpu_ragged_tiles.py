"""The element kernels where their exchanges can go wrong: element counts that leave the last
block ragged, at every way an element's points meet the wavefronts (whole elements within a wave
at p = 0 and 1, one element per wave at p = 3, elements across waves at p = 2, 4 and 5) and both
tile choices, against the long-double oracle by the FP64 floor rule
e_v <= max(1e-12, 2 f_v), f_v the double oracle's own error."""
import numpy as np
import pytest

import oracle
from paper_2308_06605_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epb", [0, 1])
@pytest.mark.parametrize("p", [0, 1, 2, 3, 4, 5])
def test_ragged_blocks(p, epb):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    m = I.box_mesh((3, 5, 3), q=max(1, min(p, 2)), curve_amp=0.04)
    kw = dict(mu=1e-2, flux="roe")
    g = fr.FRMesh(m, p, **kw)
    g.set_tiles(epb, 0)
    X = g.sol_coords()
    U = I.state_from_coords(X, I.tgv_state) + I.random_smooth_perturbation(X, seed=p, amp=0.01)
    g.set_state(U)
    R = g.residual()
    g.close()
    ld = oracle.Oracle(m, p, precision="ld", **kw).residual(U)
    d = oracle.Oracle(m, p, **kw).residual(U)
    scale = np.abs(ld).max(axis=(0, 2))
    err = np.abs(R - ld).max(axis=(0, 2)) / scale
    floor = np.abs(d - ld).max(axis=(0, 2)) / scale
    print(f"p={p} epb={epb}: err {err}, floor {floor}", flush=True)
    assert np.all(err <= np.maximum(1e-12, 2 * floor)), (err, floor)

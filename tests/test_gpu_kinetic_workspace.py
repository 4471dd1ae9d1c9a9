"""What fr_kinetic_energy keeps: the first RK register, which steps then use, and its partial sums, once."""
import pytest

from paper_2308_06605_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_device_bytes():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    g = fr.FRMesh(I.box_mesh(4, q=1), 3, mu=1e-3)
    g.set_state(I.state_from_coords(g.sol_coords(), I.tgv_state))
    held = [g.info()["device_bytes"]]
    for f in (g.kinetic_energy, g.kinetic_energy, lambda: g.rk_step(1e-4, "lsrk45", 1), g.kinetic_energy):
        f()
        held.append(g.info()["device_bytes"])
    g.close()
    assert held[1] - held[0] == 64 * 40 * 64 + 24 * (64 * 64 // 256 + 1)
    assert held[1:] == [held[1]] * 4

"""The network's kernels where their blocks end: sample counts around the 16 samples a block takes
and the 256 blocks a training pass has at most, input counts around the 16-input steps, and rows
that do and do not start on 16 bytes (the two ways a row is read), against the oracle. The gates are
those of the network's other tests: 1e-4 relative for the outputs, 5e-5 of its largest magnitude
for the gradient of each parameter array."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,n,pad", [(1, 1, 0), (5, 15, 0), (16, 16, 0), (17, 17, 3), (68, 4096, 0), (68, 4097, 1),
                                     (64, 4113, 4), (128, 8192, 0), (31, 9001, 0)])
def test_block_edges(F, n, pad):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    rng = np.random.default_rng(F + n)
    mean, std = rng.normal(size=F).astype(np.float32), rng.uniform(0.5, 2, F).astype(np.float32)
    wide = (rng.normal(size=(n, F + pad)) * np.pad(std, (0, pad)) + np.pad(mean, (0, pad))).astype(np.float32)
    t = rng.uniform(0, 2, n).astype(np.float32)
    theta = M.init_params(F, seed=n)
    net = fr.MLP(F, theta, mean, std)
    Xd, td = torch.from_numpy(wide).cuda(), torch.from_numpy(t).cuda()
    X = wide[:, :F]
    y = net.forward(Xd).cpu().numpy()
    ref = M.forward(M.effective(theta, F), X, mean, std)
    assert np.all(np.abs(y - ref) <= 1e-4 * np.abs(ref))
    loss, g = net.loss_grad(Xd, td)
    Lo, go = M.loss_and_grad(theta, X, t, mean, std)
    assert abs(loss - Lo) <= 2e-5 * Lo
    a, b = M.unpack(g, F), M.unpack(go, F)
    for k in a:
        assert np.abs(a[k] - b[k]).max() <= 5e-5 * np.abs(b[k]).max(), k
    net.close()

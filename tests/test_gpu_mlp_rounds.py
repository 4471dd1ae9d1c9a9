"""Evaluations of more samples than the chip holds at once, whose blocks loop over them: every output is
bit for bit that of the sample in a call small enough for one round, at sample counts that end inside
a round and inside a block's 16 samples and at each number of resident blocks (6, 5 and 4 per CU)."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,n", [(5, 24592), (12, 60001), (31, 20496), (68, 45007), (128, 16400)])
def test_rounds(F, n):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2308_06605_amd import fr

    rng = np.random.default_rng(F)
    mean, std = rng.normal(size=F).astype(np.float32), rng.uniform(0.5, 2, F).astype(np.float32)
    X = torch.from_numpy((rng.normal(size=(n, F)) * std + mean).astype(np.float32)).cuda()
    net = fr.MLP(F, M.init_params(F, seed=n), mean, std)
    y = net.forward(X).cpu()
    parts = torch.cat([net.forward(X[i:i + 4096]) for i in range(0, n, 4096)]).cpu()
    net.close()
    assert torch.equal(y, parts) and bool(torch.isfinite(y).all())

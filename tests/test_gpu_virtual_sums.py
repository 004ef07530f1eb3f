"""Gradients on regenerated features: quads, chunks and batches at their edges against the oracle."""
import numpy as np
import pytest

from oracle import gpga_oracle as orc
from paper_2105_09080_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,B,bad", [(1, 1, 1, False), (3, 4, 32, False), (5, 1027, 17, False), (4, 2050, 31, False),
                                       (65, 259, 4, False), (3, 300_001, 2, False), (6, 1000, 32, True)])
def test_gradient_on_regenerated_features(n, d, B, bad):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness as hx
    M = 40
    y = inputs.virtual_labels(n, M, seed=3)
    idx = inputs.batch_indices(1, n, B, M, seed=5)[0]
    X = (inputs.random_state(n, d, seed=7)[0] / np.sqrt(1.5 * d)).astype(np.float32)   # margins of order one
    G = orc.logreg_virtual_grad(9, y, X.astype(np.float64), idx, 0.5)
    if bad:
        idx = idx.copy()
        idx[2, B - 1], idx[4, 0] = M, -1
    sim = hx.Simulation(n, d, topology="ring", H=0, lr=0.1, ld=d + 1)
    sim.problem_logreg_virtual(9, y, 0.5)
    sim.set_state(X=X)
    sim.local_grad(sim.upload_batches(idx[None])[0])
    got = sim.G.cpu().numpy().astype(np.float64)
    if bad:   # the nodes with a row outside the data, and only they, are poisoned
        assert np.isnan(got[[2, 4]]).all()
        got, G = np.delete(got, [2, 4], 0), np.delete(G, [2, 4], 0)
    assert np.abs(got - G).max() <= 1e-5 * np.abs(G).max()   # fp32 sums over at most 32 samples
    sim.close()

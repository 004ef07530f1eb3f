"""Consensus distance and node mean on wide arrays: workgroups of 256 and 1024 column units, ragged widths and strides."""
import numpy as np
import pytest

from oracle import gpga_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


# 245 760 units of four columns are the first width with 1024 units a workgroup; the last ones fill little more or less than half
# of a second round and a fourth part of a fourth
@pytest.mark.parametrize("n,d,pad", [(1, 983_037, 0), (3, 983_036, 0), (5, 983_041, 3), (2, 1_048_576, 0), (6, 1_048_577, 0), (9, 983_100, 1),
                                     (4, 1_593_345, 0), (4, 1_593_341, 1), (24, 3_200_003, 0)])
def test_distance_and_mean_of_wide_arrays(hx, n, d, pad):
    import torch
    sim = hx.Simulation(n, d, topology="ring", H=0, lr=0.1, momentum=0.0, ld=d + pad)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + d)
    sim.X.normal_(1.0, 1e-3, generator=gen)   # rows close to each other: the distance is the small difference of large sums
    X = sim.X.cpu().numpy().astype(np.float64)
    want, mean = orc.consensus_error(X), X.mean(0)
    # deviations are formed in fp32 (half an ulp of 1e-3 each, of random sign), sums are fp64
    assert abs(sim.consensus_error() - want) <= 1e-7 * want
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    sim.consensus_error_static(out)   # the same partial sums, added in the same order
    assert float(out.item()) == sim.consensus_error()
    assert np.abs(sim.mean().cpu().numpy() - mean).max() <= 6.0e-8 * np.abs(mean).max()   # one rounding to fp32
    sim.close()

"""Circulant sparse W on 225 to 1024 nodes (the static exponential graph, a caller's W): every row-piece width, row
counts that leave waves and passes part empty, ragged rows, several tiles a workgroup; and the pacing of sparse-W
steps whose rows do not divide among the wavefronts."""
import numpy as np
import pytest

from oracle import gpga_oracle as orc
from paper_2105_09080_amd import inputs

pytestmark = pytest.mark.gpu

TOL = 1e-5   # of the array (the step tests' own bound)


@pytest.fixture(scope="module")
def hx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("n,d,pad,momentum,nesterov,custom", [
    (225, 16_384, 0, 0.9, False, False), (256, 16_513, 1, 0.9, True, False), (257, 8193, 0, 0.9, False, False),
    (300, 40_003, 0, 0.0, False, False), (512, 8260, 3, 0.9, False, True), (513, 4097, 0, 0.9, False, False),
    (700, 16_641, 0, 0.9, True, False), (1000, 4102, 1, 0.0, False, True), (1024, 20_000, 0, 0.9, False, False)])
def test_circulant_steps_match_the_oracle(hx, n, d, pad, momentum, nesterov, custom):
    X, M, G = inputs.random_state(n, d, seed=n + d)
    topology, W = ("custom", np.zeros((n, n))) if custom else ("expo", None)
    if custom:   # three far neighbours with different weights, none on the node itself
        for off, w in ((n // 3, 0.5), (n - 5, 0.3), (7 * n // 8, 0.2)):
            W[np.arange(n), (np.arange(n) + off) % n] = w
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=momentum, ld=d + pad)
    if custom:
        sim.set_mixing(W)
    if nesterov:
        sim.set_nesterov(True)
    for buf in sim._bufs:
        buf.fill_(7.0)
    sim.set_state(X=X, M=M, G=G, k=0)
    X_ref, M_ref = X, (M if momentum else np.zeros_like(M))
    for k in range(2):   # both directions of the ping-pong
        sim.step()
        assert (int(sim.query("step_path")), int(sim.query("step_lane_bytes"))) == (10, 16)
        X_ref, M_ref = orc.gossip_pga_step(X_ref, M_ref, G, k, topology=topology, H=0, lr=0.1, momentum=momentum,
                                           nesterov=nesterov, W=W)
    assert np.abs(host(sim.X) - X_ref).max() <= TOL * np.abs(X_ref).max()
    if momentum:
        assert np.abs(host(sim.M) - M_ref).max() <= TOL * np.abs(M_ref).max()
    assert np.array_equal(host(sim.G), G.astype(np.float32))
    for buf in sim._bufs:   # nothing beyond a row's d columns is written
        assert (host(buf)[:, d:] == 7.0).all()
    sim.close()


@pytest.mark.parametrize("n,topology", [(10, "grid"), (50, "expo"), (100, "grid")])
def test_the_pacing_rate_holds_where_rows_do_not_divide_among_wavefronts(hx, n, topology):
    # a controller that takes a launch's own shape for lateness ends at its lower limit (1 TB/s); the memory sustains 4 to 6
    sim = hx.Simulation(n, 540_000_000 // (4 * n), topology=topology, H=0, lr=0.1, momentum=0.9)
    for _ in range(80):
        sim.step()
    assert int(sim.query("step_paced")) == 1
    assert min(sim.query("pace_rate_gbs:tile"), sim.query("pace_rate_gbs:tile/1")) > 2500.0
    sim.close()


@pytest.mark.parametrize("n,d,path", [
    (700, 16_640, 10), (700, 16_656, 6), (700, 16_644, 6), (700, 24_016, 10), (700, 24_001, 6), (600, 24_001, 4), (400, 50_001, 10), (240, 70_002, 10)])
def test_rows_that_straddle_cache_lines_keep_the_other_kernels(hx, n, d, path):
    # 128-byte row pieces (more than 512 nodes) on 128-, 64-, 16- and 4-byte boundaries; wider pieces at any
    X, M, G = inputs.random_state(n, d, seed=n + d)
    sim = hx.Simulation(n, d, topology="expo", H=0, lr=0.1, momentum=0.9)
    sim.set_state(X=X, M=M, G=G, k=0)
    sim.step()
    assert int(sim.query("step_path")) == path
    X_ref, M_ref = orc.gossip_pga_step(X, M, G, 0, topology="expo", H=0, lr=0.1, momentum=0.9)
    assert np.abs(host(sim.X) - X_ref).max() <= TOL * np.abs(X_ref).max()
    assert np.abs(host(sim.M) - M_ref).max() <= TOL * np.abs(M_ref).max()
    sim.close()

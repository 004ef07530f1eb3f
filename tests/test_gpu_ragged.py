"""Rows that no vector width divides: leading dimensions and column counts with every remainder modulo the
16-byte lane, tiles whose last unit stands alone (64 and 16 lanes a tile), every step kernel."""
import numpy as np
import pytest

from oracle import gpga_oracle as orc
from paper_2105_09080_amd import inputs

pytestmark = pytest.mark.gpu

TOL = 1e-5   # of the array: a few fp32 roundings per element (the step tests' own bound)


@pytest.fixture(scope="module")
def hx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


# one unit and a bit, a lone unit behind 64 / 16 whole ones (257, 65), behind 128 and 63, and an aligned width on
# an unaligned leading dimension
WIDTHS = [(3, 3), (4, 5), (5, 5), (6, 7), (7, 7), (65, 65), (66, 66), (255, 255), (256, 257), (257, 257), (258, 259),
          (259, 260), (513, 513), (4099, 4099)]


@pytest.mark.parametrize("d,ld", WIDTHS)
@pytest.mark.parametrize("n,topology,opts", [
    (8, "ring", {}), (40, "ring", {"row_split": 4}), (8, "ring", {"row_split": 1, "blocks_per_cu": 1, "pace_gbs": 4000}),
    (12, "expo1", {}), (8, "none", {}), (9, "full", {}), (64, "full", {"row_lanes": 1}), (40, "full", {"row_lanes": 2}),
    (20, "grid", {}), (20, "grid", {"mix_lane_bytes": 8}), (20, "expo", {"mix_two_pass": 1}), (200, "grid", {}),
    (48, "grid", {"mix_band": 1}), (48, "grid", {"mix_band": 1, "mix_lane_bytes": 8}),
])
def test_step_on_ragged_rows(hx, n, topology, opts, d, ld):
    X, M, G = inputs.random_state(n, d, seed=d + n)
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=0.9, ld=ld)
    for name, v in opts.items():
        sim.set_option(name, v)
    for buf in (*sim._bufs, sim.m, sim.g):
        buf.fill_(7.0)
    sim.set_state(X=X, M=M, G=G, k=0)
    k = 0
    for _ in range(2):   # both directions of the ping-pong
        sim.step()
        X, M = orc.gossip_pga_step(X, M, G, k, topology=topology, H=0, lr=0.1, momentum=0.9)
        k += 1
    for got, want in ((host(sim.X), X), (host(sim.M), M)):
        assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    assert np.array_equal(host(sim.G), G.astype(np.float32))
    for buf in (*sim._bufs, sim.m, sim.g):   # nothing beyond a row's d columns is written
        assert (host(buf)[:, d:] == 7.0).all()
    sim.close()


@pytest.mark.parametrize("n,d,ld,k,opts,momentum,path", [
    (64, 30_003, 30_004, 4, {"cycle_kernel": 1}, 0.9, 2), (64, 30_001, 30_004, 5, {"cycle_kernel": 1}, 0.0, 2),
    (16, 257, 260, 1, {"cycle_kernel": 1, "blocks_per_cu": 1, "pace_gbs": 4000}, 0.9, 2),   # cycles of 8, a lone unit behind whole tiles
    (64, 30_003, 30_003, 4, {"cycle_kernel": 1}, 0.9, 1),                                    # forced: rows on 16-byte boundaries only
    (4, 600_001, 600_001, 1, {}, 0.9, 2), (8, 600_002, 600_007, 1, {}, 0.9, 2)])             # wide: whatever the alignment
def test_row_streaming_kernel_on_ragged_rows(hx, n, d, ld, k, opts, momentum, path):
    X, M, G = inputs.random_state(n, d, seed=d + n)
    sim = hx.Simulation(n, d, topology="expo1", H=0, lr=0.1, momentum=momentum, ld=ld)
    for name, v in opts.items():
        sim.set_option(name, v)
    for buf in (*sim._bufs, *([sim.m] if momentum else [])):
        buf.fill_(7.0)
    sim.set_state(X=X, M=M, G=G, k=k)
    trace = sim.attach_trace(k + 1)
    sim.step()
    assert int(sim.query("step_path")) == path
    X, M = orc.gossip_pga_step(X, M if momentum else np.zeros_like(M), G, k, topology="expo1", H=0, lr=0.1, momentum=momentum)
    assert np.abs(host(sim.X) - X).max() <= TOL * np.abs(X).max()
    if momentum:
        assert np.abs(host(sim.M) - M).max() <= TOL * np.abs(M).max()
    assert float(trace[k]) == pytest.approx(orc.consensus_error(X), rel=TOL)
    for buf in sim._bufs:   # nothing beyond a row's d columns is written
        assert (host(buf)[:, d:] == 7.0).all()
    sim.close()


@pytest.mark.parametrize("n,d,ld,lane_bytes", [
    (400, 501, 501, 4), (400, 504, 505, 4), (400, 501, 504, 16), (8, 36_863, 36_863, 4), (8, 36_865, 36_865, 16), (128, 18_431, 18_431, 4), (130, 18_433, 18_434, 16)])
@pytest.mark.parametrize("topology", ["ring", "full", "none"])
def test_narrow_rows_of_another_alignment_keep_four_byte_lanes(hx, n, d, ld, lane_bytes, topology):
    X, M, G = inputs.random_state(n, d, seed=d + n)
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=0.9, ld=ld)
    sim.set_state(X=X, M=M, G=G, k=0)
    sim.step()
    assert int(sim.query("step_lane_bytes")) == lane_bytes
    X, M = orc.gossip_pga_step(X, M, G, 0, topology=topology, H=0, lr=0.1, momentum=0.9)
    for got, want in ((host(sim.X), X), (host(sim.M), M)):
        assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    sim.close()

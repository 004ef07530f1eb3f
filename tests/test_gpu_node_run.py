"""Small trajectories with four lanes a node: against one kernel per stage and against plain float64 sums, around the
limits of the form (nodes, columns, samples, iterations) and with row numbers outside the data."""
import numpy as np
import pytest

from paper_2105_09080_amd import inputs

pytestmark = pytest.mark.gpu

# Both paths form margins and sums in fp64 and round state to fp32: they may differ where a margin's last bit turns a
# rounding of the coefficient, one ulp (6e-8) an iteration at most, over at most 9 iterations of a contractive problem.
TOL = 9 * 6e-8 * 2


@pytest.fixture(scope="module")
def hx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def run(hx, n, d, B, T, topology, momentum, nesterov, problem, small, bad=False, infinite=False):
    import torch
    M = 30 if B else 3
    feat, y, _ = inputs.logreg_problem(n, d, M, seed=n + d)
    if infinite:
        feat[::2, :, d - 1] = np.inf
    sim = hx.Simulation(n, d, topology=topology, H=3, lr=0.1, momentum=momentum, ld=d + 1)
    if nesterov:
        sim.set_nesterov(True)
    sim.set_option("small_run", small)
    (sim.problem_logreg if problem == "logreg" else sim.problem_lsq)(feat, y)
    idx = inputs.batch_indices(T, n, B, M, seed=3) if B else None
    if bad:
        idx[T // 2, 0, 0] = M
        idx[T // 2, n - 1, B - 1] = -1
    sim.set_state(X=inputs.random_state(n, d, seed=1)[0])
    trace = sim.attach_trace(T)
    sim.run(T, None if idx is None else sim.upload_batches(idx))
    torch.cuda.synchronize()
    assert (int(sim.query("step_path")) == 7) == bool(small)
    out = [t.cpu().numpy().copy() for t in (sim.X, sim.G, trace)] + ([sim.M.cpu().numpy().copy()] if momentum else [])
    sim.close()
    return out


@pytest.mark.parametrize("n,d,B,T,topology", [
    (1, 1, 1, 1, "ring"), (2, 3, 1, 2, "ring"), (16, 12, 1, 3, "expo1"), (17, 13, 2, 4, "grid"), (128, 20, 4, 5, "ring"),
    (127, 20, 3, 9, "expo"), (100, 10, 1, 7, "none"), (30, 5, 0, 6, "full"), (33, 12, 4, 8, "expo1"), (128, 4, 2, 9, "grid")])
@pytest.mark.parametrize("momentum,nesterov,problem", [(0.0, False, "logreg"), (0.9, False, "lsq"), (0.9, True, "logreg")])
def test_small_trajectories_match_one_kernel_per_stage(hx, n, d, B, T, topology, momentum, nesterov, problem):
    a = run(hx, n, d, B, T, topology, momentum, nesterov, problem, 1)
    b = run(hx, n, d, B, T, topology, momentum, nesterov, problem, 0)
    for u, v in zip(a, b):
        scale = np.abs(v).max() if v is not b[2] else np.linalg.norm(b[0])
        assert np.abs(u - v).max() <= TOL * max(scale, 1e-30)


@pytest.mark.parametrize("B", [1, 2, 4])
def test_row_numbers_outside_the_data_give_nan_where_they_did(hx, B):
    a = run(hx, 12, 7, B, 4, "ring", 0.9, False, "logreg", 1, bad=True)
    b = run(hx, 12, 7, B, 4, "ring", 0.9, False, "logreg", 0, bad=True)
    for u, v in zip(a[:2], b[:2]):
        assert np.array_equal(np.isnan(u), np.isnan(v)) and np.isnan(u).any()
        ok = ~np.isnan(v)
        assert not ok.any() or np.abs(u[ok] - v[ok]).max() <= TOL * np.abs(v[ok]).max()


@pytest.mark.parametrize("entries", [18, 20])   # a node: within the LDS of the four-lane form, and beyond it
def test_the_densest_mixing_matrices(hx, entries):
    import torch
    n, d, T = 128, 20, 6
    W = np.zeros((n, n))
    for off in range(entries):
        W[np.arange(n), (np.arange(n) + off * 5) % n] = 1.0 / entries
    feat, y, _ = inputs.logreg_problem(n, d, 30, seed=9)
    out = []
    for small in (1, 0):
        sim = hx.Simulation(n, d, topology="custom", H=4, lr=0.1, momentum=0.9)
        sim.set_mixing(W)
        sim.set_option("small_run", small)
        sim.problem_logreg(feat, y)
        sim.set_state(X=inputs.random_state(n, d, seed=1)[0])
        trace = sim.attach_trace(T)
        sim.run(T, sim.upload_batches(inputs.batch_indices(T, n, 1, 30, seed=3)))
        torch.cuda.synchronize()
        assert (int(sim.query("step_path")) == 7) == bool(small)
        out.append((sim.X.cpu().numpy().copy(), trace.cpu().numpy().copy()))
        sim.close()
    (xa, ta), (xb, tb) = out
    assert np.abs(xa - xb).max() <= TOL * np.abs(xb).max()
    assert np.abs(ta - tb).max() <= TOL * np.linalg.norm(xb)


@pytest.mark.parametrize("d", [1, 5, 10, 12, 18])   # with and without lanes behind the last column
@pytest.mark.parametrize("problem", ["logreg", "lsq"])
def test_an_infinite_last_feature_reaches_its_own_column_only(hx, d, problem):
    a = run(hx, 12, d, 2, 1, "none", 0.9, False, problem, 1, infinite=True)
    b = run(hx, 12, d, 2, 1, "none", 0.9, False, problem, 0, infinite=True)
    for u, v in zip(a[:2], b[:2]):
        assert np.array_equal(u, v, equal_nan=True) or np.allclose(u, v, rtol=TOL, atol=TOL * np.abs(v[np.isfinite(v)]).max(), equal_nan=True)


@pytest.mark.parametrize("d", [2, 4, 6, 8, 11, 14, 16, 17, 19])   # lanes whose columns overlap the lane before by none, some, all
@pytest.mark.parametrize("B,topology", [(1, "ring"), (2, "full"), (3, "expo1")])
def test_rows_that_the_lanes_columns_do_not_divide(hx, d, B, topology):
    a = run(hx, 20, d, B, 5, topology, 0.9, False, "logreg", 1)
    b = run(hx, 20, d, B, 5, topology, 0.9, False, "logreg", 0)
    for u, v in zip(a, b):
        scale = np.abs(v).max() if v is not b[2] else np.linalg.norm(b[0])
        assert np.abs(u - v).max() <= TOL * max(scale, 1e-30)


@pytest.mark.parametrize("n,d", [(1, 3), (15, 4), (16, 10), (17, 16), (32, 20), (33, 13), (63, 12), (64, 4), (65, 10), (128, 12), (128, 20)])
def test_the_trace_on_every_number_of_row_batches(hx, n, d):
    a = run(hx, n, d, 1, 7, "ring", 0.0, False, "logreg", 1)
    b = run(hx, n, d, 1, 7, "ring", 0.0, False, "logreg", 0)
    assert np.abs(a[2] - b[2]).max() <= TOL * np.linalg.norm(b[0]) and np.abs(a[0] - b[0]).max() <= TOL * np.abs(b[0]).max()


@pytest.mark.parametrize("d", [7, 20, 21])   # 21 columns: the general single-workgroup kernel
def test_the_trace_of_a_state_that_is_not_a_number_is_not_zero(hx, d):
    # rows outside the data at iteration 2 make two nodes NaN; it ends in a global average (H = 3), whose entry is 0
    trace = run(hx, 12, d, 1, 5, "ring", 0.9, False, "logreg", 1, bad=True)[2]
    assert np.isfinite(trace[:2]).all() and (trace[:2] > 0).all() and trace[2] == 0.0 and np.isnan(trace[3:]).all()


@pytest.mark.parametrize("n,d,ld", [(1, 1, 1), (3, 3, 4), (5, 4, 5), (40, 7, 7), (33, 257, 257), (32, 1000, 1001), (200, 1031, 1031),
                                    (4, 300_002, 300_003), (64, 262_147, 262_147), (3, 1_048_577, 1_048_577)])
def test_distance_and_mean_on_every_split(hx, n, d, ld):
    import torch
    sim = hx.Simulation(n, d, topology="ring", H=0, lr=0.1, ld=ld)
    sim.set_state(X=inputs.random_state(n, d, seed=d)[0] + 3.0)
    X = sim.X.double()
    mean, dist = X.mean(0), float((X - X.mean(0)).norm())
    # float32 rounding of the mean; the distance is a sum of squares of deviations from row 0 rounded to fp32
    assert float((sim.mean().double() - mean).abs().max()) <= 6e-8 * float(mean.abs().max())
    assert sim.consensus_error() == pytest.approx(dist, rel=3e-7, abs=1e-12)
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    sim.consensus_error_static(out)
    assert float(out.item()) == sim.consensus_error()
    x0 = torch.arange(d, dtype=torch.float32, device="cuda")
    from paper_2105_09080_amd import binding as B
    B.gpga_reset(sim.ctx, x0)
    assert torch.equal(sim.X, x0.expand(n, d))
    sim.close()

"""gpga_run on stored features with gradient sums, update and mixing in one launch, against separate calls: node counts,
widths and batches around the tiles and the splits, ragged rows, every graph, row numbers outside the data."""
import numpy as np
import pytest

from paper_2105_09080_amd import inputs

pytestmark = pytest.mark.gpu

# g is an fp64 sum rounded to fp32 on both sides; another order of that sum turns a rounding now and then: one ulp of a
# gradient, carried through T <= 4 contractive iterations.
TOL = 4 * 1.2e-7


@pytest.fixture(scope="module")
def hx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def make(hx, n, d, M, B, T, topology, H, momentum, problem, ld, bad=False):
    feat, y, _ = inputs.logreg_problem(n, d, M, seed=n + d)
    sim = hx.Simulation(n, d, topology=topology, H=H, lr=0.1, momentum=momentum, ld=ld)
    sim.set_option("small_run", 0)
    (sim.problem_logreg if problem == "logreg" else sim.problem_lsq)((feat / np.sqrt(d)).astype(np.float32), y)
    idx = inputs.batch_indices(T, n, B, M, seed=3) if B else None
    if bad:
        idx[T - 1, 0, 0], idx[T - 1, n - 1, B - 1] = M, -1
    for buf in (*sim._bufs, sim.g):
        buf.fill_(7.0)
    sim.set_state(X=inputs.random_state(n, d, seed=1)[0])
    return sim, None if idx is None else sim.upload_batches(idx)


def results(sim, momentum):
    out = [t.cpu().numpy().astype(np.float64) for t in (sim.X, sim.G)] + ([sim.M.cpu().numpy().astype(np.float64)] if momentum else [])
    edge = [b[:, sim.d:].cpu().numpy() for b in (*sim._bufs, sim.g)]
    return out, edge


@pytest.mark.parametrize("n,d,M,B,topology,H,momentum,problem,pad", [
    (1, 4, 5, 1, "ring", 2, 0.9, "logreg", 0), (2, 17, 9, 0, "ring", 0, 0.0, "lsq", 1), (8, 1003, 40, 6, "expo1", 4, 0.9, "logreg", 0),
    (128, 40, 30, 33, "grid", 3, 0.9, "lsq", 0), (5, 1001, 900, 0, "expo", 4, 0.9, "logreg", 2), (33, 2052, 20, 9, "none", 2, 0.0, "logreg", 0),
    (32, 4099, 20, 32, "expo1", 3, 0.9, "logreg", 0), (12, 16_389, 12, 17, "ring", 4, 0.9, "lsq", 3), (60, 32_771, 4, 3, "grid", 3, 0.9, "logreg", 0),
    (9, 257, 1000, 0, "full", 0, 0.9, "lsq", 0), (64, 1028, 70, 65, "ring", 2, 0.9, "logreg", 0), (100, 20_001, 4, 2, "expo", 3, 0.0, "lsq", 0)])
def test_one_launch_matches_separate_calls(hx, n, d, M, B, topology, H, momentum, problem, pad):
    import torch
    T = 4
    a, idx_a = make(hx, n, d, M, B, T, topology, H, momentum, problem, d + pad)
    b, idx_b = make(hx, n, d, M, B, T, topology, H, momentum, problem, d + pad)
    ta, tb = a.attach_trace(T), b.attach_trace(T)
    a.run(T, idx_a)
    assert int(a.query("step_path")) == 9
    for k in range(T):
        b.local_grad(None if idx_b is None else idx_b[k])
        b.step()
    torch.cuda.synchronize()
    (ra, edge), (rb, _) = results(a, momentum), results(b, momentum)
    for u, v in zip(ra, rb):
        assert np.abs(u - v).max() <= TOL * np.abs(v).max()
    assert torch.allclose(ta, tb, rtol=1e-6, atol=1e-6 * float(np.linalg.norm(rb[0])))
    for e in edge:
        assert (e == 7.0).all()   # nothing beyond a row's d columns is written
    a.close(), b.close()


@pytest.mark.parametrize("n,d,M,one_launch", [
    (100, 10, 8000, False), (128, 40, 300, False), (128, 40, 32, True), (32, 256, 200, False), (8, 1000, 1000, True), (8, 5000, 1000, False)])
def test_large_batches_on_many_nodes_keep_a_workgroup_per_node(hx, n, d, M, one_launch):
    # full batches: one launch would leave the samples of all nodes to the few workgroups that the columns make
    import torch
    sim, _ = make(hx, n, d, M, 0, 2, "ring", 0, 0.9, "lsq", d)
    ref, _ = make(hx, n, d, M, 0, 2, "ring", 0, 0.9, "lsq", d)
    sim.run(2)
    assert (int(sim.query("step_path")) == 9) == one_launch
    for _ in range(2):
        ref.local_grad()
        ref.step()
    torch.cuda.synchronize()
    for u, v in zip(results(sim, 0.9)[0], results(ref, 0.9)[0]):
        assert np.abs(u - v).max() <= TOL * np.abs(v).max()
    sim.close(), ref.close()


def test_rows_outside_the_data_poison_their_node_only(hx):
    import torch
    a, idx = make(hx, 8, 1000, 50, 9, 1, "none", 0, 0.9, "logreg", 1000, bad=True)
    a.run(1, idx)
    torch.cuda.synchronize()
    assert int(a.query("step_path")) == 9
    nan = torch.isnan(a.G).cpu().numpy()
    assert nan[0].all() and nan[7].all() and not nan[1:7].any()
    a.close()


def test_an_explicit_zero_weight_carries_what_is_not_a_number(hx):
    # entries of W that are there with weight 0: one launch multiplies them as the step kernels do, and no padding besides
    import torch
    from paper_2105_09080_amd import binding
    n, d, M = 6, 40, 12
    rows = [[(i, 0.75), ((i + 1) % n, 0.25)] + ([((i + 3) % n, 0.0)] if i == 2 else []) for i in range(n)]
    ptr = np.cumsum([0] + [len(r) for r in rows])
    col, val = [j for r in rows for j, _ in r], [w for r in rows for _, w in r]
    out = []
    for fused in (True, False):
        sim, idx = make(hx, n, d, M, 4, 1, "custom", 0, 0.9, "lsq", d)
        binding.gpga_set_mixing_csr(sim.ctx, ptr, col, val)
        x = inputs.random_state(n, d, seed=1)[0]
        x[5, 7] = np.nan
        sim.set_state(X=x)
        if fused:
            sim.run(1, idx)
        else:
            sim.local_grad(idx[0])
            sim.step()
        torch.cuda.synchronize()
        assert (int(sim.query("step_path")) == 9) == fused
        out.append(torch.isnan(sim.X).cpu().numpy())
        sim.close()
    assert np.array_equal(out[0], out[1]) and out[0][2].any() and not out[0][1].any()


def test_launch_overrides_and_large_states_keep_the_step_kernels(hx):
    a, idx = make(hx, 8, 1000, 50, 9, 2, "ring", 0, 0.9, "logreg", 1000)
    a.set_option("unroll", 2)
    a.run(2, idx)
    assert int(a.query("step_path")) == 1
    a.close()
    a, idx = make(hx, 129, 64, 5, 3, 2, "ring", 0, 0.9, "logreg", 64)
    a.run(2, idx)
    assert int(a.query("step_path")) == 1
    a.close()


@pytest.mark.parametrize("d", [3, 5, 63, 65, 130, 255, 256, 257, 258])   # one column or four a lane of the accumulate pass
@pytest.mark.parametrize("M", [7, 64])                                   # 4 or 16 wavefronts
def test_gradients_of_ragged_rows(hx, d, M):
    import torch
    n = 3
    feat, y, _ = inputs.logreg_problem(n, d, M, seed=d)
    X = inputs.random_state(n, d, seed=1)[0]
    sim = hx.Simulation(n, d, topology="ring", H=0, lr=0.1, ld=d + 1)
    sim.problem_lsq(feat, y)
    sim.g.fill_(7.0)
    sim.set_state(X=X)
    sim.local_grad()
    torch.cuda.synchronize()
    F, t = feat.astype(np.float64), y.astype(np.float64)
    res = np.einsum("nmd,nd->nm", F, X.astype(np.float32).astype(np.float64)) - t
    ref = np.einsum("nm,nmd->nd", res, F) / M
    # a coefficient and a sum are rounded to fp32 once each
    bound = 2 * 6e-8 * np.einsum("nm,nmd->nd", np.abs(res), np.abs(F)) / M + 6e-8 * np.abs(ref)
    assert (np.abs(sim.G.cpu().numpy() - ref) <= bound).all() and (sim.g[:, d:].cpu().numpy() == 7.0).all()
    sim.close()

"""gpga_run on stored features with several iterations a launch, against separate calls: slices and samples around the
registers that hold them, ragged rows, every graph, adaptive periods, launches that are given up, streams and threads."""
import threading

import numpy as np
import pytest

from paper_2105_09080_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# Margins and g are fp64 sums rounded to fp32 on both sides; another order of a sum turns a rounding now and then: one ulp,
# carried through a few contractive iterations (features of unit length, step size 0.1).
TOL = 4 * 1.2e-7


@pytest.fixture(scope="module")
def hx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def make(hx, n, d, M, batch, T, topology, H, momentum, problem="logreg", pad=0, nesterov=False, lr=0.1, stream=None, feat=None):
    rng = np.random.default_rng([n, d, M])
    if feat is None:
        feat = (rng.standard_normal((n, M, d)) / np.sqrt(d)).astype(np.float32)
    y = np.where(rng.random((n, M)) < 0.5, 1.0, -1.0).astype(np.float32)
    sim = hx.Simulation(n, d, topology=topology, H=H, lr=lr, momentum=momentum, ld=d + pad, stream=stream)
    if nesterov:
        sim.set_nesterov(True)
    sim.set_option("small_run", 0)
    (sim.problem_logreg if problem == "logreg" else sim.problem_lsq)(feat, y)
    idx = sim.upload_batches(inputs.batch_indices(T, n, batch, M, seed=3)) if batch else None
    for buf in (*sim._bufs, sim.g):
        buf.fill_(7.0)
    sim.set_state(X=inputs.random_state(n, d, seed=1)[0], M=inputs.random_state(n, d, seed=2)[0] if momentum else None)
    return sim, idx


def separate(sim, idx, T):
    for k in range(T):
        sim.local_grad(None if idx is None else idx[k])
        sim.step()


def results(sim, momentum):
    torch.cuda.synchronize()
    return [t.cpu().numpy().astype(np.float64) for t in (sim.X, sim.G, *((sim.M,) if momentum else ()))]


def assert_alike(ra, rb):
    for u, v in zip(ra, rb):
        assert np.abs(u - v).max() <= TOL * np.abs(v).max()


SHAPES = [  # rows of a thread and what holds them; slices of a node
    (4, 36, 6, 1, 5, "ring", 2, 0.9, "logreg", 0),        # one row, part of a wavefront
    (16, 257, 40, 9, 6, "expo1", 4, 0.9, "logreg", 1),    # a ragged last quad of one column
    (12, 1022, 40, 33, 4, "grid", 3, 0.9, "lsq", 0),      # ... of two
    (9, 3003, 40, 24, 5, "expo", 4, 0.0, "logreg", 3),    # ... of three; slices that are no power of two
    (128, 515, 30, 8, 3, "expo", 2, 0.9, "logreg", 0),    # most nodes, eight neighbours
    (32, 5121, 20, 32, 3, "ring", 0, 0.9, "logreg", 0),   # a column more than the wavefronts of a slice
    (20, 9999, 24, 40, 3, "expo1", 3, 0.9, "lsq", 0),     # many rows a thread
    (32, 5120, 20, 50, 3, "ring", 2, 0.9, "logreg", 0),   # the most
    (8, 1000, 100, 0, 7, "ring", 4, 0.0, "lsq", 0),       # full batches in double precision
    (30, 1002, 130, 0, 4, "none", 3, 0.9, "lsq", 0),      # full batches in single precision
    (64, 130, 12, 0, 40, "ring", 16, 0.9, "logreg", 0),   # more than one launch
    (5, 64, 30, 20, 6, "full", 0, 0.9, "logreg", 0),
]


@pytest.mark.parametrize("given_up", [False, True])
@pytest.mark.parametrize("n,d,M,batch,T,topology,H,momentum,problem,pad", SHAPES)
def test_several_iterations_a_launch_match_separate_calls(hx, n, d, M, batch, T, topology, H, momentum, problem, pad, given_up):
    a, idx_a = make(hx, n, d, M, batch, T, topology, H, momentum, problem, pad, nesterov=n == 16)
    b, idx_b = make(hx, n, d, M, batch, T, topology, H, momentum, problem, pad, nesterov=n == 16)
    if given_up:
        a.set_option("run_wait_us", 0)   # the first wait that is not met at once ends the launch; one workgroup does it again
    a.run(T, idx_a)
    assert int(a.query("step_path")) == 12 and a.k == T
    assert (a.query("run_given_up") > 0) == given_up
    separate(b, idx_b, T)
    assert_alike(results(a, momentum), results(b, momentum))
    for e in (*a._bufs, a.g):
        assert (e[:, d:].cpu().numpy() == 7.0).all()   # nothing beyond a row's d columns is written
    assert [t.data_ptr() for t in a._bufs].index(a.X.data_ptr()) == T % 2
    a.close(), b.close()


@pytest.mark.parametrize("given_up", [False, True])
@pytest.mark.parametrize("n,d,M,batch,T,topology,H,warmup,most", [
    (16, 512, 64, 8, 60, "expo1", 2, 8, 12), (9, 1203, 33, 0, 41, "expo", 2, 6, 20), (70, 301, 40, 5, 50, "grid", 3, 4, 9)])
def test_adaptive_period_decided_in_the_launch(hx, n, d, M, batch, T, topology, H, warmup, most, given_up):
    out = []
    for fused in (True, False):
        sim, idx = make(hx, n, d, M, batch, T, topology, 0, 0.9, "lsq" if not batch else "logreg", lr=0.5)
        sim.aga_enable(H, warmup, most)
        if given_up:
            sim.set_option("run_wait_us", 0)
        if fused:
            sim.run(T // 2, idx)
            periods = [sim.period]
            sim.run(T - T // 2, None if idx is None else idx[T // 2:])
            assert int(sim.query("step_path")) == 12
            assert (sim.query("run_given_up") > 0) == given_up
        else:
            for k in range(T):
                i = None if idx is None else idx[k]
                loss = sim.local_loss(i)
                sim.local_grad(i)
                sim.aga_step(loss)
                if k == T // 2 - 1:
                    periods = [sim.period]
        out.append((results(sim, 0.9), periods + [sim.period]))
        sim.close()
    assert out[0][1] == out[1][1]
    # sums of losses decide nothing here but the period: the same bound, over more iterations
    for u, v in zip(out[0][0], out[1][0]):
        assert np.abs(u - v).max() <= 4 * TOL * np.abs(v).max()


@pytest.mark.parametrize("given_up", [False, True])
@pytest.mark.parametrize("n,d,batch", [(100, 64, 1), (9, 222, 32), (12, 33, 7), (64, 128, 2)])
def test_averages_of_small_problems_are_formed_in_double_precision(hx, n, d, batch, given_up):
    """Without a step every iterate stays as it is until the average: columns whose rows cancel to 1e-6 of their size.  What
    remains is one rounding to single precision, and the rounding of fp64 sums of up to 100 rows 1e6 times the mean: 1e-8."""
    sim, idx = make(hx, n, d, 40, batch, 4, "none", 4, 0.0, lr=0.0)
    sim.set_option("small_run", 1)
    if given_up:
        sim.set_option("run_wait_us", 0)
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, d)).astype(np.float32) * 1e4
    x[n // 2:2 * (n // 2)] = -x[:n // 2]
    x[n - 1] += rng.standard_normal(d).astype(np.float32)
    if n % 2:
        x[n - 1] *= 1e-4
    sim.set_state(X=x)
    sim.run(4, idx)
    torch.cuda.synchronize()
    assert int(sim.query("step_path")) == 12 and (sim.query("run_given_up") > 0) == given_up
    want = x.astype(np.float64).mean(0)
    got = sim.X.cpu().numpy().astype(np.float64)
    assert (np.abs(got - want) <= (2.0 ** -24 + 1e-8) * np.abs(want)).all()
    sim.close()


@pytest.mark.parametrize("last", [False, True])   # workgroup 0 or 255 modulo their number, when the others have stored what they have
@pytest.mark.parametrize("T", [5, 6])
@pytest.mark.parametrize("n,d,M,batch,topology,H,momentum,adaptive", [
    (16, 257, 40, 9, "ring", 4, 0.9, False), (8, 1000, 100, 0, "expo1", 3, 0.0, False), (9, 1203, 33, 8, "expo", 2, 0.9, True),
    (20, 1001, 40, 16, "grid", 2, 0.0, True), (32, 5120, 20, 32, "ring", 0, 0.9, False)])
def test_a_launch_given_up_at_its_end_is_done_again_from_its_beginning(hx, n, d, M, batch, topology, H, momentum, adaptive, T, last):
    out = []
    for fused in (True, False):
        sim, idx = make(hx, n, d, M, batch, T, topology, 0 if adaptive else H, momentum)
        if adaptive:
            sim.aga_enable(H, 2, 9)
        sim.set_option("rows_run", int(fused))
        if fused:
            from paper_2105_09080_amd import binding as B
            for value in (-2, 256):
                with pytest.raises(B.GpgaError):
                    sim.set_option("run_give_up", value)
            sim.set_option("run_give_up", 255 if last else 0)
        sim.run(T, idx)
        assert sim.query("run_given_up") == int(fused) and sim.k == T
        assert int(sim.query("step_path")) == (12 if fused else 9)
        out.append((results(sim, momentum), sim.period))
        sim.close()
    assert out[0][1] == out[1][1]
    assert_alike(out[0][0], out[1][0])


def test_launches_that_are_given_up_again_and_again_are_left_alone_for_a_while(hx):
    T = 6
    sim, idx = make(hx, 16, 1000, 40, 8, T, "ring", 4, 0.9)
    ref, ref_idx = make(hx, 16, 1000, 40, 8, T, "ring", 4, 0.9)
    ref.set_option("rows_run", 0)
    sim.set_option("run_wait_us", 0)
    paths = []
    for call in range(6):
        if call == 4:
            sim.set_option("run_wait_us", 100000)
            sim.set_option("rows_run", 1)
        sim.run(T, idx)
        ref.run(T, ref_idx)
        torch.cuda.synchronize()
        paths.append(int(sim.query("step_path")))
    assert paths == [12, 12, 9, 9, 12, 12] and sim.query("run_given_up") == 2
    for u, v in zip(results(sim, 0.9), results(ref, 0.9)):
        assert np.abs(u - v).max() <= 6 * TOL * np.abs(v).max()
    sim.close(), ref.close()


def test_rows_outside_the_data_poison_their_node_only(hx):
    n, d, T = 8, 1001, 3
    sim, _ = make(hx, n, d, 50, 9, T, "none", 0, 0.9)
    idx = inputs.batch_indices(T, n, 9, 50, seed=3)
    idx[0, 0, 0], idx[T - 1, n - 1, 8] = 50, -1
    sim.run(T, sim.upload_batches(idx))
    torch.cuda.synchronize()
    assert int(sim.query("step_path")) == 12
    nan = torch.isnan(sim.G).cpu().numpy()
    assert nan[0].all() and nan[7].all() and not nan[1:7].any()
    sim.close()


def test_infinite_features_and_iterates_as_in_separate_calls(hx):
    n, d, M, T = 6, 331, 12, 3
    rng = np.random.default_rng(5)
    feat = (rng.standard_normal((n, M, d)) / np.sqrt(d)).astype(np.float32)
    feat[1, :, d - 1] = np.inf      # the last column of a ragged width
    feat[3, 2, 170] = -np.inf
    out = []
    for fused in (True, False):
        sim, idx = make(hx, n, d, M, 5, T, "none", 0, 0.0, feat=feat)
        x = inputs.random_state(n, d, seed=1)[0]
        x[4, 7] = np.inf
        sim.set_state(X=x)
        if fused:
            sim.run(T, idx)
            assert int(sim.query("step_path")) == 12
        else:
            separate(sim, idx, T)
        torch.cuda.synchronize()
        out.append((sim.X.cpu().numpy(), sim.G.cpu().numpy()))
        sim.close()
    for u, v in zip(*out):
        assert np.array_equal(np.isnan(u), np.isnan(v)) and np.array_equal(np.isinf(u), np.isinf(v))


def test_two_streams_and_threads(hx):
    # a launch that is under way in one stream leaves the other one iteration a launch; each keeps its own order and results
    T, rounds = 6, 12
    sims = []
    for s in range(2):
        sim, idx = make(hx, 32, 4000, 40, 16, T, ("ring", "expo1")[s], 4, 0.9, stream=torch.cuda.Stream())
        ref, ref_idx = make(hx, 32, 4000, 40, 16, T, ("ring", "expo1")[s], 4, 0.9)
        sims.append((sim, idx, ref, ref_idx))
    torch.cuda.synchronize()

    def work(sim, idx):
        for _ in range(rounds):
            sim.run(T, idx)

    threads = [threading.Thread(target=work, args=s[:2]) for s in sims]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for sim, idx, ref, ref_idx in sims:
        assert int(sim.query("step_path")) in (9, 12)
        sim.run(T, idx)                      # nothing is under way
        torch.cuda.synchronize()
        assert int(sim.query("step_path")) == 12
        ref.set_option("rows_run", 0)
        for _ in range(rounds + 1):
            ref.run(T, ref_idx)
        assert int(ref.query("step_path")) == 9
        ra, rb = results(sim, 0.9), results(ref, 0.9)
        for u, v in zip(ra, rb):
            assert np.abs(u - v).max() <= (rounds + 1) * TOL * np.abs(v).max()
        sim.close(), ref.close()


def test_contexts_in_turn_exchange_through_one_memory(hx):
    """Nothing is waited for between calls: words of other contexts and launches lie where a launch's own go, and the memory grows
    while launches that use it are under way."""
    shapes = [(8, 1000, 24, 16, "ring", 0.9), (20, 333, 24, 8, "expo", 0.0), (4, 36, 24, 5, "expo1", 0.9), (64, 700, 24, 12, "grid", 0.9),
              (32, 5120, 20, 32, "ring", 0.9), (8, 1001, 24, 0, "full", 0.0)]
    T, rounds = 4, 3
    sims = [make(hx, n, d, M, batch, T, topology, 2, momentum) for n, d, M, batch, topology, momentum in shapes]
    refs = [make(hx, n, d, M, batch, T, topology, 2, momentum) for n, d, M, batch, topology, momentum in shapes]
    for _ in range(rounds):
        for sim, idx in sims:
            sim.run(T, idx)
            assert int(sim.query("step_path")) == 12
    for (sim, _), (ref, idx), shape in zip(sims, refs, shapes):
        ref.set_option("rows_run", 0)
        for _ in range(rounds):
            ref.run(T, idx)
        for u, v in zip(results(sim, shape[-1]), results(ref, shape[-1])):
            assert np.abs(u - v).max() <= rounds * TOL * np.abs(v).max()
        sim.close(), ref.close()


def busy(stream):
    """Some 100 ms of other work in the stream: one wavefront."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(1e7))


def test_no_call_waits_for_another_streams_work(hx):
    sims = [make(hx, 8, 1000, 40, 16, 6, ("ring", "expo1")[s], 4, 0.9, stream=torch.cuda.Stream()) for s in range(2)]
    (a, idx_a), (b, idx_b) = sims
    ref, ref_idx = make(hx, 8, 1000, 40, 16, 6, "expo1", 4, 0.9)
    ref.set_option("rows_run", 0)
    b.run(6, idx_b)
    ref.run(6, ref_idx)
    torch.cuda.synchronize()
    a.run(6, idx_a)
    busy(a.stream)
    b.run(6, idx_b)                          # whether the other launch has ended or not
    b.stream.synchronize()
    assert not a.stream.query()
    ref.run(6, ref_idx)
    torch.cuda.synchronize()
    a.run(6, idx_a)
    a.stream.synchronize()
    busy(a.stream)
    b.run(6, idx_b)                          # it has
    assert int(b.query("step_path")) == 12
    b.stream.synchronize()
    assert not a.stream.query()
    ref.run(6, ref_idx)
    for u, v in zip(results(b, 0.9), results(ref, 0.9)):
        assert np.abs(u - v).max() <= 3 * TOL * np.abs(v).max()
    ref.close(), a.close(), b.close()


def test_a_launch_under_way_in_another_stream_leaves_one_iteration_a_launch(hx):
    a, idx_a = make(hx, 32, 4000, 40, 16, 32, "ring", 4, 0.9, stream=torch.cuda.Stream())
    small = [make(hx, 9, 222, 40, 16, 32, "ring", 4, 0.9, stream=torch.cuda.Stream()) for _ in range(2)]
    large = [make(hx, 20, 1001, 40, 16, 32, "expo", 4, 0.9, stream=torch.cuda.Stream()) for _ in range(2)]
    for sim, _ in small:
        sim.set_option("small_run", 1)
    torch.cuda.synchronize()
    for (b, idx_b), (ref, ref_idx), path in ((*small, 7), (*large, 9)):
        for _ in range(80):                  # 80 x 32 iterations: some 20 ms
            a.run(32, idx_a)
        b.run(32, idx_b)
        assert int(b.query("step_path")) == path and not a.stream.query()
        torch.cuda.synchronize()
        assert int(a.query("step_path")) == 12
        ref.run(32, ref_idx)
        assert int(ref.query("step_path")) == 12
        for u, v in zip(results(b, 0.9), results(ref, 0.9)):
            assert np.abs(u - v).max() <= 4 * TOL * np.abs(v).max()
        b.close(), ref.close()
    a.close()


def loaded_hip():
    import ctypes
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1
    return ctypes.CDLL(paths.pop())


@pytest.mark.parametrize("how", ["not ready", "invalid"])
def test_an_error_that_another_call_left_is_not_the_launchs_own(hx, how):
    import ctypes
    hip = loaded_hip()
    sim, idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9)
    ref, ref_idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9)
    ref.set_option("rows_run", 0)
    ref.run(4, ref_idx)
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    if how == "not ready":
        busy(other)
        assert hip.hipStreamQuery(ctypes.c_void_p(other.cuda_stream)) == 600
    else:
        assert hip.hipSetDevice(1000) != 0
    sim.run(4, idx)
    hip.hipGetLastError()
    assert int(sim.query("step_path")) == 12 and sim.k == 4
    torch.cuda.synchronize()
    assert_alike(results(sim, 0.9), results(ref, 0.9))
    sim.close(), ref.close()


def test_iterations_without_an_average_do_not_wait_under_an_adaptive_period(hx):
    T = 6
    out = []
    for fused in (True, False):
        sim, idx = make(hx, 16, 512, 64, 8, 5 * T, "expo1", 0, 0.9, stream=torch.cuda.Stream(), lr=0.5)
        sim.set_option("rows_run", int(fused))
        sim.aga_enable(T + 1, 4 * T, 16)
        sim.run(T, idx)                      # sizes the scratch; the average is the next iteration
        sim.run(T, idx[T:])                  # ... and then T - 1 without
        torch.cuda.synchronize()
        assert int(sim.query("step_path")) == (12 if fused else 9)
        busy(sim.stream)
        sim.run(1, idx[2 * T:])
        assert not sim.stream.query()
        sim.aga_enable(2 * T + 1, 4 * T, 16)
        sim.run(T, idx[2 * T:])
        sim.run(T, idx[3 * T:])
        assert not sim.stream.query()
        sim.run(T, idx[4 * T:])              # its first iteration averages
        if not fused:
            assert sim.stream.query()
        torch.cuda.synchronize()
        out.append((results(sim, 0.9), sim.period))
        sim.close()
    assert out[0][1] == out[1][1]
    for u, v in zip(out[0][0], out[1][0]):
        assert np.abs(u - v).max() <= 4 * TOL * np.abs(v).max()


def test_binding_another_stream_within_a_capture(hx):
    from paper_2105_09080_amd import binding as B
    stream, fork = torch.cuda.Stream(), torch.cuda.Stream()
    sim, idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9, stream=stream)
    ref, ref_idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9)
    for s, i in ((ref, ref_idx), (sim, idx)):
        s.set_option("rows_run", 0)
        s.run(4, i)                          # sizes the scratch
        s.set_option("rows_run", 1)
        s.run(4, i)
        assert int(s.query("step_path")) == 12
        torch.cuda.synchronize()             # so that none is under way in the other stream
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        fork.wait_stream(stream)
        B.gpga_bind(sim.ctx, sim._bufs[0], sim._bufs[1], sim.m, sim.g, sim.ld, fork.cuda_stream)
        sim.run(4, idx)
        stream.wait_stream(fork)
    for _ in range(3):
        graph.replay()
        ref.run(4, ref_idx)
    torch.cuda.synchronize()
    assert_alike(results(sim, 0.9), results(ref, 0.9))
    sim.close(), ref.close()


def test_a_captured_run_keeps_its_launches_per_iteration(hx):
    stream = torch.cuda.Stream()
    sim, idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9, stream=stream)
    ref, ref_idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9)
    with torch.cuda.stream(stream):
        sim.run(4, idx)                      # sizes the scratch
        assert int(sim.query("step_path")) == 12
        sim.set_option("rows_run", 0)
        sim.run(4, idx)
        sim.set_option("rows_run", 1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.run(4, idx)
        assert int(sim.query("step_path")) == 9
        for _ in range(3):
            graph.replay()
    torch.cuda.synchronize()
    for _ in range(5):
        ref.run(4, ref_idx)
    assert_alike(results(sim, 0.9), results(ref, 0.9))
    sim.close(), ref.close()


@pytest.mark.parametrize("n,d,batch,T,H,entries,path", [
    (104, 2000, 1, 3, 1, 0, 9),       # an average in every one of three iterations
    (104, 2000, 1, 16, 0, 0, 12),
    (64, 2000, 2, 8, 0, 64, 9),       # W of 64 entries a row: as many words an iteration and column
    (64, 2000, 2, 8, 0, 3, 12),
    (20, 333, 16, 33, 4, 0, 12),      # 32 iterations a launch: none is left over by itself
    (24, 145, 21, 33, 16, 0, 12),
])
def test_runs_take_the_form_that_measured_faster(hx, n, d, batch, T, H, entries, path):
    out = []
    for rows_run in (1, 0):
        sim, idx = make(hx, n, d, 40, batch, T, "ring", H, 0.9)
        sim.set_option("small_run", 1)
        sim.set_option("rows_run", rows_run)
        if entries:
            sim.set_mixing(sum(np.roll(np.eye(n), o, 1) for o in range(entries)) / entries)
        sim.run(T, idx)
        assert int(sim.query("step_path")) == path or not rows_run
        out.append(results(sim, 0.9))
        sim.close()
    for u, v in zip(*out):
        assert np.abs(u - v).max() <= 4 * TOL * np.abs(v).max()


def test_options_and_traces_keep_one_iteration_a_launch(hx):
    sim, idx = make(hx, 16, 1000, 40, 8, 4, "ring", 0, 0.9)
    sim.set_option("rows_run", 0)
    sim.run(4, idx)
    assert int(sim.query("step_path")) == 9
    sim.set_option("rows_run", 1)
    sim.attach_trace(8)
    sim.run(4, idx)
    assert int(sim.query("step_path")) == 9
    from paper_2105_09080_amd import binding as B
    for name, value in (("rows_run", 2), ("run_wait_us", -1)):
        with pytest.raises(B.GpgaError):
            sim.set_option(name, value)
    sim.close()

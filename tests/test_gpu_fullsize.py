"""Parity at the benchmark's full sizes, in the launch configuration bench.py times.

* cfg3 / cfg4 shapes: ONE fused step per kernel variant compared with the oracle on
  EVERY element (all n x d of X and M), in column chunks: the paced ring walk, the
  paced one-peer walk over long cycles, the row-streaming kernel over cycles of 16,
  8, 4 and 2 rows and the global average.  The oracle's step needs no random numbers
  (it is advanced from the GPU's own X, M, G), so a chunk is a few BLAS calls.
* cfg5 at its full shape (n = 1024, d = 10^6, virtual features), H = 8, 2H + 1 steps
  per topology, every step in lock-step: complete gradient rows of eight nodes spread
  over 0..1023 against the oracle's regenerated features, the fused step on column
  slabs of all rows, the consensus distance on those slabs.
* a cfg5 replica (d = 4096, M = 64) at the STATED step size 0.05, the whole H sweep on
  both graphs: T = 1000 GPU steps with lock-step checks at a sample of steps spread over
  the whole run, and a free-running comparison (with the oracle's own fp32-storage
  against all-float64 distance beside it) over the first 72 steps.
* the sparse-W kernels (whole tile, sliding window, two passes) in the launch configurations
  large problems get: every element of one step on 1.0-1.6e9 elements.
* the same replica under Gossip-AGA (Algorithm 2): 96 iterations in lock-step, minibatch
  losses, period decisions and states against the oracle's.
"""
import math
import queue
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
from scipy.special import expit
from threadpoolctl import threadpool_limits

from oracle import gpga_oracle as orc
from paper_2105_09080_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL_STEP = 1e-5
TOL_FINAL = 1e-4


@pytest.fixture(scope="module")
def hx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2105_09080_amd import harness
    return harness


def rel_errors(got, ref):
    scale_max = max(np.abs(ref).max(), 1e-300)
    scale_f = max(np.linalg.norm(ref), 1e-300)
    diff = got - ref
    return np.abs(diff).max() / scale_max, np.linalg.norm(diff) / scale_f


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


# ------------------------------------------------------------------ cfg3 / cfg4: every element of one step

_PINNED = {}


def _pinned_slots(count, elems):
    """`count` sets of five page-locked float32 staging buffers of `elems` elements each, kept for the
    whole test module (copies from the GPU into page-locked memory run several times faster)."""
    key = (count, elems)
    if key not in _PINNED:
        _PINNED.clear()
        _PINNED[key] = [[torch.empty(elems, dtype=torch.float32, pin_memory=True) for _ in range(5)] for _ in range(count)]
    return _PINNED[key]


def _full_width_lockstep(sim, k, kw, what, workers=12, clone_x=False, expect=None):
    """One gpga_step at iteration k from the state the buffers hold, checked on all n x d
    elements.  x stays in the old ping-pong buffer (except on the two-pass sparse-W path,
    which leaves x^(k+1/2) there: clone_x) and g is not written by the step; m is updated
    in place, so it is cloned on the device first."""
    n, d = sim.n, sim.d
    sim.set_state(k=k)
    X_old, G, M_old = (sim.X.clone() if clone_x else sim.X), sim.G, sim.M.clone()
    sim.step()
    torch.cuda.synchronize()
    if expect is not None:   # (step_path, step_paced) as gpga_query reports them: the variant meant is the one that ran
        took = (int(sim.query("step_path")), int(sim.query("step_paced")))
        assert took == expect, f"{what}: ran as path {took[0]}, paced {took[1]}; expected {expect}"
    X_new, M_new = sim.X, sim.M
    assert X_new.data_ptr() != X_old.data_ptr()
    # Chunks of 16M elements come to the host through page-locked staging buffers (the main thread copies,
    # a slot is reused once its chunk has been checked); the workers run the oracle on pieces of 1M
    # elements, small enough to stay in the caches, with one BLAS thread each (a threaded BLAS serialises
    # the workers on such small products); the errors are put together again relative to the whole chunk.
    chunk = max(1024, (1 << 24) // n)
    piece = max(256, (1 << 20) // n)
    slots = _pinned_slots(workers + 2, n * chunk)
    free = queue.SimpleQueue()
    for slot in slots:
        free.put(slot)

    def check(c0, c1, slot):
        try:
            Xo, Mo, Gg, Xn, Mn = (b[: n * (c1 - c0)].view(n, c1 - c0).numpy() for b in slot)
            acc = {"x": [0.0, 0.0, 0.0, 0.0], "m": [0.0, 0.0, 0.0, 0.0]}   # max |diff|, max |ref|, sum diff^2, sum ref^2
            for s0 in range(0, c1 - c0, piece):
                sl = slice(s0, s0 + piece)
                X1, M1 = orc.gossip_pga_step(Xo[:, sl].astype(np.float64), Mo[:, sl].astype(np.float64),
                                             Gg[:, sl].astype(np.float64), k, **kw)
                for key, got, ref in (("x", Xn[:, sl], X1), ("m", Mn[:, sl], M1)):
                    diff = got - ref
                    a = acc[key]
                    a[0], a[1] = max(a[0], np.abs(diff).max()), max(a[1], np.abs(ref).max())
                    a[2] += float(np.vdot(diff, diff))
                    a[3] += float(np.vdot(ref, ref))
            err = {key: max(a[0] / max(a[1], 1e-300), math.sqrt(a[2]) / max(math.sqrt(a[3]), 1e-300)) for key, a in acc.items()}
            return c0, err["x"], err["m"]
        finally:
            free.put(slot)

    with threadpool_limits(limits=1), ThreadPoolExecutor(workers) as pool:
        futures = []
        for c0 in range(0, d, chunk):
            c1 = min(d, c0 + chunk)
            slot = free.get()                       # waits until a staging slot is free
            for b, t in zip(slot, (X_old, M_old, G, X_new, M_new)):
                b[: n * (c1 - c0)].view(n, c1 - c0).copy_(t[:, c0:c1])
            futures.append(pool.submit(check, c0, c1, slot))
        results = [f.result() for f in futures]
    worst_x = max(r[1] for r in results)
    worst_m = max(r[2] for r in results)
    bad = [r for r in results if r[1] > TOL_STEP or r[2] > TOL_STEP]
    assert not bad, f"{what}: chunks (first column, X error, M error) over {TOL_STEP:g}: {bad[:5]}"
    if orc.is_global_step(k, kw["H"]):
        assert bool((X_new == X_new[0:1]).all()), f"{what}: rows differ after the global average"
    print(f"{what}: all {sim.n} x {d} elements, worst X {worst_x:.2e}, worst M {worst_m:.2e}", flush=True)
    del M_old


def _random_resident_state(sim, seed):
    """Test inputs written straight into the bound buffers (device-side draws; the oracle is
    handed the very same arrays back, so no second generator is involved)."""
    gen = torch.Generator(device=sim.device)
    gen.manual_seed(seed)
    sim.X.normal_(0.0, 1.0, generator=gen)
    sim.M.normal_(0.0, 0.3, generator=gen)
    torch.cuda.synchronize()


# (topology, k) -> kernel variant on the n = 64 shapes with H = 48 (one-peer offset 2^(k mod 6))
CFG3_VARIANTS = [   # the last entry: (step_path, step_paced) the step must report (1 walk, 2 row-streaming, 3 global average)
    ("ring", 0, "paced ring walk", (1, 1)),
    ("ring", 47, "global average", (3, 1)),
    ("expo1", 0, "paced one-peer walk, offset 1 (one cycle of 64 rows)", (1, 1)),
    ("expo1", 1, "paced one-peer walk, offset 2 (two cycles of 32 rows)", (1, 1)),
    ("expo1", 2, "row-streaming kernel, offset 4 (cycles of 16 rows)", (2, 1)),
    ("expo1", 3, "row-streaming kernel, offset 8 (cycles of 8 rows)", (2, 1)),
    ("expo1", 4, "row-streaming kernel, offset 16 (cycles of 4 rows)", (2, 1)),
    ("expo1", 5, "row-streaming kernel, offset 32 (cycles of 2 rows)", (2, 1)),
]


@pytest.mark.parametrize("topology,k,what,expect", CFG3_VARIANTS, ids=[f"{t}-k{k}" for t, k, _, _ in CFG3_VARIANTS])
def test_cfg3_every_element_of_one_step_per_kernel_variant(hx, topology, k, what, expect):
    # one test per variant: each lasts seconds, so the run never stays silent for long
    c = inputs.CONFIGS["cfg3"]
    n, d = c["n"], c["d"]
    kw = dict(topology=topology, H=c["H"], lr=c["lr"], momentum=c["momentum"])
    sim = hx.Simulation(n, d, **kw)
    sim.problem_synthetic(c["seed"], c["grad_var"])
    _random_resident_state(sim, 100 + k)
    sim.set_state(k=k)
    sim.local_grad()
    _full_width_lockstep(sim, k, kw, f"cfg3 {topology} k={k} ({what})", expect=expect)
    sim.close()
    del sim
    torch.cuda.empty_cache()


@pytest.mark.parametrize("k,what,expect", [(1, "paced one-peer walk, offset 2", (1, 1)), (5, "global average", (3, 1))], ids=["k1", "k5"])
def test_cfg4_every_element_of_a_gossip_and_a_global_step(hx, k, what, expect):
    c = inputs.CONFIGS["cfg4"]
    n, d = c["n"], c["d"]
    kw = dict(topology="expo1", H=c["H"], lr=c["lr"], momentum=c["momentum"])
    sim = hx.Simulation(n, d, **kw)
    sim.problem_synthetic(c["seed"], c["grad_var"])
    _random_resident_state(sim, 200 + k)
    sim.set_state(k=k)
    sim.local_grad()
    _full_width_lockstep(sim, k, kw, f"cfg4 expo1 k={k} ({what})", expect=expect)
    sim.close()
    del sim
    torch.cuda.empty_cache()


@pytest.mark.parametrize("topology,k,what,expect", [("ring", 0, "paced ring walk", (1, 1)), ("expo1", 4, "row-streaming kernel, cycles of 4 rows", (2, 1)),
                                                    ("ring", 47, "global average", (3, 1))], ids=["ring-k0", "expo1-k4", "ring-k47"])
def test_cfg3_every_element_of_one_step_with_nesterov_momentum(hx, topology, k, what, expect):
    # the Nesterov variants of the kernels (App. F.1 names the optimizer) in the launch configuration of cfg3
    c = inputs.CONFIGS["cfg3"]
    n, d = c["n"], c["d"]
    kw = dict(topology=topology, H=c["H"], lr=c["lr"], momentum=c["momentum"])
    sim = hx.Simulation(n, d, **kw)
    sim.set_nesterov(True)
    sim.problem_synthetic(c["seed"], c["grad_var"])
    _random_resident_state(sim, 300 + k)
    sim.set_state(k=k)
    sim.local_grad()
    _full_width_lockstep(sim, k, dict(kw, nesterov=True), f"cfg3 {topology} k={k} ({what}, Nesterov)", expect=expect)
    sim.close()
    del sim
    torch.cuda.empty_cache()


SPARSE_AT_SIZE = [   # the last entry: (step_path, step_paced): 4 whole tile, 5 sliding window, 6 two passes, 10 circulant W
    (64, 25_600_000, "grid", {}, "whole-tile kernel, 16-byte lanes, paced", (4, 1)),
    (64, 25_600_000, "expo", {}, "whole-tile kernel, 16-byte lanes, paced", (4, 1)),
    (128, 12_800_000, "expo", {}, "whole-tile kernel, 128 KiB tile, 16 wavefronts", (4, 1)),
    (256, 6_400_000, "expo", {"mix_lane_bytes": 4}, "whole-tile kernel, 4-byte lanes, 16 wavefronts", (4, 0)),
    (256, 6_400_000, "expo", {}, "circulant W, 512-byte row pieces", (10, 0)),
    (256, 6_400_000, "grid", {}, "sliding-window kernel, paced", (5, 1)),
    (1024, 1_000_000, "grid", {}, "sliding-window kernel, 8-byte lanes, paced", (5, 1)),
    (1024, 1_000_000, "expo", {"mix_two_pass": 1}, "two passes", (6, 0)),
    (1024, 1_000_000, "expo", {}, "circulant W, 128-byte row pieces", (10, 0)),
]


@pytest.mark.parametrize("n,d,topology,opts,what,expect", SPARSE_AT_SIZE,
                         ids=["-".join([f"{n}x{d}", t, *o]) for n, d, t, o, _, _ in SPARSE_AT_SIZE])
def test_sparse_W_every_element_of_one_step_at_full_size(hx, n, d, topology, opts, what, expect):
    # the sparse-W kernels in the launch configurations large problems get (synthetic gradients)
    kw = dict(topology=topology, H=0, lr=0.1, momentum=0.9)
    sim = hx.Simulation(n, d, **kw)
    for name, v in opts.items():
        sim.set_option(name, v)
    sim.problem_synthetic(7, 1e-3)
    _random_resident_state(sim, 400)
    sim.set_state(k=0)
    sim.local_grad()
    G_before = sim.G[:, ::997].clone()
    _full_width_lockstep(sim, 0, kw, f"{n} x {d}, {topology} ({what})", clone_x=(what == "two passes"), expect=expect)
    assert torch.equal(sim.G[:, ::997], G_before), "the step wrote to g"
    sim.close()
    del sim
    torch.cuda.empty_cache()


# ------------------------------------------------------------------ cfg5 at its full shape

def _virtual_rows_f32(c, node, samples, d, chunk=1 << 17):
    """Feature rows of one node (len(samples) x d) as the float32 array they stand for."""
    out = np.empty((len(samples), d), dtype=np.float32)
    for c0 in range(0, d, chunk):
        cc = np.arange(c0, min(d, c0 + chunk))
        out[:, c0:c0 + len(cc)] = orc.virtual_features(c["seed"], node, samples, cc, c["mu_var"]).astype(np.float32)
    return out


def _logistic_row(Hf32, y_b, x_row):
    """Oracle gradient row from materialised feature rows (Sec. 5.1 loss)."""
    Hd = Hf32.astype(np.float64)
    z = Hd @ x_row
    coef = -y_b * expit(-y_b * z) / len(y_b)
    return Hd.T @ coef


def test_cfg5_full_shape_lockstep_over_two_averaging_periods(hx):
    c = inputs.CONFIGS["cfg5"]
    n, d, M, B, H = c["n"], c["d"], c["M"], c["B"], 8
    T = 2 * H + 1
    y = inputs.virtual_labels(n, M, c["seed"])
    idx = inputs.batch_indices(T, n, B, M, c["seed"])
    nodes = [0, 1, 127, 300, 511, 512, 777, 1023]
    cols = np.union1d(inputs.slab_columns(d, 16, 256), np.arange(d - 1024, d))
    sims = {}
    for topology in c["topologies"]:
        sim = hx.Simulation(n, d, topology=topology, H=H, lr=c["lr"], momentum=c["momentum"])
        sim.problem_logreg_virtual(c["seed"], y, c["mu_var"])
        sims[topology] = (sim, sim.upload_batches(idx), dict(topology=topology, H=H, lr=c["lr"], momentum=c["momentum"]))
    cols_d = torch.as_tensor(cols, device="cuda")
    nodes_d = torch.as_tensor(nodes, device="cuda")
    slab = lambda t: host(t.index_select(1, cols_d))
    worst = {"G": 0.0, "X": 0.0, "M": 0.0}
    for k in range(T):
        # the features of step k are the same for both graphs (same minibatch table): regenerate once
        with ThreadPoolExecutor(len(nodes)) as pool:
            feats = list(pool.map(lambda i: _virtual_rows_f32(c, i, np.asarray(idx[k][i], dtype=np.int64), d), nodes))
        for topology, (sim, idx_d, kw) in sims.items():
            sim.local_grad(idx_d[k])
            Xn = host(sim.X.index_select(0, nodes_d))
            G_ref = np.stack([_logistic_row(feats[j], y[i].astype(np.float64)[idx[k][i]], Xn[j])
                              for j, i in enumerate(nodes)])
            e = max(rel_errors(host(sim.G.index_select(0, nodes_d)), G_ref))
            worst["G"] = max(worst["G"], e)
            assert e <= TOL_STEP, f"cfg5 {topology}: gradient rows at step {k}: {e:.2e}"
            Xs, Ms, Gs = slab(sim.X), slab(sim.M), slab(sim.G)
            X1, M1 = orc.gossip_pga_step(Xs, Ms, Gs, k, **kw)
            sim.step()
            Xg = slab(sim.X)
            ex, em = max(rel_errors(Xg, X1)), max(rel_errors(slab(sim.M), M1))
            worst["X"], worst["M"] = max(worst["X"], ex), max(worst["M"], em)
            assert ex <= TOL_STEP and em <= TOL_STEP, f"cfg5 {topology}: lock-step X {ex:.2e} M {em:.2e} at step {k}"
            ce = sim.consensus_error()
            if orc.is_global_step(k, H):
                assert ce == 0.0, f"cfg5 {topology}: consensus distance {ce} right after a global average"
            else:   # slab columns are a sample of the columns: same per-column spread up to sampling noise
                assert ce == pytest.approx(orc.consensus_error(X1) * math.sqrt(d / len(cols)), rel=0.1)
        del feats
    print(f"cfg5 full shape, H={H}, {T} steps x 2 graphs: worst G rows {worst['G']:.2e}, X {worst['X']:.2e}, M {worst['M']:.2e}")
    for sim, _, _ in sims.values():
        sim.close()
    sims.clear()
    torch.cuda.empty_cache()


# ------------------------------------------------------------------ cfg5 replica at the stated step size

_REPLICA = {}


def _replica():
    """n = 1024 nodes as in cfg5 with d = 4096 and M = 64, so that the oracle can hold the feature
    array (materialised once from its own counter RNG) and follow the non-separable iteration."""
    if not _REPLICA:
        c = inputs.CONFIGS["cfg5"]
        n, d, M, B, T = c["n"], 4096, 64, c["B"], c["T"]
        y = inputs.virtual_labels(n, M, c["seed"])
        idx = inputs.batch_indices(T, n, B, M, c["seed"])
        with ThreadPoolExecutor(8) as pool:
            rows = list(pool.map(lambda i: orc.virtual_features(c["seed"], i, np.arange(M), np.arange(d),
                                                                c["mu_var"]).astype(np.float32), range(n)))
        _REPLICA.update(n=n, d=d, M=M, B=B, T=T, y=y, idx=idx, feat=np.stack(rows))
    return _REPLICA


def _lock_steps(T, H):
    """Steps at which the GPU state is checked in lock-step: the first 17 (two periods of H = 8 and
    one more), the steps around the first two, a middle and the last three global averages, and a
    sample spread over the whole run."""
    picks = set(range(min(T, 17))) | set(range(0, T, 37)) | {T - 2, T - 1}
    if H > 0:
        glob = list(range(H - 1, T, H))
        for g in glob[:2] + glob[len(glob) // 2:][:1] + glob[-3:]:
            picks |= {g - 1, g, g + 1}
    return sorted(s for s in picks if 0 <= s < T)


@pytest.mark.parametrize("topology", ["ring", "expo1"])
@pytest.mark.parametrize("H", [1, 8, 64, 0])
def test_cfg5_replica_stated_step_size_lockstep_through_1000_steps(hx, topology, H):
    c = inputs.CONFIGS["cfg5"]
    r = _replica()
    n, d, T, y, idx, feat = r["n"], r["d"], r["T"], r["y"], r["idx"], r["feat"]
    kw = dict(topology=topology, H=H, lr=c["lr"], momentum=c["momentum"])
    sim = hx.Simulation(n, d, **kw)
    sim.problem_logreg_virtual(c["seed"], y, c["mu_var"])
    idx_d = sim.upload_batches(idx)
    checks = set(_lock_steps(T, H))
    worst = 0.0
    for k in range(T):
        sim.local_grad(idx_d[k])
        if k in checks:
            Xg, Gg, Mg = host(sim.X), host(sim.G), host(sim.M)
            e = max(rel_errors(Gg, orc.logreg_grad(feat, y, Xg, idx[k])))
            assert e <= TOL_STEP, f"G at step {k}: {e:.2e}"
            X1, M1 = orc.gossip_pga_step(Xg, Mg, Gg, k, **kw)
        sim.step()
        if k in checks:
            Xn = host(sim.X)
            ex, em = max(rel_errors(Xn, X1)), max(rel_errors(host(sim.M), M1))
            worst = max(worst, e, ex, em)
            assert ex <= TOL_STEP and em <= TOL_STEP, f"lock-step at step {k}: X {ex:.2e} M {em:.2e}"
            ce, ce_ref = sim.consensus_error(), orc.consensus_error(X1)
            if H == 1 or orc.is_global_step(k, H):
                assert ce == 0.0
            else:   # the consensus distance is a seminorm: it moves by at most ||X_gpu - X_oracle||_F
                assert abs(ce - ce_ref) <= np.linalg.norm(Xn - X1) + TOL_STEP * ce_ref
    print(f"cfg5 replica {topology} H={H}: T={T} at lr={c['lr']}, {len(checks)} lock-step checks, worst {worst:.2e}")
    sim.close()


@pytest.mark.parametrize("topology", ["ring", "expo1"])
def test_cfg5_replica_stated_step_size_free_running(hx, topology):
    # Free-running GPU and oracle trajectories at the stated step size.  With gamma = 0.05 on features
    # of squared norm ~ 1.5 d the iteration amplifies rounding: the oracle with fp32 storage and the same
    # oracle in float64 drift apart on their own (the "floor", printed).  The floor is what ONE rounding
    # per element and step (the fp32 store) grows into; a GPU step rounds about eight times per element
    # (gradient, two in the momentum, two in the update, three in the mix), each perturbation amplified by
    # the same dynamics, so the iterates are held to TOL_FINAL while 16 x floor stays below it and to
    # 16 x floor after that.  Beyond that bound free-running parity at this step size is unpinned; the
    # per-step parity of the same run is what the lock-step test above asserts.
    c = inputs.CONFIGS["cfg5"]
    r = _replica()
    n, d, y, idx, feat = r["n"], r["d"], r["y"], r["idx"], r["feat"]
    H, T = 8, 72
    kw = dict(topology=topology, H=H, lr=c["lr"], momentum=c["momentum"])
    sim = hx.Simulation(n, d, **kw)
    sim.problem_logreg_virtual(c["seed"], y, c["mu_var"])
    idx_d = sim.upload_batches(idx)
    ref = orc.GossipPGA(n, d, storage="f32", **kw)
    ref64 = orc.GossipPGA(n, d, storage="f64", **kw)
    report = []
    for k in range(T):
        sim.local_grad(idx_d[k])
        sim.step()
        ref.step(orc.logreg_grad(feat, y, ref.X, idx[k]))
        ref64.step(orc.logreg_grad(feat, y, ref64.X, idx[k]))
        if k in (7, 16, 35, T - 1):
            err = max(rel_errors(host(sim.X), ref.X))
            floor = max(rel_errors(ref.X, ref64.X))
            report.append((k + 1, err, floor))
            assert err <= max(TOL_FINAL, 16.0 * floor), f"after {k + 1} steps: GPU vs oracle {err:.2e}, oracle floor {floor:.2e}"
    print(f"cfg5 replica {topology} free-running at lr={c['lr']}: (steps, GPU vs oracle, oracle fp32-storage vs float64) "
          + ", ".join(f"({t}, {e:.2e}, {f:.2e})" for t, e, f in report))
    sim.close()


# ------------------------------------------------------------------ adaptive period (Algorithm 2) on the replica

@pytest.mark.parametrize("topology", ["ring", "expo1"])
def test_cfg5_replica_gossip_aga_lockstep(hx, topology):
    # Algorithm 2 on n = 1024 nodes with the virtual-feature logistic problem at the stated step size:
    # every iteration the oracle's Gossip-AGA is put on the GPU's state (X, M; its own counter C,
    # F_init and H carry over), fed the oracle's gradients and minibatch losses at that state, and
    # must reach the same period decision and, within 1e-5, the same next state.
    c = inputs.CONFIGS["cfg5"]
    r = _replica()
    n, d, y, idx, feat = r["n"], r["d"], r["y"], r["idx"], r["feat"]
    T, H_init, K_w, H_max = 96, 4, 24, 32
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=c["lr"], momentum=c["momentum"])
    sim.problem_logreg_virtual(c["seed"], y, c["mu_var"])
    sim.aga_enable(H_init, K_w, H_max)
    idx_d = sim.upload_batches(idx[:T])
    ref = orc.GossipAGA(n, d, topology=topology, H_init=H_init, warmup_iters=K_w, H_max=H_max, lr=c["lr"],
                        momentum=c["momentum"], storage="f32")
    periods, worst = [], 0.0
    for k in range(T):
        loss = sim.local_loss(idx_d[k])
        sim.local_grad(idx_d[k])
        Xg, Mg = host(sim.X), host(sim.M)
        loss_ref = orc.logreg_loss(feat, y, Xg, idx[k])
        e_loss = np.abs(host(loss) - loss_ref).max() / max(np.abs(loss_ref).max(), 1e-300)
        assert e_loss <= TOL_STEP, f"minibatch losses at step {k}: {e_loss:.2e}"
        ref.pga.X, ref.pga.M = Xg.copy(), Mg.copy()
        ref.step(orc.logreg_grad(feat, y, Xg, idx[k]), loss_ref)
        sim.aga_step(loss)
        assert sim.period == ref.H, f"period differs at step {k}: {sim.period} vs {ref.H}"
        periods.append(sim.period)
        ex, em = max(rel_errors(host(sim.X), ref.X)), max(rel_errors(host(sim.M), ref.M))
        worst = max(worst, e_loss, ex, em)
        assert ex <= TOL_STEP and em <= TOL_STEP, f"lock-step at step {k}: X {ex:.2e} M {em:.2e}"
        if ref.history and ref.history[-1][0] == k:
            assert bool((sim.X == sim.X[0:1]).all()), f"rows differ after the global average of step {k}"
    assert len(ref.history) >= 3 and len(set(periods)) > 1, (ref.history, "the period never adapted")
    print(f"cfg5 replica Gossip-AGA {topology}: periods {sorted(set(periods))}, averages at {[h[0] for h in ref.history]}, worst {worst:.2e}")
    sim.close()


# Free-running walks of few rows: one wavefront a workgroup on 16-byte rows, four on others, batches of 2, 4 and 8 rows with
# and without rows behind the last batch; the last case is the first size of its row count that is paced again.
@pytest.mark.parametrize("n,d,topology,k,momentum,expect", [
    (8, 8_400_004, "ring", 0, 0.9, (1, 0)), (8, 8_400_004, "full", 0, 0.9, (3, 0)), (8, 8_400_004, "expo1", 0, 0.9, (2, 0)),
    (8, 8_400_004, "none", 0, 0.9, (1, 0)), (11, 6_200_000, "ring", 0, 0.9, (1, 0)), (3, 22_400_000, "ring", 0, 0.9, (1, 0)),
    (3, 22_400_000, "full", 0, 0.9, (3, 0)), (5, 13_500_001, "ring", 0, 0.9, (1, 0)), (20, 3_400_000, "expo1", 0, 0.9, (1, 0)),
    (32, 2_200_003, "ring", 0, 0.9, (1, 0)), (32, 2_200_000, "expo1", 1, 0.9, (2, 0)), (64, 2_560_000, "ring", 0, 0.9, (1, 1))])
def test_free_running_walks_of_few_rows(hx, n, d, topology, k, momentum, expect):
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=momentum)
    sim.problem_synthetic(5, 1e-3)
    _random_resident_state(sim, seed=n + d)
    sim.local_grad()
    kw = dict(topology=topology, H=0, lr=0.1, momentum=momentum)
    _full_width_lockstep(sim, k, kw, f"free-running {topology} {n} x {d}", expect=expect)
    sim.close()
    torch.cuda.empty_cache()


# Sizes that run free by themselves: a rate, a residency, the shortest paced cycle or the persistent one-peer kernel asked for
# by itself is what the step gets; expect = (step_path, step_paced).
@pytest.mark.parametrize("n,d,topology,k,opts,expect", [
    (8, 16_800_000, "ring", 0, {}, (1, 0)), (8, 16_800_000, "ring", 0, {"pace_gbs": 5000}, (1, 1)),
    (8, 16_800_000, "full", 0, {"pace_gbs": 5000}, (3, 1)), (8, 16_800_000, "expo1", 0, {"pace_gbs": 5000}, (2, 1)),
    (20, 6_800_000, "expo1", 2, {"pace_gbs": 5000}, (1, 1)), (8, 16_800_000, "ring", 0, {"blocks_per_cu": 2}, (1, 1)),
    (8, 16_800_000, "full", 0, {"blocks_per_cu": 2}, (3, 1)), (8, 16_800_000, "ring", 0, {"pace_min_cycle": 8}, (1, 1)),
    (8, 16_800_000, "expo1", 1, {"cycle_kernel": 1}, (2, 1)), (16, 600_000, "expo1", 0, {"pace_gbs": 4000}, (2, 1)),
    (8, 16_800_000, "ring", 0, {"pace_gbs": 0}, (1, 0))])
def test_launches_asked_for_on_few_rows(hx, n, d, topology, k, opts, expect):
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=0.9)
    for name, value in opts.items():
        sim.set_option(name, value)
    sim.problem_synthetic(5, 1e-3)
    _random_resident_state(sim, seed=n + d)
    sim.local_grad()
    _full_width_lockstep(sim, k, dict(topology=topology, H=0, lr=0.1, momentum=0.9), f"{topology} {n} x {d} {opts}", expect=expect)
    sim.close()
    torch.cuda.empty_cache()


# Free-running steps with the consensus trace and, in the batches of rows that untraced walks take, without: lone wavefronts and
# workgroups of four, one-peer offsets with several cycles a tile (12 rows: two cycles of 6; 20: four of 5), no momentum, Nesterov
# momentum; expect = (step_path, step_paced, trace_fused if traced).  X and M are checked against the step in float64; the trace sums the stored fp32 values in fp64, so only rounding of some 1e8
# additions (about 1e-12 for pairwise orders) stands between it and torch's figure.
@pytest.mark.parametrize("n,d,topology,k,momentum,nesterov,expect", [
    (8, 8_400_004, "ring", 0, 0.0, False, (1, 0, 1)), (8, 8_400_004, "ring", 0, 0.9, True, (1, 0, 1)),
    (8, 8_400_004, "full", 0, 0.0, False, (3, 0, 0)), (8, 8_400_004, "full", 0, 0.9, True, (3, 0, 0)),
    (8, 8_400_004, "expo1", 1, 0.0, False, (2, 0, 1)), (16, 4_200_004, "expo1", 0, 0.9, True, (2, 0, 1)),
    (20, 6_800_000, "expo1", 2, 0.9, False, (1, 0, 1)), (12, 11_200_004, "expo1", 1, 0.0, False, (1, 0, 1)),
    (20, 6_800_000, "expo1", 3, 0.9, True, (1, 0, 1)), (4, 33_600_000, "ring", 0, 0.9, False, (1, 0, 1)),
    (8, 2_000_000, "expo1", 0, 0.9, False, (2, 0, 1)), (2, 67_200_000, "expo1", 0, 0.9, False, (2, 0, 1))])
@pytest.mark.parametrize("traced", [True, False])
def test_trace_of_free_running_steps(hx, n, d, topology, k, momentum, nesterov, expect, traced):
    sim = hx.Simulation(n, d, topology=topology, H=0, lr=0.1, momentum=momentum)
    if nesterov:
        sim.set_nesterov(True)
    gen = torch.Generator(device=sim.device)
    gen.manual_seed(n + d)
    for t in (sim.X, sim.M, sim.G):
        if t is not None:
            t.normal_(0.0, 1.0, generator=gen)
    x, g = sim.X, sim.G
    m = sim.M.double() if momentum else None
    trace = sim.attach_trace(k + 1) if traced else None
    sim.set_state(k=k)
    sim.step()
    torch.cuda.synchronize()
    assert (int(sim.query("step_path")), int(sim.query("step_paced")), int(sim.query("trace_fused"))) == (*expect[:2], expect[2] * traced)
    lr, mu = float(np.float32(0.1)), float(np.float32(momentum))
    mom = mu * m + g if momentum else g
    y = x - lr * (g + mu * mom if nesterov else mom).double()
    if topology == "full":
        want = y.mean(dim=0, keepdim=True).expand(n, d)
    elif topology == "ring":
        want = (torch.roll(y, 1, 0) + y + torch.roll(y, -1, 0)) / 3
    else:
        want = (y + torch.roll(y, -orc.one_peer_shift(n, k), 0)) / 2
    assert float((sim.X - want).abs().max()) <= TOL_STEP * float(want.abs().max())
    if momentum:
        assert float((sim.M - mom).abs().max()) <= TOL_STEP * float(mom.abs().max())
    del y, want, mom, m
    if traced:
        dist = 0.0 if topology == "full" else float((sim.X - sim.X.double().mean(dim=0)).norm())
        assert abs(float(trace[k]) - dist) <= 1e-9 * dist
    sim.close()
    torch.cuda.empty_cache()


# gpga_tune runs the kinds of step that are paced; where none is, the caller's arrays and what gpga_query reports stay as they were.
@pytest.mark.parametrize("n,d,topology,H,kinds", [
    (8, 25_600_000, "ring", 4, ()), (8, 16_800_000, "full", 0, ()), (20, 6_800_000, "expo1", 6, ()), (8, 16_800_000, "none", 4, ()),
    (300, 450_000, "expo", 0, ()), (64, 2_560_000, "ring", 4, ("ring", "global")), (64, 2_560_000, "none", 4, ("global",))])
def test_tune_runs_paced_steps_only(hx, n, d, topology, H, kinds):
    sim = hx.Simulation(n, d, topology=topology, H=H, lr=0.1, momentum=0.9)
    gen = torch.Generator(device=sim.device)
    gen.manual_seed(n + d)
    arrays = (*sim._bufs, sim.M, sim.G)
    for t in arrays:
        t.normal_(0.0, 1.0, generator=gen)
    kept = [t.clone() for t in arrays]
    sim.tune(4)
    torch.cuda.synchronize()
    assert all(torch.equal(t, u) for t, u in zip(arrays, kept)) == (not kinds)
    assert sim.k == 0 and int(sim.query("step_path")) == (3 if kinds else 0)
    ran = {name: sum(sim.query(f"pace_launches:{name}{way}") for way in ("", "/1")) for name in ("global", "ring", "self", "tile")}
    assert ran == {name: 4 * (name in kinds) for name in ran}
    sim.close()
    torch.cuda.empty_cache()

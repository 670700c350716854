"""Where a small network leaves the one launch for many steps to the kernels of the whole network: the same results on
both sides of the line and across it, with the estimate of the vehicles on the road right, too low and too high; no
slower than the kernel-by-kernel path where many are on the road; and the reverse sweep of such a run."""
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    assert torch.cuda.is_available()
    import paper_2007_03614_amd as M
    return M


def _same(a, b, where):
    sa, sb = a.state(), b.state()
    for k in sa:
        assert np.array_equal(np.asarray(sa[k]), np.asarray(sb[k])), (where, k)
    for x, y in zip(a.edge_stats(), b.edge_stats()):
        assert np.array_equal(x, y), where


def _grid(n, within_s, mode=0, spread=0.0):
    w = W.config1(n_vehicles=n)
    w.depart_step = (w.depart_step.astype(np.int64) * within_s // 600).astype(np.int32)
    w.params.intersection_mode, w.params.v0_spread = mode, spread
    return w


# 1,024 vehicles in all take the one launch always; 6,000 cross the line and come back
@pytest.mark.parametrize("n,within_s,mode,spread", [(1024, 30, 0, 0.0), (1025, 30, 1, 0.05), (6000, 600, 0, 0.05),
                                                    (6000, 600, 1, 0.0)])
def test_both_sides_of_the_line(M, n, within_s, mode, spread):
    w = _grid(n, within_s, mode, spread)
    a, b = M.Sim(w), M.Sim(w)
    for steps in (1, 15, 17, 600, 1030, 700):
        a.step(steps)
        b.step_timed(steps)
        _same(a, b, a.n_active)
        a.write_state(a.state())
        b.write_state(b.state())


@pytest.mark.parametrize("members", [2, 63, 64])
def test_ensembles_across_the_line(M, members):
    w = _grid(6000, 600)
    scen = [(6000 - 40 * k, np.zeros(0, np.int32)) for k in range(members)]
    a, b = M.Sim(w, scenarios=scen), M.Sim(w, scenarios=scen)
    for steps in (500, 300, 900):
        a.step(steps)
        b.step_timed(steps)
        _same(a, b, a.n_active)


def _dense(n_wait=0, due=0):
    """The 10x10 grid with 2,880 on the road from the start, and vehicles that wait."""
    w, s = W.probe_r(W.grid_network(10, 10), density=0.15, route_len=400, params=W.base_params(1), seed=1)
    n = w.n_vehicles
    assert n == 2880
    w.depart_step = np.full(n, due, np.int32)
    if n_wait:
        w = W.Workload(w.name, w.net, np.arange(n + n_wait + 1, dtype=np.int64) * 400,
                       np.concatenate([w.route_edges, np.tile(w.route_edges[:400], n_wait)]),
                       np.concatenate([w.depart_step, np.full(n_wait, 10 ** 6, np.int32)]),
                       np.zeros(n + n_wait, np.uint8), np.full(n + n_wait, 0.2, np.float32), w.params, w.n_steps)
        first = w.route_edges[w.route_off[n:-1]]
        s = {k: np.concatenate([v, first if k == "edge" else np.full(n_wait, -1 if k in ("held_since", "tau_in", "t_arr")
                                                                      else 0, v.dtype)])
             if isinstance(v, np.ndarray) else v for k, v in s.items()}
    return w, s


# 2,880 vehicles; more than 3,072 with most still waiting; all of them ahead of their departure steps
@pytest.mark.parametrize("n_wait,due", [(0, 0), (1000, 0), (1000, 500_000)])
def test_no_slower_than_kernel_by_kernel(M, n_wait, due):
    w, s = _dense(n_wait, due)
    a, b = M.Sim(w), M.Sim(w)
    best = [np.inf, np.inf]
    for _ in range(5):
        a.write_state(s)
        a.n_active
        t = time.perf_counter()
        a.step(320)
        a.n_active
        best[0] = min(best[0], time.perf_counter() - t)
        b.write_state(s)
        best[1] = min(best[1], sum(b.step_timed(320)[0].values()) * 1e-3)
    _same(a, b, "dense")
    # the four kernels without the gaps between them, against all of the call; one workgroup takes twice that
    print("step, kernels [us]:", best[0] / 320 * 1e6, best[1] / 320 * 1e6)
    assert best[0] < 1.6 * best[1], best


def test_gradient_of_a_dense_run(M, oracle_mod):
    """1,900 on the road on average: the reverse sweep by the kernels of the whole network, whatever the interval of
    the checkpoints; 1e-3 relative to the oracle's FP64 adjoint, the contract of the differentiable form.
    (300 steps: in the gridlock that follows the oracle's replay is not a number.)"""
    w = _grid(9000, 300)
    steps, grads = 300, []
    for every in (100, 64):
        w.params.record_every = every
        sim = M.Sim(w)
        sim.step(steps)
        assert sim.counters()["active_sum"] > 1536 * steps
        mean, cnt = sim.mean_travel_times()
        target = np.asarray(w.net.length, np.float64) / w.net.limit
        grads.append(sim.backward(np.where(cnt > 0, 2.0 * (mean - target), 0.0)))
        sim.close()
    assert np.array_equal(grads[0], grads[1])
    w.params.record_every = 0
    o = oracle_mod.OracleSim(w)
    o.enable_record()
    o.step(steps)
    assert np.array_equal(o.edge_stats()[1], cnt)
    _, _, og = o.replay(o.theta(w), target, (cnt > 0).astype(np.uint8), grad=True)
    og = og.reshape(-1, 5)
    assert np.linalg.norm(grads[0] - og) <= 1e-3 * np.linalg.norm(og)

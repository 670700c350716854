"""Ensembles of small networks, many steps per launch: last members without vehicles (whose layouts would begin past
the last slot), with everybody on the road and with nobody left, and refused departures counted over all members,
against the kernel-by-kernel path."""
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


NONE = np.zeros(0, np.int32)


def _same(a, b, where):
    sa, sb = a.state(), b.state()
    for k in sa:
        assert np.array_equal(np.asarray(sa[k]), np.asarray(sb[k])), (where, k)
    for x, y in zip(a.edge_stats(), b.edge_stats()):
        assert np.array_equal(x, y), where
    assert a.counters() == b.counters(), where


# 1,024 and 2,048 vehicles fill whole pages of the slot arrays
@pytest.mark.parametrize("members", [[1024, 0], [1024, 1024, 0, 0], [0, 700, 0], [0, 0]])
@pytest.mark.parametrize("spread", [0.0, 0.05])
def test_last_members_without_vehicles(M, members, spread):
    w = W.config1(n_vehicles=1024)
    w.depart_step = (w.depart_step // 20).astype(np.int32)
    w.params.v0_spread = spread
    scen = [(n, NONE) for n in members]
    a, b = M.Sim(w, scenarios=scen), M.Sim(w, scenarios=scen)
    for steps in (1, 2, 63, 130, 1500):
        a.step(steps)
        b.step_timed(steps)
        _same(a, b, a.state()["t"])


def test_everybody_on_the_road(M):
    """A written state without a free slot: the empty member's first layout is at its end."""
    w, s = W.probe_r(W.grid_network(10, 10), density=0.05, route_len=40, params=W.base_params(1), seed=2)
    n = w.n_vehicles
    scen = [(n, NONE), (0, NONE)]
    a, b = M.Sim(w, scenarios=scen), M.Sim(w, scenarios=scen)
    for sim in (a, b):
        sim.write_state(s)
    a.step(1)
    b.step_timed(1)
    _same(a, b, "one step")
    a.step(400)
    b.step_timed(400)
    _same(a, b, "more")


@pytest.mark.parametrize("steps", [1, 70, 1100])
def test_refused_departures_over_all_members(M, steps):
    """A written state in which the first member is ahead of its demand (on the road before their departure steps)
    while the second one's departures wait at one lane: the count is of all members' vehicles together."""
    w, s = W.probe_r(W.grid_network(10, 10), density=0.05, route_len=40, params=W.base_params(1), seed=2)
    n, q = w.n_vehicles, 400
    route = w.route_edges[:40]
    w2 = W.Workload("ahead", w.net, np.arange(n + q + 1, dtype=np.int64) * 40,
                    np.concatenate([w.route_edges, np.tile(route, q)]),
                    np.concatenate([np.full(n, 600, np.int32), np.full(q, 100, np.int32)]),
                    np.zeros(n + q, np.uint8), np.full(n + q, 0.2, np.float32), w.params, w.n_steps)
    both = {}
    for k, a in s.items():
        if not isinstance(a, np.ndarray):
            both[k] = a
            continue
        gone, waits = (2, 0) if k == "status" else (0, 0)
        first = w2.route_edges[w2.route_off[:-1]]
        rest = first[n:] if k == "edge" else np.full(q, gone, a.dtype)
        out = np.zeros(n + q, a.dtype) if k != "edge" else first + w.net.n_edges
        both[k] = np.concatenate([a, rest, out]).astype(a.dtype)
    both["held_since"][:] = -1
    both["t"] = 590
    assert both["status"][:n].all() and not both["status"][n + q:].any()
    scen = [(n + q, NONE)] * 2
    a, b = M.Sim(w2, scenarios=scen), M.Sim(w2, scenarios=scen)
    for sim in (a, b):
        sim.write_state(both)
    a.step(steps)
    b.step_timed(steps)
    _same(a, b, steps)
    # the second member's 400 wait at most, fewer than the first is ahead until step 600
    assert n > q and (a.counters()["insert_denied"] == 0) == (steps == 1)

"""Commit with one thread per lane: edges of every lane count, where lane numbers skip to the next workgroup's block
(256 is no multiple of 3, 5, 6 and 7), and edges that several vehicles leave in one step, whose travel times add up
in vehicle order.  Against the oracle, both kinds of intersections."""
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


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("lanes", [1, 3, 5, 6, 7, 8, "mixed"])
def test_lane_counts(M, oracle_mod, lanes, mode):
    from test_gpu_parity import compare_states
    w = W.config1(n_vehicles=4000)
    net = W.grid_network(14, 13, lanes=2 if lanes == "mixed" else lanes)
    if lanes == "mixed":
        two_way = {}
        rng = np.random.default_rng(3)
        for e, (a, b) in enumerate(zip(net.edge_from.tolist(), net.edge_to.tolist())):
            net.lanes[e] = two_way.setdefault((min(a, b), max(a, b)), rng.integers(1, 9))
        W.turn_lane_masks(net)
    w.net = net
    rng = np.random.default_rng(4)
    o, d = rng.integers(0, 13, 4000), net.n_nodes - 1 - rng.integers(0, 13, 4000)      # one side to the other
    w.route_off, w.route_edges, ok = W.shortest_routes(net, o, d)
    assert ok.all()
    w.params.intersection_mode = mode
    w.depart_step = (w.depart_step // 4).astype(np.int32)
    g, orc = M.Sim(w), oracle_mod.OracleSim(w)
    for steps in (40, 260, 300):
        g.step_timed(steps)                     # the kernels of the whole network, also where lanes are few
        orc.step(steps)
        assert compare_states(g.state(), orc.state(), f"step {orc.t}")
    gs, gc = g.edge_stats()
    os_, oc = orc.edge_stats()
    assert np.array_equal(gc, oc) and np.array_equal(gs, os_)
    assert dict(zip(M.COUNTERS, g.state()["counters"].tolist())) == orc.counters()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("lanes", [3, "mixed"])
def test_many_lanes(M, oracle_mod, lanes, mode):
    """Above 190,000 lanes a thread of the commit takes four lanes."""
    from test_gpu_parity import compare_states
    rows = 140
    net = W.grid_network(rows, rows, lanes=3)
    rng = np.random.default_rng(5)
    if lanes == "mixed":
        two_way = {}
        for e, (a, b) in enumerate(zip(net.edge_from.tolist(), net.edge_to.tolist())):
            net.lanes[e] = two_way.setdefault((min(a, b), max(a, b)), rng.integers(1, 9))
        W.turn_lane_masks(net)
    assert net.lanes.sum() > 190_000
    w = W.config1(n_vehicles=6000)
    w.net = net
    o = rng.integers(0, net.n_nodes, 6000)
    d = (o + rng.integers(1, 4, 6000) + rows * rng.integers(0, 3, 6000)) % net.n_nodes
    near = rng.integers(0, 60, 3000)                 # half of the trips in one corner, which fills up
    o[:3000], d[:3000] = near, near + 2 * rows + rng.integers(1, 9, 3000)
    w.route_off, w.route_edges, ok = W.shortest_routes(net, o, d)
    assert ok.all()
    w.params.intersection_mode = mode
    w.depart_step = (w.depart_step // 8).astype(np.int32)
    g, orc = M.Sim(w), oracle_mod.OracleSim(w)
    for steps in (30, 120, 150):
        g.step(steps)
        orc.step(steps)
        assert compare_states(g.state(), orc.state(), f"step {orc.t}")
    gs, gc = g.edge_stats()
    os_, oc = orc.edge_stats()
    assert gc.sum() > 1000 and np.array_equal(gc, oc) and np.array_equal(gs, os_)
    assert dict(zip(M.COUNTERS, g.state()["counters"].tolist())) == orc.counters()

"""More lane-change draws in a step than a workgroup lists: every vehicle of a dense edge whose route leaves it from lane
0 alone wants to move over, and both its gaps lie where the noise decides.  300 vehicles are one ordinary tile (384
listed draws) or a step of the one-workgroup kernel, 1,000 and 1,400 a tile of the 1,024-thread kernel (2,048), 2,000
its global-memory tile.  Against the oracle, bit for bit."""
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


def _queue(n, spread):
    lanes = 8
    length = 16.0 * (n // lanes + 4)
    net = W.grid_network(2, 3, spacing=length, lanes=lanes)
    net.conn_mask[:] = 1
    o, d = np.array([0]), np.array([2])
    _, route, ok = W.shortest_routes(net, o, d)
    assert ok.all() and len(route) == 2
    p = W.base_params(1)
    p.v0_spread = spread
    w = W.Workload("queue", net, 2 * np.arange(n + 1, dtype=np.int64), np.tile(route, n), np.zeros(n, np.int32),
                   np.zeros(n, np.uint8), np.linspace(0.05, 0.40, n).astype(np.float32), p, 0)
    i = np.arange(n)
    lane = i % lanes
    x = length - 2.0 - 16.0 * (i // lanes) - 8.0 * (lane % 2)
    rng = np.random.default_rng(n)
    init = dict(status=np.ones(n, np.uint8), edge=np.full(n, int(route[0]), np.int32), lane=lane.astype(np.int32),
                cursor=np.zeros(n, np.int32), x=x.astype(np.float32), v=rng.uniform(0, 3, n).astype(np.float32),
                held_since=np.full(n, -1, np.int32), mand=np.zeros(n, np.uint8), ww=np.zeros(n, np.int32),
                tau_in=np.zeros(n), t_arr=np.full(n, -1.0), counters=None, t=0)
    return w, init


@pytest.mark.parametrize("spread", [0.0, 0.1])
@pytest.mark.parametrize("n", [8, 300, 1000, 1400, 2000])
def test_full_lists(M, oracle_mod, n, spread):
    from test_gpu_parity import compare_states
    w, init = _queue(n, spread)
    whole, runs, orc = M.Sim(w), M.Sim(w), oracle_mod.OracleSim(w)
    for s in (whole, runs):
        s.write_state(init)
    orc.write_state(0, init)
    for steps in (1, 1, 2, 16, 40):
        whole.step_timed(steps)                  # the kernels of the whole network
        runs.step(steps)
        orc.step(steps)
        for s in (whole, runs):
            assert compare_states(s.state(), orc.state(), f"step {orc.t}")
    assert orc.counters()["lane_changes"] > n // 4


@pytest.mark.parametrize("n,spread", [(2600, 0.1), (1300, 0.25)])
def test_own_limits_after_a_written_state(M, oracle_mod, n, spread):
    """Every driver's limit is unknown after a written state: 2,600 on one edge are more than the 1,024-thread kernel
    lists (2,048).  Then they are carried from step to step, and drawn for the vehicles that enter the next edge."""
    from test_gpu_parity import compare_states
    w, init = _queue(n, spread)
    g, orc = M.Sim(w), oracle_mod.OracleSim(w)
    g.write_state(init)
    orc.write_state(0, init)
    for steps in (1, 1, 30, 200):
        g.step(steps)
        orc.step(steps)
        assert compare_states(g.state(), orc.state(), f"step {orc.t}")
    assert orc.counters()["transfers"] > 0
    mid = g.state()
    h = M.Sim(w)
    h.write_state(mid)
    h.step_timed(25)
    orc.step(25)
    assert compare_states(h.state(), orc.state(), f"step {orc.t}")

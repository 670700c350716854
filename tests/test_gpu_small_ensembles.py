"""Ensembles of small networks, many steps per launch: last members without vehicles (whose layouts would begin past
the last slot), with everybody on the road and with nobody left, against the kernel-by-kernel path."""
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

"""Many steps of a small network in one launch, against the kernel-by-kernel path (sim_step_timed, which the
parity tests hold to the oracle) and the oracle: launches of odd lengths and across 64- and 1,024-step words, tiles
cut in pieces, the hand-over to the kernels of the whole network where too many vehicles could be on the road,
ensembles with empty members, and the gridlock detector over scenarios."""
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


def _grid(n, within_s, mode=0, spread=0.0, classes=1):
    w = W.config1(n_vehicles=n, n_classes=classes)
    w.depart_step = (w.depart_step.astype(np.int64) * within_s // 600).astype(np.int32)
    w.params.intersection_mode, w.params.v0_spread = mode, spread
    return w


# 1,100 and more on the road fill more than one tile; above 3,072 vehicles the path depends on the demand so far
@pytest.mark.parametrize("n,within_s,mode,spread", [(1, 600, 0, 0.0), (300, 60, 1, 0.05), (3072, 60, 0, 0.0),
                                                    (3073, 60, 1, 0.0), (9000, 300, 0, 0.05)])
def test_equals_kernel_by_kernel(M, n, within_s, mode, spread):
    w = _grid(n, within_s, mode, spread, classes=1 if n < 1000 else 4)
    a, b = M.Sim(w), M.Sim(w)
    for steps in (1, 2, 61, 64, 129, 400, 1100):
        a.step(steps)
        b.step_timed(steps)
        _same(a, b, a.state()["t"])
        assert a.n_active == b.n_active
    mid = a.state()
    c = M.Sim(w)
    c.write_state(mid)
    c.step_timed(3)              # the other path in between
    c.step(70)
    a.step(73)
    sa, sc = a.state(), c.state()
    if mode == 0:                # case 1 restarts its round-robin at a written state
        for k in sa:
            assert np.array_equal(np.asarray(sa[k]), np.asarray(sc[k])), k


@pytest.mark.parametrize("members", [2, 7])
def test_ensemble_equals_kernel_by_kernel(M, members):
    w = _grid(5000, 600)
    n = [0, 1, 700, 3000, 5000, 64, 1200][:members] if members > 2 else [900, 4000]
    scen = [(k, np.array([3, 40], np.int32) if i % 2 else np.zeros(0, np.int32)) for i, k in enumerate(n)]
    a, b = M.Sim(w, scenarios=scen), M.Sim(w, scenarios=scen)
    for steps in (1, 63, 65, 300, 1030, 7):
        a.step(steps)
        b.step_timed(steps)
        _same(a, b, a.state()["t"])
    a.step_timed(2)
    b.step(2)
    _same(a, b, "paths swapped")


def test_long_run_equals_the_oracle(M, oracle_mod):
    from test_gpu_parity import compare_states
    w = _grid(2000, 200, mode=1, spread=0.05, classes=4)
    g, o = M.Sim(w), oracle_mod.OracleSim(w)
    for steps in (500, 1500):
        g.step(steps)
        o.step(steps)
        assert compare_states(g.state(), o.state(), f"step {o.t}")
    assert dict(zip(M.COUNTERS, g.state()["counters"].tolist())) == o.counters()


def test_gridlock_of_an_ensemble(M):
    """Two stopped rings stall together; a third scenario that has not departed keeps no one moving."""
    from test_oracle_sim import stopped_ring
    w, st = stopped_ring()
    n = w.n_vehicles
    scen = [(n, np.zeros(0, np.int32))] * 2
    s2 = W.replicate_state({k: v for k, v in st.items() if k != "t"}, w.net.n_edges, 2)
    s2.update(t=st["t"], counters=None)
    a, b = M.Sim(w, scenarios=scen), M.Sim(w, scenarios=scen)
    for sim in (a, b):
        sim.write_state(s2)
    a.step(599)
    assert a.counters()["gridlock_steps"] == 0
    a.step(131)
    b.step_timed(730)
    assert a.counters() == b.counters() and a.counters()["gridlock_steps"] == 131

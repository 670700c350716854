"""State I/O on the device: sizes on both sides of each way through it (written by the kernel into pinned memory up to
2,048 vehicles, one copy up to 1 MiB, a copy per field above), both slot buffers, lanes of one to a thousand vehicles,
skipped fields, and refusals that leave the handle as it was."""
import ctypes

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


def _equal(a, b, skip=()):
    for k in a:
        if k not in skip:
            assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), k


def _workload(n):
    if n <= 4000:
        return W.config1(n_vehicles=n)
    return W.scaled_config2(n, 30, 30, 10_800)


@pytest.mark.parametrize("n", [1, 2048, 2049, 20000, 23000])
@pytest.mark.parametrize("shift", [0, 1])
def test_round_trip(M, n, shift):
    w = _workload(n)
    a, b = M.Sim(w), M.Sim(w)
    a.step(300 if n <= 4000 else 9000)
    s = a.state()
    s["t"] += shift                              # the other slot buffer
    a.write_state(s)
    b.step(7)
    b.write_state(s)
    _equal(s, a.state())
    _equal(s, b.state())
    a.step(40)
    b.step(40)
    _equal(a.state(), b.state())
    assert a.n_active == b.n_active


def test_long_lanes_and_ties(M, oracle_mod):
    """An 8 km edge with hundreds of vehicles a lane, written in id order (far from lane order)."""
    from test_gpu_parity import compare_states
    w = W.single_edge_workload(length=8000.0, lanes=2, n_vehicles=1500)
    perm = np.random.default_rng(1).permutation(1500)
    x = np.empty(1500, np.float32)
    x[perm] = (np.arange(1500) // 2 * 10.0 + 100.0).astype(np.float32)       # two lanes side by side: equal positions
    lane = np.empty(1500, np.int32)
    lane[perm] = np.arange(1500) % 2
    n = 1500
    s = dict(status=np.ones(n, np.uint8), edge=w.route_edges.copy(), lane=lane, cursor=np.zeros(n, np.int32), x=x,
             v=np.full(n, 2.0, np.float32), held_since=np.full(n, -1, np.int32), mand=np.zeros(n, np.uint8),
             ww=np.zeros(n, np.int32), tau_in=np.zeros(n), t_arr=np.full(n, -1.0), counters=None, t=10)
    g, o = M.Sim(w), oracle_mod.OracleSim(w)
    g.write_state(s)
    o.write_state(10, s)
    got = g.state()
    _equal({k: v for k, v in s.items() if k != "counters"}, got)
    g.step(30)
    o.step(30)
    assert compare_states(g.state(), o.state(), "step 40")


@pytest.mark.parametrize("n", [500, 23000])
def test_skipped_fields(M, n):
    w = _workload(n)
    sim = M.Sim(w)
    sim.step(200 if n <= 4000 else 7000)
    full = sim.state()
    x, lane = np.empty(n, np.float32), np.empty(n, np.int32)
    st = M.SimState()
    st.x, st.lane = x.ctypes.data, lane.ctypes.data
    assert M._lib.sim_read_state(sim._h, ctypes.byref(st)) == 0
    assert np.array_equal(x, full["x"]) and np.array_equal(lane, full["lane"]) and st.t == full["t"]


@pytest.mark.parametrize("what", ["overlap", "nan", "queue"])
def test_refusal_of_a_large_state(M, what):
    w = _workload(23000)
    sim, twin = M.Sim(w), M.Sim(w)
    sim.step(9000)
    twin.step(9000)
    s = sim.state()
    bad = {k: (np.array(v, copy=True) if isinstance(v, np.ndarray) else v) for k, v in s.items()}
    act = np.nonzero(s["status"] == 1)[0]
    if what == "overlap":
        key = s["edge"][act].astype(np.int64) * 8 + s["lane"][act]
        order = np.lexsort((-s["x"][act], key))
        k = next(j for j in range(order.size - 1) if key[order[j]] == key[order[j + 1]])
        lead, fol = int(act[order[k]]), int(act[order[k + 1]])
        bad["x"][fol] = np.float32(s["x"][lead] - 1.0)
        words = f"vehicles {lead} and {fol} overlap"
    elif what == "nan":
        bad["v"][act[3]] = np.nan
        bad["v"][act[9]] = np.inf
        words = f"vehicle {act[3]}: x or v out of range"
    else:
        gone = np.nonzero(s["status"] == 2)[0]
        q = W.entry_lanes(w)
        first = w.route_edges[w.route_off[:-1]]
        key = first[gone].astype(np.int64) * 8 + q[gone]
        order = np.lexsort((gone, w.depart_step[gone], key))
        k = next(j for j in range(order.size - 1) if key[order[j]] == key[order[j + 1]])
        v = int(gone[order[k]])
        bad["status"][v], bad["cursor"][v] = 0, 0
        words = f"vehicle {gone[order[k + 1]]} departed before"
    for _ in range(2):
        with pytest.raises(M.SimError) as ei:
            sim.write_state(bad)
        assert ei.value.name == "SIM_EINVAL" and words in str(ei.value), str(ei.value)
    sim.step(25)
    twin.step(25)
    _equal(sim.state(), twin.state())
    sim.write_state(s)
    _equal(s, sim.state())

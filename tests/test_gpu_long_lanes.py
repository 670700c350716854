"""Written states with long lanes: ranks looked up in sorted chunks of 1,024 on lanes of more than 256 vehicles, lanes
that end at, before and behind a chunk's end, long and short lanes side by side; lanes with more vehicles than they
can hold are refused without a comparison of every pair."""
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


def _lanes(counts):
    """A ring of one-lane edges with counts[e] vehicles on edge e, ids in no order: (workload, state)."""
    n_edges, n = len(counts), int(np.sum(counts))
    w = W.ring_road(n, n_nodes=n_edges, edge_len=8.0 * max(counts) + 100.0, laps=1)
    rng = np.random.default_rng(n)
    fwd = w.route_edges[:n_edges]                                   # edge of each place around the ring
    place = rng.permutation(np.repeat(np.arange(n_edges), counts))
    cursor = (place - np.arange(n) % n_edges) % n_edges
    x = np.empty(n, np.float32)
    for e in range(n_edges):
        ids = rng.permutation(np.nonzero(place == e)[0])
        x[ids] = (np.arange(ids.size) * 7.5 + 20.0 + rng.uniform(0, 1.5, ids.size)).astype(np.float32)
    return w, dict(status=np.ones(n, np.uint8), edge=fwd[place], lane=np.zeros(n, np.int32), cursor=cursor.astype(np.int32),
                   x=x, v=np.full(n, 1.0, np.float32), held_since=np.full(n, -1, np.int32), mand=np.zeros(n, np.uint8),
                   ww=np.zeros(n, np.int32), tau_in=np.zeros(n), t_arr=np.full(n, -1.0), counters=None, t=10)


@pytest.mark.parametrize("counts", [[255, 256, 257, 1], [1024, 1024], [1023, 1025, 3], [300, 724, 300, 5, 9, 2000, 40],
                                    [1, 9000, 1, 257], [257] * 24])
def test_order(M, oracle_mod, counts):
    from test_gpu_parity import compare_states
    w, s = _lanes(counts)
    g, o = M.Sim(w), oracle_mod.OracleSim(w)
    for shift in (0, 1):                                            # both slot buffers
        s["t"] = 10 + shift
        g.write_state(s)
        got = g.state()
        for k in s:
            if k != "counters":
                assert np.array_equal(np.asarray(s[k]), np.asarray(got[k])), k
    o.write_state(11, s)
    g.step(12)
    o.step(12)
    assert compare_states(g.state(), o.state(), "step 23")


@pytest.mark.parametrize("apart", [1, 700, 3000])
def test_overlap_on_a_long_lane_is_refused(M, apart):
    w, s = _lanes([5000, 10])
    sim = M.Sim(w)
    sim.write_state(s)
    lane = np.nonzero(s["edge"] == np.bincount(s["edge"]).argmax())[0]
    order = lane[np.argsort(-s["x"][lane])]
    bad = dict(s, x=s["x"].copy())
    bad["x"][order[apart]] = bad["x"][order[apart - 1]]             # equal positions: the larger id is ahead
    a, b = sorted((int(order[apart - 1]), int(order[apart])), reverse=True)
    with pytest.raises(M.SimError) as ei:
        sim.write_state(bad)
    assert ei.value.name == "SIM_EINVAL" and f"vehicles {a} and {b} overlap" in str(ei.value)
    got = sim.state()
    assert all(np.array_equal(s[k], got[k]) for k in s if k not in ("counters", "t"))


def _best(f, k=5):
    t = []
    for _ in range(k):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return min(t)


def test_time_of_a_long_lane(M):
    """32,000 vehicles on one lane against the same on 160 lanes (a comparison of every pair: six times)."""
    (w1, s1), (w2, s2) = _lanes([32000, 1]), _lanes([200] * 160)
    a, b = M.Sim(w1), M.Sim(w2)
    one, many = _best(lambda: a.write_state(s1)), _best(lambda: b.write_state(s2))
    print("one lane, 160 lanes [us]:", one * 1e6, many * 1e6)
    assert one < 3.0 * many


def test_time_of_a_refusal(M):
    """128,000 vehicles on one lane of 200 m are refused in the time of a few accepted writes of as many (and of sorting
    them on the host to name two that overlap), not of comparing every pair."""
    n = 128000
    w = W.single_edge_workload(length=200.0, n_vehicles=n)
    sim = M.Sim(w)
    ok = sim.state()
    bad = dict(ok, status=np.ones(n, np.uint8), x=np.linspace(1, 190, n).astype(np.float32))

    def refused():
        with pytest.raises(M.SimError) as ei:
            sim.write_state(bad)
        assert ei.value.name == "SIM_EINVAL" and "overlap" in str(ei.value)
    t_ok, t_bad = _best(lambda: sim.write_state(ok)), _best(refused)
    after = sim.state()
    assert all(np.array_equal(np.asarray(ok[k]), np.asarray(after[k])) for k in ok)
    print("accepted, refused [us]:", t_ok * 1e6, t_bad * 1e6)
    assert t_bad < 10.0 * t_ok

"""The reverse sweep's two forms (one launch per segment on a small network, three kernels per step otherwise) and the
register sizes of its parameter sums (1, 4 and 16 classes), against the oracle's FP64 adjoint of the same decisions:
1e-3 relative, the contract of the differentiable form.  Segments that end inside the run, and the same bits for any
checkpoint interval."""
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


def _workload(net_kind, classes, n):
    w = W.config1(n_vehicles=n, n_classes=classes)
    w.params = W.jitter_params(w.params, 0.1, seed=classes)
    if net_kind == "large":                          # 728 edges of 3 lanes: past one workgroup's tables
        w.net = W.grid_network(14, 14, lanes=3)
        rng = np.random.default_rng(2)
        o = rng.integers(0, 196, n)
        w.route_off, w.route_edges, ok = W.shortest_routes(w.net, o, (o + rng.integers(1, 196, n)) % 196)
        assert ok.all()
    w.depart_step = (w.depart_step // 3).astype(np.int32)
    return w


@pytest.mark.parametrize("net_kind", ["small", "large"])
@pytest.mark.parametrize("classes", [1, 2, 4, 5, 16])
def test_gradient(M, oracle_mod, net_kind, classes):
    steps = 850
    w = _workload(net_kind, classes, 1200)
    grads = []
    for every in (100, 64):
        w.params.record_every = every
        sim = M.Sim(w)
        sim.step(steps)
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
    rel = np.linalg.norm(grads[0] - og) / np.linalg.norm(og)
    print("relative gradient error vs FP64 adjoint:", rel)
    assert rel <= 1e-3

"""Routes where a few edges cost many times the mean (jammed or closed roads): no waiting node is below the raised
threshold and the label trees start again from the smallest waiting label, with 512 and with 1,024 threads.  The CPU
tests of the kernel's rounds show that these costs get there.  Routes equal the oracle's edge for edge."""
import numpy as np
import pytest

import workloads as W
from test_route_rounds import gap_costs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    assert torch.cuda.is_available()
    import paper_2007_03614_amd as M
    return M


@pytest.mark.parametrize("size", ["small", "large"])          # 400 nodes; above 16,384
@pytest.mark.parametrize("kind", ["corner 40", "corner 1e6", "way in", "chain", "jams"])
def test_gaps_above_the_threshold_step(M, oracle_mod, kind, size):
    shape = {"small": (20, 20), "large": (130, 130)}[size]
    if kind == "chain":
        shape = (2, shape[0] * shape[1] // 2)
    net = W.grid_network(*shape)
    n = net.n_nodes
    rng = np.random.default_rng(3)
    cost, dest = gap_costs(net, kind, rng)
    o = np.concatenate([[0, 7, n // 2 - 1, n - 2, n - 1, 0, n - 1], rng.integers(0, n, 12)]).astype(np.int32)
    d = np.concatenate([[dest] * 5, [n - 1, 5], np.full(6, dest), rng.integers(0, n, 6)]).astype(np.int32)
    keep = o != d
    o, d = o[keep], d[keep]
    off, edges = M.shortest_routes(net, cost, o, d)
    assert off[-1] == edges.size
    for q in range(o.size):
        assert edges[off[q]:off[q + 1]].tolist() == oracle_mod.route(net, cost, int(o[q]), int(d[q])), q

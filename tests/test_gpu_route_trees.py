"""The label trees in LDS (networks of at most 40,400 nodes and 8 out-edges a
node) where they can go wrong: the node limit from both sides, nodes whose
in-edges fill several records and overflow a frontier list, parallel edges, and
costs of very different size.  Routes equal the oracle's edge for edge."""
from types import SimpleNamespace

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


def _check(M, oracle_mod, net, cost, o, d):
    o, d = np.asarray(o, np.int32), np.asarray(d, np.int32)
    off, edges = M.shortest_routes(net, cost, o, d)
    assert off[-1] == edges.size
    for q in range(o.size):
        assert edges[off[q]:off[q + 1]].tolist() == oracle_mod.route(net, cost, int(o[q]), int(d[q])), q


@pytest.mark.parametrize("rows,cols", [(200, 202), (201, 201)])
@pytest.mark.parametrize("kind", ["uniform", "perturbed"])
def test_node_limit(M, oracle_mod, rows, cols, kind):
    net = W.grid_network(rows, cols)
    V = net.n_nodes
    f = 1.0 if kind == "uniform" else np.random.default_rng(rows).uniform(0.5, 2.0, net.n_edges)
    cost = (net.length / net.limit * f).astype(np.float32)
    mid = rows // 2 * cols + cols // 2
    _check(M, oracle_mod, net, cost, [0, V - 1, cols - 1, 0, mid], [V - 1, 0, V - cols, mid, V - 1])


def _network(edges, n_nodes):
    fr, to = np.array(sorted(set(edges)), np.int32).T
    return SimpleNamespace(edge_from=fr, edge_to=to, n_nodes=n_nodes, n_edges=fr.size,
                           length=np.full(fr.size, 100.0, np.float32), limit=np.full(fr.size, 10.0, np.float32))


@pytest.mark.parametrize("tails", [3, 4, 5, 7, 8, 1023, 1024, 1025, 5000])
def test_many_in_edges(M, oracle_mod, tails):
    """Nodes 1..tails lead into node 0, and node k into node k + 1: an edge straight to 0 or around by its
    neighbours.  Records of four in-edges, and more waiting nodes than a list's 1,024."""
    edges = [(k, 0) for k in range(1, tails + 1)] + [(k, k + 1) for k in range(1, tails)] + [(0, 1)]
    net = _network(edges, tails + 1)
    cost = np.random.default_rng(tails).uniform(1.0, 30.0, net.n_edges).astype(np.float32)
    o = np.unique(np.linspace(1, tails, min(tails, 40)).astype(np.int32))
    _check(M, oracle_mod, net, cost, np.concatenate([o, o[-1:]]), np.concatenate([np.zeros(o.size, np.int32), [1]]))


@pytest.mark.parametrize("scale", [1e-30, 1.0, 1e30])
def test_costs_of_very_different_size(M, oracle_mod, scale):
    net = W.grid_network(12, 13)
    rng = np.random.default_rng(5)
    cost = (scale * 10.0 ** rng.uniform(-3.0, 3.0, net.n_edges)).astype(np.float32)
    o = rng.integers(0, net.n_nodes, 200)
    d = rng.integers(0, net.n_nodes, 200)
    d[o == d] = (d[o == d] + 1) % net.n_nodes
    _check(M, oracle_mod, net, cost, o, d)


def test_parallel_edges(M):
    """Two edges between the same nodes, the dearer first: the cheaper one; equal: the lower id."""
    net = SimpleNamespace(edge_from=np.array([0, 0, 1, 1], np.int32), edge_to=np.array([1, 1, 2, 2], np.int32),
                          n_nodes=3, n_edges=4, length=np.full(4, 100.0, np.float32),
                          limit=np.full(4, 10.0, np.float32))
    off, edges = M.shortest_routes(net, np.array([5, 4, 3, 3], np.float32), np.array([0], np.int32),
                                   np.array([2], np.int32))
    assert off.tolist() == [0, 2] and edges.tolist() == [1, 2]

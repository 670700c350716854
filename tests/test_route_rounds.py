"""The rounds of the label-tree kernel on the CPU: its source compiled for the host, each thread of a workgroup a
coroutine that runs from barrier to barrier (route_tree_host.cpp), with one thread as far ahead of the others as the
barriers allow.  Every thread passes the same barriers and the routes equal the oracle's where an edge costs many times
the mean, so that no waiting node is below the raised threshold and it starts again from the smallest label."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("route_tree")
    with open(os.path.join(ROOT, "paper_2007_03614_amd", "csrc", "routing.hpp")) as f:
        src = f.read()
    src = src.replace("#include <hip/hip_runtime.h>", "").replace("#pragma once", "")
    src = src.replace("extern __shared__", "extern").replace("__shared__", "static")
    (d / "kernels.inc").write_text(src)
    so = str(d / "route_tree.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-fno-strict-aliasing", "-ffp-contract=off",
                           "-w", f'-DKERNELS="{d}/kernels.inc"', os.path.join(ROOT, "tests", "route_tree_host.cpp"),
                           "-o", so])
    L = ctypes.CDLL(so)
    L.route_tree_step.restype = ctypes.c_float
    return L


def _step(lib, cost):
    return lib.route_tree_step(cost.ctypes.data_as(ctypes.c_void_p), cost.size)


IN = np.dtype([("tail", np.int32, 4), ("cost", np.float32, 4)])
OUT = np.dtype([("head", np.int32), ("cost", np.float32)])


def _arrays(net, cost):
    V, E = net.n_nodes, net.n_edges
    order = np.lexsort((np.arange(E), net.edge_from))
    off = np.zeros(V + 1, np.int32)
    off[1:] = np.cumsum(np.bincount(net.edge_from, minlength=V))
    out = np.zeros(E, OUT)
    out["head"], out["cost"] = net.edge_to[order], cost[order]
    rec = np.zeros(V, IN)                # nodes of at most four in-edges: one record each
    rec["tail"] = -1
    fill = np.zeros(V, int)
    for e in range(E):
        v = net.edge_to[e]
        rec[v]["tail"][fill[v]], rec[v]["cost"][fill[v]] = net.edge_from[e], cost[e]
        fill[v] += 1
    return order, off, out, rec


def _run(lib, net, cost, queries, nt, order):
    """The kernel's routes of (origin, destination) pairs, and how often the threshold started again."""
    perm, off, out, rec = _arrays(net, cost)
    V = net.n_nodes
    dests = sorted({d for _, d in queries})
    qord = np.argsort([dests.index(d) for _, d in queries], kind="stable").astype(np.int32)
    qoff = np.searchsorted([dests.index(queries[i][1]) for i in qord], range(len(dests) + 1)).astype(np.int32)
    origin = np.array([o for o, _ in queries], np.int32)
    dests = np.array(dests, np.int32)
    tab = np.full((dests.size, V), -9, np.int32)
    length = np.full(len(queries), -9, np.int32)
    jumps, lines = ctypes.c_int(0), (ctypes.c_int * 2)()
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    rc = lib.route_tree(nt, order, dests.size, V, p(rec), p(off), p(out), p(dests), min(V + 1, 1024),
                        ctypes.c_float(_step(lib, cost)), p(tab), p(qoff), p(qord), p(origin), p(length), ctypes.byref(jumps), lines)
    assert rc == 0, f"threads wait at the barriers of lines {lines[0]} and {lines[1]}"
    routes = []
    for i, (o, d) in enumerate(queries):
        row, v, r = tab[dests.tolist().index(d)], o, []
        while v != d:
            r.append(int(perm[row[v]]))
            v = int(net.edge_to[r[-1]])
        assert length[i] == len(r)
        routes.append(r)
    return routes, jumps.value


def gap_costs(net, kind, rng):
    """Travel times with a few edges many times the mean: (costs, destination)."""
    cost = (net.length / net.limit * rng.uniform(0.5, 2.0, net.n_edges)).astype(np.float32)
    n = net.n_nodes
    if kind in ("corner 40", "corner 1e6"):          # the last node's only ways out are jammed or closed
        cost[net.edge_from == n - 1] = np.float32(kind.split()[1]) * cost.mean()
        return cost, 0
    if kind == "way in":                             # the only ways into the destination
        cost[net.edge_to == n - 1] *= np.float32(400.0)
        return cost, n - 1
    if kind == "chain":                              # several gaps one after another along a street of two rows
        band = np.arange(n) % (n // 2) * 5 // (n // 2)
        cost[band[net.edge_from] != band[net.edge_to]] *= np.float32(2000.0)
        return cost, 0
    assert kind == "jams"                            # 2 % of the edges at 30 times their time
    cost[rng.random(net.n_edges) < 0.02] *= np.float32(30.0)
    return cost, n // 2


@pytest.mark.parametrize("order", [1, -1])
@pytest.mark.parametrize("kind", ["corner 40", "corner 1e6", "way in", "chain", "jams"])
def test_gaps_above_the_threshold_step(lib, oracle_mod, kind, order):
    net = W.grid_network(2, 200) if kind == "chain" else W.grid_network(20, 20)
    rng = np.random.default_rng(3)
    cost, dest = gap_costs(net, kind, rng)
    n = net.n_nodes
    queries = [(o, dest) for o in (0, 7, n // 2 - 1, n - 2, n - 1) if o != dest] + [(0, n - 1), (n - 1, 5)]
    routes, jumps = _run(lib, net, cost, queries, 256, order)
    assert jumps > 0 or kind == "jams"
    for (o, d), r in zip(queries, routes):
        assert r == oracle_mod.route(net, cost, o, d)


@pytest.mark.parametrize("price", [1e6, 1e30])
def test_step_without_closed_roads(lib, price):
    """Closed roads leave the threshold step as it is (to the mean's sampling), and costs without any are all in it."""
    rng = np.random.default_rng(4)
    for n in (1, 2, 5, 40000):
        cost = rng.uniform(1.0, 40.0, n).astype(np.float32)
        plain = _step(lib, cost)
        assert plain == pytest.approx(16.0 * cost.mean(dtype=np.float64), rel=1e-6)
        for share in (0.0, 0.01, 0.05):
            c = cost.copy()
            c[rng.permutation(n)[:int(share * n)]] = price
            assert _step(lib, c) == pytest.approx(plain, rel=0.02)
    two = np.concatenate([cost, [1e3, 1e5, 1e9]]).astype(np.float32)
    assert _step(lib, two) == pytest.approx(plain, rel=0.02)

"""The work that a program using this package has it do, as cases that can be timed.

``listed()`` names the standing cases, ``draw(rng)`` makes more of the same ranges, ``prepare(case, seed)``
builds what a program holds before the call (a handle in mid-run, a saved state, edge costs), ``run(state)``
makes one pass through the public entry points and ``work(case)`` says what that pass cannot do without.

Road networks and routed trips are the city: they are the same for every seed and made once per process.
The seed draws what changes from day to day: departures, driver classes, anticipation times, positions,
observed costs, queries.
"""
import ctypes
import functools
import math

import numpy as np
import torch

import workloads as W

RING_EDGE_M, RING_EDGES = 100.0, 10
BYTES_PER_UPDATE = 28        # x, v, id and lane word read, x, v and lane word written
FLOPS_PER_UPDATE = 60        # Eq. (1) and the integration of one vehicle
STATE_BYTES = 50             # one vehicle's record in a read or written state


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # a one-lane ring road, stepped and read out every step: a live view or a controller in the loop
        dict(name="ring_live", kind="ring", vehicles=50, steps=1),
        # one minute from a saved state of the 10x10 grid: the smallest what-if question
        dict(name="grid_minute", kind="window", net="grid", vehicles=2000, start=600, steps=120, classes=1, mode=0,
             spread=0.0),
        # a town (30x30 blocks and its ring highway) five minutes on from a saved state
        dict(name="town_window", kind="window", net="town", rows=30, vehicles=15000, start=10200, steps=600, classes=1,
             mode=0, spread=0.0),
        # the perturbed 100x100 grid with ring highway, 200,000 trips, from its 08:00 state
        dict(name="city_window", kind="window", net="town", rows=100, vehicles=200000, start=10800, steps=900,
             classes=1, mode=0, spread=0.0),
        # a smaller city with every node flashing red, four driver classes, each driver at a speed of its own
        dict(name="city_flashing", kind="window", net="town", rows=60, vehicles=60000, start=9000, steps=600, classes=4,
             mode=1, spread=0.05),
        # the whole metropolitan lattice, half a million vehicles on the road, from a saved state
        dict(name="metro_window", kind="window", net="metro", rows=473, density=0.05, steps=900, classes=4, mode=0,
             spread=0.0),
        # queues everywhere, 30 % of jam density on every lane: travel times read every 30 s of simulated time
        dict(name="dense_feed", kind="feed", rows=120, density=0.3, steps=60),
        # 32 what-if scenarios of the 10x10 grid in one handle, means read every minute
        dict(name="scenarios", kind="scenarios", members=32, vehicles=13000, steps=120),
        # one iteration of the calibration loop: five parameter sets, flashing red, means of the edges
        dict(name="calibration_sets", kind="sets", members=5, vehicles=2000, steps=1200),
        # the gradient of the mean travel times with respect to the parameters of four classes
        dict(name="gradient", kind="gradient", vehicles=2000, classes=4, steps=1200, record=120),
        # re-routing a city's trips on current travel times
        dict(name="routes_city", kind="routes", net="town", rows=100, queries=200000, dests=0),
        # the same on a metropolitan lattice, to its busiest destinations
        dict(name="routes_metro", kind="routes", net="metro", rows=200, queries=20000, dests=400),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ring", "grid", "town", "metro", "feed", "scenarios", "sets", "gradient", "routes", "routes"])
    if kind == "ring":
        return dict(kind="ring", vehicles=rng.randint(20, 100), steps=_log(rng, 1, 64))
    if kind == "grid":
        return dict(kind="window", net="grid", vehicles=_log(rng, 300, 4000), start=rng.randint(200, 900),
                    steps=rng.randint(40, 600), classes=rng.choice([1, 4]), mode=rng.choice([0, 0, 1]),
                    spread=rng.choice([0.0, 0.0, 0.05]))
    if kind == "town":
        rows = rng.randint(15, 60)
        return dict(kind="window", net="town", rows=rows, vehicles=rng.randint(8, 20) * rows * rows,
                    start=rng.randint(7200, 12000), steps=rng.randint(100, 900), classes=rng.choice([1, 4]),
                    mode=rng.choice([0, 0, 1]), spread=rng.choice([0.0, 0.0, 0.05]))
    if kind == "metro":
        return dict(kind="window", net="metro", rows=_log(rng, 40, 300), density=round(rng.uniform(0.04, 0.12), 3),
                    steps=rng.randint(100, 900), classes=4, mode=rng.choice([0, 0, 1]),
                    spread=rng.choice([0.0, 0.0, 0.05]))
    if kind == "feed":
        return dict(kind="feed", rows=rng.randint(40, 130), density=round(rng.uniform(0.2, 0.3), 3),
                    steps=rng.randint(20, 120))
    if kind == "scenarios":
        return dict(kind="scenarios", members=_log(rng, 2, 48), vehicles=rng.randint(6000, 16000),
                    steps=rng.randint(30, 240))
    if kind == "sets":
        return dict(kind="sets", members=rng.randint(2, 5), vehicles=rng.randint(500, 3000),
                    steps=rng.randint(300, 1800))
    if kind == "gradient":
        return dict(kind="gradient", vehicles=rng.randint(300, 2000), classes=rng.choice([1, 2, 4]),
                    steps=rng.randint(240, 1200), record=rng.choice([60, 100, 120]))
    if rng.random() < 0.6:
        return dict(kind="routes", net="town", rows=rng.randint(10, 100), queries=_log(rng, 500, 100000), dests=0)
    return dict(kind="routes", net="metro", rows=rng.randint(130, 200), queries=_log(rng, 500, 20000),
                dests=rng.randint(50, 400))


# --------------------------------------------------------------------------- the city
@functools.lru_cache(maxsize=None)
def _metro(rows):
    return W.metro_network(rows=rows, cols=rows, n_segments=int(round(274_504 * rows * rows / (473 * 474))))


@functools.lru_cache(maxsize=None)
def _town_net(rows):
    return W.perturbed_grid_ring(rows=rows, cols=rows)


@functools.lru_cache(maxsize=None)
def _town_trips(rows, vehicles):
    return W.scaled_config2(vehicles, rows, rows, 21_600)


@functools.lru_cache(maxsize=None)
def _grid_trips(vehicles):
    return W.config1(n_vehicles=vehicles)


def _drivers(w, rng, classes, spread=0.0, mode=0, record=0):
    """The workload with this day's drivers: trips in another order, classes and anticipation times."""
    n = w.n_vehicles
    perm = rng.permutation(n)
    lens = np.diff(w.route_off)[perm]
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(lens)
    at = np.repeat(w.route_off[:-1][perm] - off[:-1], lens) + np.arange(int(off[-1]))
    p = W.jitter_params(W.base_params(classes, int(rng.integers(1 << 30))), 0.1 if classes > 1 else 0.0,
                        int(rng.integers(1 << 30)))
    p.intersection_mode, p.v0_spread, p.record_every = mode, spread, record
    return W.Workload(w.name, w.net, off, w.route_edges[at], w.depart_step,
                      rng.integers(0, classes, n).astype(np.uint8), rng.uniform(0.05, 0.40, n).astype(np.float32), p,
                      w.n_steps)


# --------------------------------------------------------------------------- inputs
def prepare(case, seed):
    import paper_2007_03614_amd as M
    torch.cuda.current_device()
    rng = np.random.default_rng([seed, 7])
    return globals()["_prepare_" + case["kind"]](M, case, rng, seed)


def _ring_inputs(case, seed):
    """Vehicles around the ring at nearly even spacing and nearly equal speed: (workload, state)."""
    n, rng = case["vehicles"], np.random.default_rng([seed, 7])
    w = W.ring_road(n, n_nodes=RING_EDGES, edge_len=RING_EDGE_M, laps=600)
    w.params.seed = int(rng.integers(1 << 30))
    around = RING_EDGES * RING_EDGE_M
    gap = around / n
    pos = (np.arange(n) + rng.uniform(-0.2, 0.2, n)) * gap
    pos = np.mod(pos, around)
    # edge numbers follow the ring: step k of any route is k edges on from its first
    k = np.minimum((pos / RING_EDGE_M).astype(np.int64), RING_EDGES - 1)
    first = np.arange(n) % RING_EDGES
    cursor = np.mod(k - first, RING_EDGES)
    x = (pos - k * RING_EDGE_M).astype(np.float32)
    v = (np.clip((gap * 0.8 - 7.0) / 1.6, 0.0, 13.0) * rng.uniform(0.8, 1.0, n)).astype(np.float32)
    s = dict(status=np.ones(n, np.uint8), edge=w.route_edges[w.route_off[:-1] + cursor], lane=np.zeros(n, np.int32),
             cursor=cursor.astype(np.int32), x=x, v=v, held_since=np.full(n, -1, np.int32), mand=np.zeros(n, np.uint8),
             ww=np.zeros(n, np.int32), tau_in=np.full(n, 50.0), t_arr=np.full(n, -1.0), counters=None, t=100)
    return w, s, k


def _prepare_ring(M, case, rng, seed):
    w, s, _ = _ring_inputs(case, seed)
    sim = M.Sim(w)
    sim.write_state(s)
    return dict(kind="ring", sim=sim, steps=case["steps"])


def _filled(M, case, seed, route, settle):
    """The metropolitan lattice with vehicles evenly on every lane, after `settle` steps."""
    w, s = W.probe_r(_metro(case["rows"]), density=case["density"], route_len=route, seed=seed)
    w.params.intersection_mode, w.params.v0_spread = case.get("mode", 0), case.get("spread", 0.0)
    sim = M.Sim(w)
    sim.write_state(s)
    sim.step(settle)
    return sim


def _prepare_window(M, case, rng, seed):
    if case["net"] == "metro":
        sim = _filled(M, case, seed, 64, 120)
        return dict(kind="window", sim=sim, saved=sim.state(), steps=case["steps"])
    base = _grid_trips(case["vehicles"]) if case["net"] == "grid" else _town_trips(case["rows"], case["vehicles"])
    sim = M.Sim(_drivers(base, rng, case["classes"], case["spread"], case["mode"]))
    sim.step(case["start"])
    return dict(kind="window", sim=sim, saved=sim.state(), steps=case["steps"])


def _prepare_feed(M, case, rng, seed):
    return dict(kind="feed", sim=_filled(M, case, seed, 32, 600), steps=case["steps"])


def _prepare_scenarios(M, case, rng, seed):
    base = _grid_trips(int(1.2 * case["vehicles"]))
    w = _drivers(base, rng, 1)
    w.depart_step = rng.integers(0, 21_600, w.n_vehicles).astype(np.int32)          # 3 h of steady demand
    scen = W.ensemble_scenarios(case["members"], case["vehicles"], w.net.n_edges, seed)
    sim = M.Sim(w, scenarios=[(n, cut) for n, cut in scen])
    sim.step(600)
    return dict(kind="scenarios", sim=sim, steps=case["steps"])


def _prepare_sets(M, case, rng, seed):
    w = _drivers(_grid_trips(case["vehicles"]), rng, 1, mode=1)
    sets = np.array([[1.0, 1.5, 1.0, 2.0, 2.0]]) * rng.uniform(0.8, 1.2, (case["members"], 5))
    lo, hi = np.array([0.5, 0.1, 1.0, 1.0, 1.0]), np.array([1.2, 2.0, 10.0, 10.0, 5.0])
    sets = np.clip(sets, lo, hi).astype(np.float32)
    return dict(kind="sets", M=M, w=w, steps=case["steps"],
                scenarios=[(w.n_vehicles, np.zeros(0, np.int32), s.reshape(1, 5)) for s in sets])


def _prepare_gradient(M, case, rng, seed):
    w = _drivers(_grid_trips(case["vehicles"]), rng, case["classes"])
    p = w.params
    theta = torch.tensor(np.stack([p.v0_factor, p.T, p.a, p.b, p.s0], 1).astype(np.float64), requires_grad=True)
    target = torch.from_numpy(np.asarray(w.net.length, np.float64) / w.net.limit * rng.uniform(1.0, 1.3, w.net.n_edges))
    return dict(kind="gradient", M=M, w=w, theta=theta, target=target, steps=case["steps"], record=case["record"])


def _prepare_routes(M, case, rng, seed):
    net = _town_net(case["rows"]) if case["net"] == "town" else _metro(case["rows"])
    cost = (net.length / net.limit * rng.uniform(1.0, 3.0, net.n_edges)).astype(np.float32)
    q = case["queries"]
    o = rng.integers(0, net.n_nodes, q)
    pool = rng.choice(net.n_nodes, case["dests"], replace=False) if case["dests"] else np.arange(net.n_nodes)
    d = pool[rng.integers(0, pool.size, q)]
    o = np.where(o == d, (d + 1) % net.n_nodes, o).astype(np.int32)
    d = d.astype(np.int32)
    # a program on the C interface: its network, its queries, and buffers of its own for the routes
    fn = ctypes.CDLL(M.LIB_PATH).sim_shortest_routes
    fn.argtypes = [ctypes.c_void_p] * 2 + [ctypes.c_int32] + [ctypes.c_void_p] * 4 + [ctypes.c_int64, ctypes.c_void_p]
    fn.restype = ctypes.c_int32
    keep = [np.ascontiguousarray(a, t) for a, t in (
        (net.edge_from, np.int32), (net.edge_to, np.int32), (net.length, np.float32), (net.limit, np.float32),
        (net.lanes, np.uint8), (net.conn_off, np.int32), (net.conn_to, np.int32), (net.conn_mask, np.uint8))]
    sn = M.SimNetwork(net.n_nodes, net.n_edges, *[a.ctypes.data for a in keep])
    off = np.zeros(q + 1, np.int64)
    edges = np.zeros(q * int(1.2 * case["rows"] + 40), np.int32)
    total = np.zeros(1, np.int64)
    args = (ctypes.addressof(sn), cost.ctypes.data, q, o.ctypes.data, d.ctypes.data, off.ctypes.data, edges.ctypes.data,
            edges.size, total.ctypes.data)
    return dict(kind="routes", fn=fn, args=args, off=off, edges=edges, total=total, keep=(keep, sn, cost, o, d))


# --------------------------------------------------------------------------- one pass
def run(state):
    kind = state["kind"]
    if kind == "ring":
        state["sim"].step(state["steps"])
        return state["sim"].state()
    if kind == "window":
        sim = state["sim"]
        sim.write_state(state["saved"])
        sim.step(state["steps"])
        return sim.state()
    if kind == "feed":
        state["sim"].step(state["steps"])
        return state["sim"].edge_stats()
    if kind == "scenarios":
        state["sim"].step(state["steps"])
        return state["sim"].mean_travel_times()
    if kind == "sets":
        sim = state["M"].Sim(state["w"], scenarios=state["scenarios"])
        sim.step(state["steps"])
        out = sim.mean_travel_times()
        sim.close()
        return out
    if kind == "gradient":
        theta = state["theta"]
        theta.grad = None
        mean = state["M"].edge_mean_travel_time(theta, state["w"], state["steps"], state["record"])
        ((mean - state["target"]) ** 2 * (mean > 0)).sum().backward()
        return mean.detach(), theta.grad
    if state["fn"](*state["args"]) != 0:
        raise RuntimeError("sim_shortest_routes failed")
    return state["off"], state["edges"], state["total"]


# --------------------------------------------------------------------------- what a pass cannot do without
def _lattice_vehicles(case):
    # lanes per edge of the metropolitan recipe, and its log-normal lengths (median 120 m) in whole vehicles
    edges, lanes = 549_008 * case["rows"] ** 2 / (473 * 474), 1.978
    z = np.arange(-4.0, 4.0, 0.01)
    length = np.clip(120.0 * np.exp(0.5 * z), 25.0, 2000.0)
    wt = np.exp(-0.5 * z * z)
    return edges, edges * lanes * float((np.floor(case["density"] * length / 7.0) * wt).sum() / wt.sum())


def work(case):
    kind, steps = case["kind"], case.get("steps", 0)
    if kind == "ring":
        active, io = case["vehicles"], case["vehicles"] * STATE_BYTES
    elif kind == "window" and case["net"] == "metro":
        active = _lattice_vehicles(case)[1]
        io = 2 * active * STATE_BYTES
    elif kind == "window":
        share = 0.17 if case["net"] == "grid" else 3.2e-4 * case["rows"] ** 1.5   # longer trips in a larger town
        active, io = share * case["vehicles"], 2 * case["vehicles"] * STATE_BYTES
    elif kind == "feed":
        edges, active = _lattice_vehicles(case)
        io = 16 * edges
    elif kind == "scenarios":
        active, io = case["members"] * case["vehicles"] * 0.012, 16 * 360 * case["members"]
    elif kind == "sets":
        active = 0.2 * case["members"] * case["vehicles"]
        io = case["members"] * (case["vehicles"] * STATE_BYTES + 16 * 360)
    elif kind == "gradient":
        # the forward's updates, and once more in reverse with the 64-bit adjoints of x and v
        active, io = 0.15 * case["vehicles"], case["vehicles"] * STATE_BYTES
        return dict(bytes=io + steps * active * (2 * BYTES_PER_UPDATE + 32), flops=steps * active * 3 * FLOPS_PER_UPDATE)
    else:
        nodes = case["rows"] ** 2 if case["net"] == "metro" else 0.99 * case["rows"] ** 2 + 40
        deg = 2.45 if case["net"] == "metro" else 3.56
        dests = case["dests"] or nodes * (1.0 - math.exp(-case["queries"] / nodes))
        hops = 0.68 * math.sqrt(nodes)
        # every destination's label of every node from its out-edges; every route edge written once
        return dict(bytes=12.0 * nodes * deg + 4.0 * case["queries"] * hops + 4.0 * dests * nodes,
                    flops=2.0 * dests * nodes * deg)
    return dict(bytes=io + BYTES_PER_UPDATE * active * steps, flops=FLOPS_PER_UPDATE * active * steps)


# --------------------------------------------------------------------------- the ring in 64 bits
def exact(case, seed):
    """Positions, speeds and edge-entry times of the ring road in 64 bits.  The other cases have no such value:
    traffic at intersections decides by comparisons, and one of them that falls the other way in 64 bits sends the
    run another way; routes are whole numbers."""
    if case["kind"] != "ring":
        return None
    w, s, k = _ring_inputs(case, seed)
    p, n, L, dt = w.params, case["vehicles"], RING_EDGE_M, 0.5
    T, a, b, s0, ln = (float(q[0]) for q in (p.T, p.a, p.b, p.s0, p.veh_len))
    v0 = float(np.float32(w.net.limit[0]))
    x, v, tau = s["x"].astype(np.float64), s["v"].astype(np.float64), s["tau_in"].copy()
    k = k.copy()
    order = np.argsort(k * L + x)                       # around the ring: each one's leader is the next
    lead = np.empty(n, np.int64)
    lead[order] = np.roll(order, -1)
    for t in range(s["t"], s["t"] + case["steps"]):
        same = (k[lead] == k) & (x[lead] > x)
        ahead = (k[lead] == (k + 1) % RING_EDGES) & ~same
        rear = x[lead] - ln
        gap = np.where(same, rear - x, np.where(ahead, L - x + rear, np.inf))
        phi = np.maximum(a * (1.0 - (v / v0) ** 4), -b)
        dyn = np.maximum(v * T + v * (v - v[lead]) / (2.0 * math.sqrt(a * b)), 0.0)
        acc = phi - np.where(np.isfinite(gap), a * ((s0 + dyn) / np.maximum(gap, 0.1)) ** 2, 0.0)
        vn = v + acc * dt
        stop = vn < 0.0
        xn = np.where(stop, x - v * v / (2.0 * np.where(stop, acc, -1.0)), x + v * dt + 0.5 * acc * dt * dt)
        vn = np.maximum(vn, 0.0)
        xn = np.where(same & (xn > rear), rear, xn)
        over = xn >= L
        tau = np.where(over, (t + (L - x) / np.where(over, xn - x, 1.0)) * dt, tau)
        k = np.where(over, (k + 1) % RING_EDGES, k)
        x, v = np.where(over, xn - L, xn), vn
    return dict(status=None, edge=None, lane=None, cursor=None, x=x, v=v, held_since=None, mand=None, ww=None,
                tau_in=tau, t_arr=None, counters=None, t=None)

"""The work that programs have this library do, as cases that can be timed and compared.

Every case goes through the Python binding as a user's program does: link costs, one step of the link-flow
iteration, shortest-path trees, all-or-nothing assignments, whole Frank-Wolfe solves, an interval of a day with
its residual demand, and the calibration pass.  Networks are of the two kinds the benchmark has: square grids
(static assignment, every zone pair) and road-like planar networks numbered along a Hilbert curve, with dead
ends, runs of two-neighbour nodes and three speed tiers (15-minute intervals, gravity-like demand).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2104_12911_amd import qdta

DEV = "cuda"
INF = float("inf")
CAPS = np.array([900.0, 1800.0, 3600.0], dtype=np.float32)
SPEEDS = np.array([40.0, 60.0, 100.0]) / 3.6


# ---------------------------------------------------------------------------
# Networks (the topology is a function of its sizes; the seed draws what varies)
# ---------------------------------------------------------------------------
class Net:
    def __init__(self, n, tail, head, xy, **links):
        order = np.lexsort((head, tail))
        self.n, self.m, self.xy = n, order.size, xy
        self.tail = tail[order].astype(np.int32)
        self.col = head[order].astype(np.int32)
        self.row_ptr = np.zeros(n + 1, dtype=np.int32)
        np.cumsum(np.bincount(self.tail, minlength=n), out=self.row_ptr[1:])
        self.links = {k: v[order] for k, v in links.items()}


@functools.lru_cache(maxsize=4)
def grid(side):
    """side x side nodes, a link each way between neighbours."""
    node = np.arange(side * side)
    right, down = node[node % side < side - 1], node[node < side * (side - 1)]
    tail = np.concatenate([right, right + 1, down, down + side])
    head = np.concatenate([right + 1, right, down + side, down])
    xy = np.stack([node % side, node // side], axis=1) * 500.0
    return Net(side * side, tail, head, xy)


def _hilbert(ix, iy, order):
    ix, iy = ix.astype(np.int64), iy.astype(np.int64)
    d = np.zeros_like(ix)
    s = 1 << (order - 1)
    while s:
        rx, ry = (ix & s) > 0, (iy & s) > 0
        d += s * s * ((3 * rx) ^ ry)
        flip = rx & ~ry
        ix, iy = np.where(flip, s - 1 - ix, ix), np.where(flip, s - 1 - iy, iy)
        ix, iy = np.where(ry, ix, iy), np.where(ry, iy, ix)
        s >>= 1
    return d


def _spanning_edges(n, u, v, w):
    """Which edges are in the minimum spanning tree (Boruvka)."""
    order = np.argsort(w, kind="stable")
    u, v = u[order], v[order]
    comp = np.arange(n)
    live = np.arange(u.size)
    tree = np.zeros(u.size, dtype=bool)
    none = u.size
    while True:
        cu, cv = comp[u[live]], comp[v[live]]
        keep = cu != cv
        live, cu, cv = live[keep], cu[keep], cv[keep]
        if not live.size:
            break
        a, b = np.full(n, none), np.full(n, none)
        a[cu[::-1]] = live[::-1]                 # the last write is the lightest edge
        b[cv[::-1]] = live[::-1]
        best = np.minimum(a, b)
        c = np.nonzero(best < none)[0]
        e = best[c]
        tree[e] = True
        other = comp[u[e]] + comp[v[e]] - c
        up = np.arange(n)
        up[c] = other
        two = (up[up] == np.arange(n)) & (np.arange(n) < up)
        up[two] = np.nonzero(two)[0]
        while not np.array_equal(up, up[up]):
            up = up[up]
        comp = up[comp]
    out = np.zeros(order.size, dtype=bool)
    out[order] = tree
    return out


@functools.lru_cache(maxsize=4)
def road(n, oneway):
    """A road-like planar network of n nodes: the minimum spanning tree of jittered lattice points and the shortest
    other lattice edges up to 1.28 n, with arterials every 2 km and highways every 10 km.  Tree edges are two-way
    (so that every node reaches every other); `oneway` is the share of the others that is one-way."""
    rng = np.random.default_rng(20000 + n)
    kx = max(2, math.ceil(math.sqrt(1.2 * n)))
    step = 148.0
    node = np.arange(n)
    c, r = node % kx, node // kx
    xy = (np.stack([c, r], axis=1) + rng.uniform(-0.4, 0.4, (n, 2))) * step
    right = node[(c < kx - 1) & (node + 1 < n)]
    down = node[node + kx < n]
    u, v = np.concatenate([right, down]), np.concatenate([right + 1, down + kx])
    line = np.concatenate([r[right], c[down]])   # the lattice line an edge runs along
    tier = np.where(line % 68 == 34, 2, np.where(line % 14 == 7, 1, 0)).astype(np.int8)
    length = np.sqrt(((xy[u] - xy[v]) ** 2).sum(1))
    w = np.where(tier > 0, 0.01, 1.0) * length
    tree = _spanning_edges(n, u, v, w)
    rest = np.nonzero(~tree)[0]
    rest = rest[np.argsort(w[rest], kind="stable")][:max(0, int(round(1.28 * n)) - int(tree.sum()))]
    single = rest[(rng.random(rest.size) < oneway) & (tier[rest] < 2)]
    both = np.concatenate([np.nonzero(tree)[0], np.setdiff1d(rest, single)])
    swap = rng.random(single.size) < 0.5
    tail = np.concatenate([u[both], v[both], np.where(swap, v[single], u[single])])
    head = np.concatenate([v[both], u[both], np.where(swap, u[single], v[single])])
    e = np.concatenate([both, both, single])
    at = np.argsort(_hilbert(c, r, max(1, int(kx).bit_length())), kind="stable")
    new = np.empty(n, dtype=np.int64)
    new[at] = node
    net = Net(n, new[tail], new[head], xy[at], tier=tier[e], length=length[e])
    net.kx, net.step, net.new = kx, step, new
    return net


def attributes(net, rng):
    """Free-flow times (s) and capacities (veh/h) of a network's links."""
    if not net.links:
        return rng.uniform(30.0, 120.0, net.m).astype(np.float32), rng.choice(CAPS, net.m)
    tier = net.links["tier"]
    t = net.links["length"] / SPEEDS[tier] * rng.uniform(0.9, 1.2, net.m)
    return np.maximum(t, 0.5).astype(np.float32), CAPS[tier]


def zones_of(net, count):
    pick = np.random.default_rng(30000 + count).choice(net.n, min(count, net.n), replace=False)
    return np.sort(pick).astype(np.int32)


def grid_demand(net, zones, rng, mean=20.0):
    """About Poisson(mean) trips for every ordered zone pair."""
    o, d = np.repeat(zones, zones.size), np.tile(zones, zones.size)
    keep = o != d
    return o[keep], d[keep], np.maximum(rng.poisson(mean, int(keep.sum())), 1).astype(np.float64)


def road_demand(net, zones, legs, carried, trips, rng):
    """`legs` zone-to-zone legs, nearer zones more often, and `carried` legs of trips already under way, from any
    node some kilometres from their destination (what earlier intervals leave).  Who travels where goes with the
    network, how many trips with the seed."""
    pairs = np.random.default_rng([zones.size, legs, carried])
    d = zones[pairs.integers(0, zones.size, legs)]
    cand = zones[pairs.integers(0, zones.size, (6, legs))]
    far = np.where(cand == d, INF, ((net.xy[cand] - net.xy[d]) ** 2).sum(2))
    o = cand[np.argmin(far, axis=0), np.arange(legs)]
    t = 1.0 + rng.poisson(max(trips - 1.0, 0.0), legs)
    if carried:
        d2 = zones[pairs.integers(0, zones.size, carried)]
        ang, rad = pairs.uniform(0, 2 * np.pi, carried), pairs.exponential(10_000.0, carried)
        p = np.rint((net.xy[d2] + rad[:, None] * np.stack([np.cos(ang), np.sin(ang)], axis=1)) / net.step)
        c = np.clip(p[:, 0], 0, net.kx - 1).astype(np.int64)
        r = np.clip(p[:, 1], 0, (net.n - 1) // net.kx).astype(np.int64)
        o2 = net.new[np.minimum(r * net.kx + c, net.n - 1)].astype(np.int32)
        t2 = np.maximum(rng.exponential(0.3, carried), 0.001)
        o, d, t = np.concatenate([o, o2]), np.concatenate([d, d2]), np.concatenate([t, t2])
    return o, d, t


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one evaluation of the link costs of the small test grid, in a caller's own loop: the smallest call
        dict(name="costs_grid20", op="costs", net="grid", side=20, zones=40, so=False),
        # the link-flow half of an iteration (step size, update) on the benchmark's regional network
        dict(name="step_region", op="step", net="road", n=550_000, oneway=1.0, zones=10, so=False, ls="ksection"),
        # the same on the metro network with the other line search and the other objective
        dict(name="step_metro_qn_so", op="step", net="road", n=100_000, oneway=0.0, zones=10, so=True, ls="qn"),
        # complete trees to every zone of the small grid: accessibility tables, and what latency costs
        dict(name="trees_grid20", op="trees", net="grid", side=20, dests=40, free=True),
        # complete trees of the metro network to a handful of destinations, under congested costs
        dict(name="trees_metro", op="trees", net="road", n=100_000, oneway=0.0, dests=100, free=False),
        # static assignment of one uneven, heavily loaded grid under the costs of a later iteration
        dict(name="aon_grid151", op="aon", net="grid", side=151, zones=300, rule="ceil", dt=INF, load=4.0),
        # the metro interval of the benchmark: 1,000 destinations, truncated at 15 minutes
        dict(name="aon_metro", op="aon", net="road", n=100_000, oneway=0.0, zones=1000, legs=316_000, carried=0,
             rule="ceil", dt=900.0, load=1.0),
        # the regional peak interval: 5,000 destinations, carried legs: the largest call
        dict(name="aon_region", op="aon", net="road", n=550_000, oneway=1.0, zones=5000, legs=261_000, carried=939_000,
             rule="ceil", dt=900.0, load=1.0),
        # a whole small static solve: an iteration is a chain of small launches
        dict(name="solve_grid20", op="solve", net="grid", sides="20", zones=40, iters=50, ls="ksection", so=False),
        # several uneven grids advanced together in one context
        dict(name="solve_batch8", op="solve", net="grid", sides="51,64,77,99,112,131,150,180", zones=150, iters=3,
             ls="ksection", so=False),
        # one interval of a day on the 1/20-scale network: demand in, solve, residual demand out
        dict(name="interval_town", op="interval", net="road", n=27_500, oneway=1.0, zones=250, legs=13_000,
             carried=60_000, rule="ceil", iters=6, ls="ksection"),
        # one step of an OD calibration through the frozen-path model: forward and backward
        dict(name="calib_metro", op="calib", net="road", n=100_000, oneway=0.0, zones=300, legs=60_000, dt=900.0,
             iters=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["costs", "step", "trees", "aon", "aon", "solve", "interval", "calib"])
    is_grid = rng.random() < 0.5
    one = rng.choice([0.0, 0.5, 1.0])
    rule = rng.choice(["ceil", "ceil", "floor", "none", "progress"])
    so, ls = rng.random() < 0.25, rng.choice(["ksection", "ksection", "qn", "msa"])
    where = dict(net="road", n=_log(rng, 300, 550_000), oneway=one)
    if is_grid:
        where = dict(net="grid", side=_log(rng, 3, 224))
    if op == "costs":
        return dict(op=op, **where, zones=8, so=so)
    if op == "step":
        return dict(op=op, **where, zones=8, so=so, ls=rng.choice(["ksection", "qn"]))
    if op == "trees":
        n = where.get("n") or where["side"] ** 2
        return dict(op=op, **where, dests=_log(rng, 1, max(2, min(1000, 10_000_000 // n, n))), free=rng.random() < 0.5)
    if op == "aon" and is_grid:
        return dict(op=op, **where, zones=_log(rng, 2, 600), rule="ceil", dt=INF, load=rng.choice([0.0, 1.0, 4.0]))
    if op == "aon":
        where["n"] = _log(rng, 300, 300_000)
        zones = _log(rng, 2, 2500)
        return dict(op=op, **where, zones=zones, legs=zones * _log(rng, 5, 100), carried=zones * _log(rng, 1, 200),
                    rule=rule, dt=rng.choice([450.0, 900.0]), load=rng.choice([0.0, 1.0]))
    if op == "solve":
        sides = [str(_log(rng, 5, 160)) for _ in range(rng.randint(1, 6))]
        return dict(op=op, net="grid", sides=",".join(sides), zones=_log(rng, 3, 150), iters=rng.randint(2, 5), ls=ls,
                    so=so)
    if op == "interval":
        zones = _log(rng, 10, 400)
        return dict(op=op, net="road", n=_log(rng, 1000, 60_000), oneway=one, zones=zones,
                    legs=zones * _log(rng, 5, 60), carried=zones * _log(rng, 1, 200), rule=rule, iters=rng.randint(1, 6), ls=ls)
    zones = _log(rng, 5, 300)
    return dict(op=op, net="road", n=_log(rng, 1000, 100_000), oneway=one, zones=zones, legs=zones * _log(rng, 10, 200),
                dt=rng.choice([900.0, INF]), iters=rng.randint(1, 4))


RULES = {"none": qdta.RULE_NONE, "ceil": qdta.RULE_CEIL, "floor": qdta.RULE_FLOOR, "progress": qdta.RULE_PROGRESS}
SEARCH = {"ksection": qdta.LS_KSECTION, "qn": qdta.LS_QN, "msa": qdta.LS_MSA}


def _options(case):
    kw = {}
    if case.get("so"):
        kw["objective"] = qdta.OBJ_SO
    if "ls" in case:
        kw["ls_mode"] = SEARCH[case["ls"]]
    if "rule" in case:
        kw["trunc_rule"] = RULES[case["rule"]]
    if "iters" in case:
        kw["fixed_iters"] = case["iters"]
    if case["op"] in ("interval", "calib"):
        kw["keep_history"] = 1
    return qdta.default_opts(**kw)


def _net(case, side=None):
    return grid(side or case["side"]) if case["net"] == "grid" else road(case["n"], case["oneway"])


def _flows(rng, cap, dt, m):
    """Link flows of a loaded network (2^-20 vehicle): most links below capacity, some far above it."""
    hours = 1.0 if math.isinf(dt) else dt / 3600.0
    veh = cap * hours * rng.lognormal(-0.8, 0.8, m) * (rng.random(m) < 0.8)
    return np.rint(veh * qdta.FX).astype(np.int64)


def _loaded_costs(rng, c0, load):
    r = rng.lognormal(-1.0, 0.5 + 0.25 * load, c0.size) if load else np.zeros(c0.size)
    return (c0 * (1.0 + 0.15 * r ** 4)).astype(np.float32)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def prepare(case, seed):
    rng = np.random.default_rng([seed, 77])
    op, opts = case["op"], _options(case)
    ctx = qdta.Context(0)
    s = {"op": op, "opts": opts, "ctx": ctx}
    if op == "solve":
        nets = [grid(int(k)) for k in case["sides"].split(",")]
        for i, net in enumerate(nets):
            ctx.add_network(net.n, net.row_ptr, net.col, *attributes(net, rng))
            ctx.set_demand(i, *grid_demand(net, zones_of(net, min(case["zones"], net.n // 2)), rng), INF)
        m = sum(net.m for net in nets)
        s["f"] = torch.empty(m, dtype=torch.int64, device=DEV)
        s["cost"] = torch.empty(m, dtype=torch.float32, device=DEV)
        return s
    net = _net(case)
    c0, cap = attributes(net, rng)
    ctx.add_network(net.n, net.row_ptr, net.col, c0, cap)
    zones = zones_of(net, case.get("zones", 8))
    if op in ("costs", "step"):
        # an interval of 15 minutes on roads, static on grids; the demand only sets the interval length
        dt = INF if case["net"] == "grid" else 900.0
        ctx.set_demand(0, zones[:1], zones[1:2], np.ones(1), dt)
        s["f"] = _dev(_flows(rng, cap, dt, net.m))
        ctx.layout()
        if op == "costs":
            s["cost"] = torch.empty(net.m, dtype=torch.float32, device=DEV)
        else:
            s["y"], s["next"] = _dev(_flows(rng, cap, dt, net.m)), torch.empty(net.m, dtype=torch.int64, device=DEV)
            s["alpha"] = torch.empty(1, dtype=torch.float64, device=DEV)
        return s
    if op == "trees":
        dests = zones_of(net, case["dests"])
        s["dest"], s["cost"] = _dev(dests), _dev(_loaded_costs(rng, c0, 0.0 if case["free"] else 1.0))
        s["dist"] = torch.empty((dests.size, net.n), dtype=torch.float32, device=DEV)
        s["succ"] = torch.empty((dests.size, net.n), dtype=torch.int32, device=DEV)
        return s
    if case["net"] == "grid":
        legs = grid_demand(net, zones, rng)
    else:
        legs = road_demand(net, zones, case["legs"], case.get("carried", 0), 1.24 if net.n > 300_000 else 3.2, rng)
    dt = case.get("dt", 900.0)
    if op == "interval":
        s.update(legs=legs, dt=dt, f=torch.empty(net.m, dtype=torch.int64, device=DEV))
        room = (case["iters"] + 2) * legs[0].size  # the day's table of pending legs
        s["pending"] = [np.zeros(room, t) for t in (np.int32, np.int32, np.int64, np.float32)]
        return s
    ctx.set_demand(0, *legs, dt)
    if op == "aon":
        s["cost"] = _dev(_loaded_costs(rng, c0, case["load"]))
        s["y"] = torch.empty(net.m, dtype=torch.int64, device=DEV)
        s["stop"] = torch.empty(ctx.layout().total_legs, dtype=torch.int32, device=DEV)
        return s
    # calib: a solved interval with its paths recorded, observed counts on some links, a perturbed demand
    ctx.solve(opts)
    ctx.adjoint_record(opts)
    d = ctx.legs()[2] / qdta.FX
    s["demand"] = _dev(d * np.exp(0.5 * rng.standard_normal(d.size)))
    s["cap"] = _dev(cap)
    s["links"] = _dev(rng.choice(net.m, max(1, net.m // 50), replace=False))
    s["counts"] = _dev(rng.exponential(100.0, max(1, net.m // 50)))
    return s


def run(state):
    ctx, opts, op = state["ctx"], state["opts"], state["op"]
    if op == "costs":
        ctx.bpr(opts, state["f"], state["cost"])
        return state["cost"]
    if op == "step":
        ctx.line_search(opts, state["f"], state["y"], 3, state["alpha"])
        state["next"].copy_(state["f"])
        ctx.fw_update(state["next"], state["y"], state["alpha"])
        return {"alpha": state["alpha"], "flows": state["next"]}
    if op == "trees":
        ctx.trees(opts, 0, state["cost"], state["dest"], state["dist"], state["succ"])
        return {"dist": state["dist"], "succ": state["succ"]}
    if op == "aon":
        ctx.aon(opts, state["cost"], state["y"], state["stop"])
        return {"y": state["y"], "stop": state["stop"]}
    if op == "solve":
        stats, _ = ctx.solve(opts)
        ctx.get_flows(state["f"])
        ctx.get_costs(opts, state["cost"])
        return {"flows": state["f"], "cost": state["cost"], "gap": [t["gap"] for t in stats],
                "objective": [t["objective"] for t in stats]}
    if op == "interval":
        ctx.set_residual(0, [], [], [])
        ctx.set_demand(0, *state["legs"], state["dt"])
        stats, _ = ctx.solve(opts)
        ctx.get_flows(state["f"])
        ctx.advance_interval(opts)
        *legs, done = ctx.residual(0, with_delay=True)
        for table, col in zip(state["pending"], legs):
            table[:col.size] = col
            table[col.size:] = 0
        return {"flows": state["f"], "gap": stats[0]["gap"], "objective": stats[0]["objective"],
                "pending": state["pending"], "count": legs[0].size, "done": done}
    d, cap = state["demand"].clone().requires_grad_(), state["cap"].clone().requires_grad_()
    flows = qdta.frozen_path_flows(ctx, opts, d, cap)
    loss = ((flows[state["links"]] - state["counts"]) ** 2).sum()
    loss.backward()
    return {"flows": flows.detach(), "demand": d.grad, "cap": cap.grad}


def work(case):
    """Bytes: the network, the costs or flows and the demand in, the results out, once for every pass of the method
    over them.  Operations: for trees an addition and a comparison per link and destination, for a line search the
    30 or so of each evaluation."""
    op = case["op"]
    if op == "solve":
        nets = [grid(int(k)) for k in case["sides"].split(",")]
        z = [min(case["zones"], net.n // 2) for net in nets]
        b = sum(44 * net.m + 16 * q * (q - 1) for net, q in zip(nets, z))
        return {"bytes": (case["iters"] + 1) * b,
                "flops": (case["iters"] + 1) * sum(2 * net.m * q + 30 * 96 * net.m for net, q in zip(nets, z))}
    net = _net(case)
    n, m = net.n, net.m
    if op == "costs":
        return {"bytes": 20 * m, "flops": 8 * m}
    if op == "step":
        return {"bytes": (24 + 24) * m, "flops": 30 * (96 if case["ls"] == "ksection" else 6) * m}
    if op == "trees":
        q = min(case["dests"], n)
        return {"bytes": 12 * m + 4 * n + 8 * q * n, "flops": 2 * q * m}
    q = min(case["zones"], n)
    legs = q * (q - 1) if case["net"] == "grid" else case["legs"] + case.get("carried", 0)
    if op == "aon":
        return {"bytes": 20 * m + 4 * n + 20 * legs, "flops": 2 * q * m}
    if op == "interval":
        k = case["iters"]
        return {"bytes": (k + 1) * (44 * m + 4 * n + 16 * legs) + (k + 1) * 20 * legs,
                "flops": (k + 1) * (2 * q * m + 30 * 96 * m)}
    k = case["iters"]
    return {"bytes": (k + 1) * 40 * m + (k + 1) * 24 * legs, "flops": k * 30 * 96 * m + 2 * (k + 1) * 100 * legs}


def exact(case, seed):
    op = case["op"]
    if op not in ("costs", "step", "trees"):
        return None                               # sums over paths of other iterations' trees
    rng = np.random.default_rng([seed, 77])
    net = _net(case)
    c0, cap = (a.astype(np.float64) for a in attributes(net, rng))
    dt = INF if case["net"] == "grid" else 900.0
    kappa = 1.0 if math.isinf(dt) else 3600.0 / dt
    if op == "costs":
        f = _flows(rng, cap.astype(np.float32), dt, net.m) / qdta.FX
        return c0 * (1.0 + 0.15 * (5.0 if case["so"] else 1.0) * (f * kappa / cap) ** 4)
    if op == "step":
        if case["ls"] != "ksection":
            return None
        f = _flows(rng, cap.astype(np.float32), dt, net.m) / qdta.FX
        t = _flows(rng, cap.astype(np.float32), dt, net.m) / qdta.FX - f
        g = 0.15 * (5.0 if case["so"] else 1.0)

        def slope(a):
            return float((t * c0 * (1.0 + g * (((f + a * t) * kappa) / cap) ** 4)).sum())

        lo, hi = 0.0, 1.0                         # the root of the objective's derivative, or an end
        if slope(0.0) >= 0.0 or slope(1.0) < 0.0:
            return {"alpha": np.array([0.0 if slope(0.0) >= 0.0 else 1.0]), "flows": None}
        for _ in range(45):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if slope(mid) < 0.0 else (lo, mid)
        return {"alpha": np.array([0.5 * (lo + hi)]), "flows": None}
    if net.n > 2000:
        return None
    cost = _loaded_costs(rng, c0.astype(np.float32), 0.0 if case["free"] else 1.0).astype(np.float64)
    dests = zones_of(net, case["dests"])
    dist = np.full((net.n, dests.size), np.inf)
    dist[dests, np.arange(dests.size)] = 0.0
    while True:                                   # Bellman-Ford on all destinations at once
        best = np.minimum(dist, np.minimum.reduceat(dist[net.col] + cost[:, None], net.row_ptr[:-1], axis=0))
        if np.array_equal(best, dist):
            return {"dist": dist.T, "succ": None}
        dist = best

"""The kernels at the sizes where their work splits change: GPU against the oracle through the C ABI.  Integer
sums and flows are exact in any order, so the tolerance is zero throughout."""
from __future__ import annotations

import numpy as np
import pytest

from synth.networks import Network

pytestmark = pytest.mark.gpu

FX = 1 << 20


@pytest.fixture(scope="module")
def q():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2104_12911_amd import qdta
    qdta.lib()
    return qdta


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def i128(lo, hi):
    return (int(hi) << 64) | (int(lo) & ((1 << 64) - 1))


def parallel_links(m, rng, cap):
    """Two nodes and m links from one to the other."""
    return Network(2, np.array([0, m, m], np.int32), np.ones(m, np.int32),
                   rng.uniform(1.0, 100.0, m).astype(np.float32), (cap * rng.uniform(1.0, 4.0, m)).astype(np.float32))


# links: one, either side of a 256-link tile and of a 2,048-link chunk, several chunks; step sizes: one, a few that
# do not divide the workgroup, the most; demand: ordinary, terms beyond 2^66 (and 2^84), an interval length whose
# kappa is beyond 2^60 (true divisions)
@pytest.mark.parametrize("m", [1, 63, 255, 256, 257, 2047, 2048, 2049, 70_001])
@pytest.mark.parametrize("K,beta,objective", [(1, 4, 0), (3, 4, 1), (7, 3, 0), (32, 4, 0), (33, 16, 1), (64, 1, 1)])
def test_line_search_sums_at_split_edges(q, orc, m, K, beta, objective):
    import torch
    rng = np.random.default_rng(m * 100 + K)
    for kind in ("ordinary", "large", "short"):
        if kind == "large" and beta > 4:
            continue
        if kind == "short" and beta != 1:
            continue
        net = parallel_links(m, rng, 900.0 if kind != "large" else 10.0)
        veh = {"ordinary": 300.0, "large": 1e5, "short": 1e-3}[kind]
        dt = {"ordinary": 900.0, "large": 900.0, "short": 1e-16}[kind]
        f = (rng.uniform(0.0, veh, m) * FX).astype(np.int64)
        y = (rng.uniform(0.0, veh, m) * FX).astype(np.int64) * rng.integers(0, 2, m)
        alphas = np.linspace(0.0, 1.0, K) if K > 1 else np.array([0.37])
        Co, Do, _ = orc.ls_eval(f, y, net.fftt, net.cap, 0.15, beta, dt, alphas, objective=objective)
        with q.Context() as ctx:
            ctx.add(net)
            ctx.set_demand(0, [], [], [], dt)
            ctx.layout()
            for call in (ctx.ls_eval, ctx.ls_eval_noalloc):
                sums = torch.zeros(K * 4, dtype=torch.int64, device="cuda")
                call(q.default_opts(beta=beta, objective=objective), dev(f), dev(y), dev(alphas), sums)
                s = sums.cpu().numpy().reshape(K, 2, 2)
                for k in range(K):
                    assert i128(*s[k, 0]) == Co[k], (kind, k)
                    assert i128(*s[k, 1]) == Do[k], (kind, k)


@pytest.mark.parametrize("m", [1, 257, 2049, 70_001])
@pytest.mark.parametrize("K", [3, 32, 64])
@pytest.mark.parametrize("mode", [0, 1])
def test_step_size_at_split_edges(q, orc, m, K, mode):
    """The decision in the last workgroup of a pass, several searches on one context."""
    import torch
    rng = np.random.default_rng(m + K)
    net = parallel_links(m, rng, 900.0)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], 900.0)
        a = torch.zeros(1, dtype=torch.float64, device="cuda")
        for j in (1, 2, 9):
            f = (rng.uniform(0.0, 300.0, m) * FX).astype(np.int64)
            y = (rng.uniform(0.0, 900.0, m) * FX).astype(np.int64) * rng.integers(0, 2, m)
            ao, _, _ = orc.line_search(f, y, net.fftt, net.cap, 0.15, 4, 900.0, j, ls_mode=mode, K=K)
            ctx.line_search(q.default_opts(ls_mode=mode, K=K), dev(f), dev(y), j, a)
            assert float(a.cpu()[0]) == ao, (j, mode)


@pytest.mark.parametrize("legs", [1, 127, 128, 129, 511, 513, 199_999, 200_001, 201_217])
def test_walk_at_split_edges(q, orc, legs):
    """Legs either side of a workgroup's run and of the change from one leg per thread to two."""
    import torch
    import synth
    rng = np.random.default_rng(legs)
    net = synth.grid_network(30, rng)
    nodes = net.n
    pair = rng.choice(nodes * nodes, min(4 * legs, nodes * nodes), replace=False)
    o, d = (pair // nodes).astype(np.int32), (pair % nodes).astype(np.int32)
    keep = np.nonzero(o != d)[0][:legs]
    o, d = o[keep], d[keep]
    assert o.size == legs
    trips = rng.uniform(0.1, 5.0, legs)
    cost = (net.fftt * rng.uniform(1.0, 3.0, net.m)).astype(np.float32)
    lo, ld, lw = orc.demand_legs(o, d, trips)
    for dt, rule in ((float("inf"), 0), (900.0, 1)):
        ref_y, ref_stop = orc.aon(net, cost, lo, ld, lw, dt, rule=rule)[:2]
        with q.Context() as ctx:
            ctx.add(net)
            ctx.set_demand(0, o, d, trips, dt)
            y = torch.empty(net.m, dtype=torch.int64, device="cuda")
            stop = torch.empty(legs, dtype=torch.int32, device="cuda")
            ctx.aon(q.default_opts(trunc_rule=rule), dev(cost), y, stop)
            assert np.array_equal(y.cpu().numpy(), ref_y)
            assert np.array_equal(stop.cpu().numpy(), ref_stop)


def hub_net(rng, leaves, arms):
    """A ring of `arms` nodes around a hub that every leaf has a link to and from: the hub's record row is longer than
    one piece of a step (4), than a packed count (63) or than the LDS buffer (512), by `leaves`."""
    n = 1 + leaves + arms
    tail, head = [], []
    for v in range(1, 1 + leaves):
        tail += [v, 0]
        head += [0, v]
    ring = list(range(1 + leaves, n))
    for i, v in enumerate(ring):
        w = ring[(i + 1) % arms]
        tail += [v, w, v, 1 + i % leaves]
        head += [w, v, 1 + i % leaves, v]
    tail, head = np.array(tail), np.array(head)
    order = np.lexsort((head, tail))
    row = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(tail, minlength=n), out=row[1:])
    m = tail.size
    return Network(n, row, head[order].astype(np.int32), rng.integers(1, 9, m).astype(np.float32),
                   np.full(m, 900.0, np.float32))


@pytest.mark.parametrize("leaves", [3, 4, 5, 8, 9, 62, 63, 64, 257, 1500])
@pytest.mark.parametrize("kernel", [1, 4])
def test_search_rows_and_queues_at_edges(q, orc, leaves, kernel):
    """Rows cut into pieces, rows that do not pack, buffers that overflow into the rings, equal candidates (whole-number
    costs), every workgroup size, tiny and huge bucket widths."""
    import torch
    rng = np.random.default_rng(leaves)
    net = hub_net(rng, leaves, 40)
    dests = np.unique(rng.integers(0, net.n, 6)).astype(np.int32)
    ref = [orc.tree(net, net.fftt, int(t)) for t in dests]
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], float("inf"))
        dist = torch.empty((dests.size, net.n), dtype=torch.float32, device="cuda")
        succ = torch.empty((dests.size, net.n), dtype=torch.int32, device="cuda")
        for shape in (1, 2, 3, 4, 5, 6):
            for scale in (0.01, 1.0, 1e6):
                o = q.default_opts(sssp_kernel=kernel, sssp_shape=shape, delta_scale=scale)
                ctx.trees(o, 0, dev(net.fftt), dev(dests), dist, succ)
                for k in range(dests.size):
                    assert np.array_equal(dist[k].cpu().numpy(), ref[k][0]), (shape, scale, k)
                    assert np.array_equal(succ[k].cpu().numpy(), ref[k][1]), (shape, scale, k)


@pytest.mark.parametrize("legs", [1, 129, 3000])
def test_residual_walk_counts_completed_weight_of_mixed_instances(q, orc, legs):
    """A workgroup of the residual walk whose legs belong to several instances: completed and unfinished weight of
    each instance, against the oracle's residual."""
    import synth
    rng = np.random.default_rng(legs)
    nets, dems = [], []
    for k in (5, 7, 6):
        net = synth.grid_network(k, rng)
        o, d = rng.integers(0, net.n, legs).astype(np.int32), rng.integers(0, net.n, legs).astype(np.int32)
        nets.append(net)
        dems.append((o, d, rng.uniform(0.1, 5.0, legs)))
    with q.Context() as ctx:
        opts = q.default_opts(fixed_iters=3, keep_history=1, ls_mode=q.LS_MSA)
        for i, (net, dm) in enumerate(zip(nets, dems)):
            ctx.add(net)
            ctx.set_demand(i, *dm, 300.0)
        ctx.solve(opts)
        ctx.advance_interval(opts)
        got = [ctx.residual(i) for i in range(3)]
    for (net, dm), (ro, rd, rw, done) in zip(zip(nets, dems), got):
        lo, ld, lw = orc.demand_legs(*dm)
        ref = orc.fw_solve(net, lo, ld, lw, dt_s=300.0, rule=orc.RULE_CEIL, fixed_iters=3, ls_mode=orc.LS_MSA,
                           keep_history=True)
        eo, ed, ew, edone = orc.residual(net, ref.f, ref.hist_alpha, ref.hist_cost, lo, ld, lw, dt_s=300.0)[:4]
        eo, ed, ew = orc.merge_legs(eo, ed, ew)[:3]
        assert np.array_equal(ro, eo) and np.array_equal(rd, ed) and np.array_equal(rw, ew)
        assert done == edone


@pytest.mark.parametrize("m", [1, 255, 257, 2047, 2049, 5000])
@pytest.mark.parametrize("stop_rule,ls_mode", [(0, 0), (1, 0), (1, 1), (0, 2)])
def test_stop_tests_at_split_edges(q, orc, m, stop_rule, ls_mode):
    """Gap, objective change, stall and update decided by the last workgroup of an instance, two instances together:
    flows, step sizes and why each stopped, against the oracle."""
    import torch
    rng = np.random.default_rng(m)
    nets = [parallel_links(m, rng, 300.0), parallel_links(max(1, m // 3), rng, 900.0)]
    trips = [40.0 * m, 2.0]
    opts = q.default_opts(stop_rule=stop_rule, ls_mode=ls_mode, tol=1e-3, max_iter=12)
    with q.Context() as ctx:
        for i, net in enumerate(nets):
            ctx.add(net)
            ctx.set_demand(i, [0], [1], [trips[i]], float("inf"))
        for again in range(2):
            st, _ = ctx.solve(opts)
            f = torch.empty(sum(net.m for net in nets), dtype=torch.int64, device="cuda")
            ctx.get_flows(f)
            f = f.cpu().numpy()
            at = 0
            for i, net in enumerate(nets):
                o, d, w = orc.demand_legs(np.array([0], np.int32), np.array([1], np.int32), np.array([trips[i]]))
                ref = orc.fw_solve(net, o, d, w, stop_rule=stop_rule, ls_mode=ls_mode, tol=1e-3, max_iter=12,
                                   keep_history=False)
                assert np.array_equal(f[at:at + net.m], ref.f)
                assert (st[i]["iters"], st[i]["stopped_by"]) == (ref.iters, ref.stopped_by)
                assert st[i]["gap"] == ref.gap and st[i]["last_alpha"] == ref.last_alpha
                at += net.m


@pytest.mark.parametrize("hubs", [3, 12, 40])
@pytest.mark.parametrize("kernel", [1, 4])
def test_search_queues_fuller_than_the_network(q, orc, hubs, kernel):
    """Every leaf is lowered by each hub in turn while its earlier entries wait, all in one bucket: the near queue
    takes several times the node count, and its overflow goes to the far queue."""
    import torch
    leaves = 1000
    n = 1 + hubs + leaves
    tail, head, cost = [], [], []
    for i in range(hubs):
        tail.append(1 + i), head.append(0), cost.append(1.0 + i)
        for v in range(1 + hubs, n):
            tail.append(v), head.append(1 + i), cost.append(4.0 * (hubs - i))
    for v in range(1 + hubs, n):
        tail.append(0), head.append(v), cost.append(1.0)
    tail, head, cost = np.array(tail), np.array(head), np.array(cost, np.float32)
    order = np.lexsort((head, tail))
    row = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(tail, minlength=n), out=row[1:])
    net = Network(n, row, head[order].astype(np.int32), cost[order], np.full(tail.size, 900.0, np.float32))
    ref = orc.tree(net, net.fftt, 0)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], float("inf"))
        dist = torch.empty((1, n), dtype=torch.float32, device="cuda")
        succ = torch.empty((1, n), dtype=torch.int32, device="cuda")
        for shape in (0, 1, 2, 3, 4, 5, 6):
            for scale in (0.05, 1e6):
                o = q.default_opts(sssp_kernel=kernel, sssp_shape=shape, delta_scale=scale)
                ctx.trees(o, 0, dev(net.fftt), dev(np.zeros(1, np.int32)), dist, succ)
                assert np.array_equal(dist[0].cpu().numpy(), ref[0]), (shape, scale)
                assert np.array_equal(succ[0].cpu().numpy(), ref[1]), (shape, scale)


@pytest.mark.parametrize("n", [1, 2, 33, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("row", [4, 8, 9])
def test_trees_of_small_networks(q, orc, n, row):
    """Around the sizes where the trees of a small network change form (256, 512, 1,024, 2,048 and 4,096 nodes, rows of
    4 and of 8 links), with nodes that reach no destination and whole-number costs that tie."""
    import torch
    rng = np.random.default_rng(n * 16 + row)
    deg = rng.integers(0, row + 1, n)
    deg[rng.integers(0, n)] = row
    ptr = np.zeros(n + 1, np.int32)
    np.cumsum(deg, out=ptr[1:])
    m = int(ptr[-1])
    near = (np.repeat(np.arange(n), deg) + rng.integers(-40, 41, m)) % n
    net = Network(n, ptr, near.astype(np.int32), rng.integers(1, 6, m).astype(np.float32), np.full(m, 900.0, np.float32))
    dests = rng.integers(0, n, 300 if n in (2048, 2049) else 5).astype(np.int32)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], float("inf"))
        dist = torch.empty((dests.size, n), dtype=torch.float32, device="cuda")
        succ = torch.empty((dests.size, n), dtype=torch.int32, device="cuda")
        ctx.trees(q.default_opts(), 0, dev(net.fftt), dev(dests), dist, succ)
        for k in list(range(5)) + [dests.size - 1]:
            ref = orc.tree(net, net.fftt, int(dests[k]))
            assert np.array_equal(dist[k].cpu().numpy(), ref[0]), k
            assert np.array_equal(succ[k].cpu().numpy(), ref[1]), k


@pytest.mark.parametrize("leaves", [3, 4, 5, 62, 63, 64, 257])
def test_walk_through_long_rows(q, orc, leaves):
    """Legs through a hub whose row is one to many turns of four lanes, or does not pack, with ties on the way."""
    import torch
    rng = np.random.default_rng(leaves)
    net = hub_net(rng, leaves, 40)
    pair = rng.choice(net.n * net.n, min(700, net.n * net.n), replace=False)
    o, d = (pair // net.n).astype(np.int32), (pair % net.n).astype(np.int32)
    o, d = o[o != d], d[o != d]
    trips = rng.uniform(0.1, 5.0, o.size)
    legs = orc.demand_legs(o, d, trips)
    for dt, rule in ((float("inf"), 0), (10.0, 1)):
        ref_y, ref_stop = orc.aon(net, net.fftt, *legs, dt, rule=rule)[:2]
        with q.Context() as ctx:
            ctx.add(net)
            ctx.set_demand(0, o, d, trips, dt)
            y = torch.empty(net.m, dtype=torch.int64, device="cuda")
            stop = torch.empty(o.size, dtype=torch.int32, device="cuda")
            ctx.aon(q.default_opts(trunc_rule=rule), dev(net.fftt), y, stop)
            assert np.array_equal(y.cpu().numpy(), ref_y)
            assert np.array_equal(stop.cpu().numpy(), ref_stop)


@pytest.mark.parametrize("legs", [1, 90, 1500])
def test_path_loading_runs(q, orc, legs):
    """Recorded paths of less than one run of the loading (4,096 links), of about one and of many, with legs of no
    demand: the replayed flows are the oracle's, bit for bit."""
    import torch
    import synth
    from oracle import adjoint as adj
    rng = np.random.default_rng(legs)
    net = synth.grid_network(40, rng)
    pair = rng.choice(net.n * net.n, 2 * legs + 8, replace=False)
    o, d = (pair // net.n).astype(np.int32), (pair % net.n).astype(np.int32)
    keep = np.nonzero(o != d)[0][:legs]
    o, d, trips = o[keep], d[keep], rng.uniform(0.1, 5.0, legs)
    lo, ld, lw = orc.demand_legs(o, d, trips)
    res = orc.fw_solve(net, lo, ld, lw, dt_s=float("inf"), fixed_iters=2, keep_history=True)
    paths = adj.frozen_paths(net, lo, ld, lw, res.hist_cost, float("inf"))
    demand = rng.uniform(0.0, 9.0, legs) * (rng.random(legs) < 0.8)
    ref = adj.forward_contract(paths, net.m, demand, net.fftt, net.cap, 0.15, 4, float("inf"))[0]
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, o, d, trips, float("inf"))
        opts = q.default_opts(fixed_iters=2, keep_history=1)
        ctx.solve(opts)
        ctx.adjoint_record(opts)
        f = torch.empty(net.m, dtype=torch.float64, device="cuda")
        ctx.model_forward(opts, dev(demand), None, f)
        assert np.array_equal(f.cpu().numpy() * FX, ref.astype(np.float64))


@pytest.mark.parametrize("kernel", [1, 4])
def test_search_from_a_last_node_without_in_links(q, orc, kernel):
    """No chains, and the highest-numbered node has out-links only, so its record row is empty and no record lies
    behind it (32 records: the buffer holds nothing else).  Every tree reaches that node."""
    import torch
    n, pairs = 6, [(a, b) for a in range(5) for b in range(5) if a != b]
    pairs += [(5, b) for b in (0, 0, 0, 1, 1, 1, 2, 2, 2, 3, 3, 4)]
    tail, head = np.array(pairs).T
    ptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(tail, minlength=n), out=ptr[1:])
    assert tail.size == 32 and not (head == 5).any()
    cost = np.random.default_rng(3).integers(1, 6, 32).astype(np.float32)
    net = Network(n, ptr, head.astype(np.int32), cost, np.full(32, 900.0, np.float32))
    dests = np.arange(n, dtype=np.int32)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], float("inf"))
        dist = torch.empty((n, n), dtype=torch.float32, device="cuda")
        succ = torch.empty((n, n), dtype=torch.int32, device="cuda")
        for shape in (0, 1, 2, 3, 4, 5, 6):
            ctx.trees(q.default_opts(sssp_kernel=kernel, sssp_shape=shape), 0, dev(cost), dev(dests), dist, succ)
            for t in range(n):
                ref = orc.tree(net, cost, t)
                assert np.array_equal(dist[t].cpu().numpy(), ref[0]), (shape, t)
                assert np.array_equal(succ[t].cpu().numpy(), ref[1]), (shape, t)


@pytest.mark.parametrize("n", [1, 2, 7])
@pytest.mark.parametrize("ls_mode", [1, 2])
def test_line_search_starts_from_the_running_iteration(q, n, ls_mode):
    """The first step size of a search is a function of the iteration index alone, 2 / (2 + j) or 1 / (j + 1), and a
    quasi-Newton search that any slope satisfies returns it: iteration n of a solve, two instances, three times."""
    rng = np.random.default_rng(n)
    want = 2.0 / (2.0 + n) if ls_mode == 1 else 1.0 / (n + 1.0)
    opts = q.default_opts(ls_mode=ls_mode, T1=1e300, fixed_iters=n)
    with q.Context() as ctx:
        for i, m in enumerate((300, 5000)):
            ctx.add(parallel_links(m, rng, 300.0))
            ctx.set_demand(i, [0], [1], [40.0 * m], float("inf"))
        for _ in range(3):
            st, _ = ctx.solve(opts)
            assert [s["last_alpha"] for s in st] == [want, want]
            assert [s["iters"] for s in st] == [n, n]


@pytest.mark.parametrize("tree_waves", [1, 4])
@pytest.mark.parametrize("kernel", [0, 1])
def test_tie_fallback_of_many_trees(q, orc, kernel, tree_waves):
    """Most trees of a network whose dear links absorb the cheap ones are finished by the tie fallback, on as many
    workgroups as the queues of the tree form hold: flows and stop nodes against the oracle."""
    import torch
    import synth
    rng = np.random.default_rng(11)
    net = synth.grid_network(9, rng)
    cost = np.where(rng.random(net.m) < 0.5, rng.uniform(1e8, 4e8, net.m), rng.uniform(0.5, 8.0, net.m))
    cost = cost.astype(np.float32)
    pair = rng.choice(net.n * net.n, 2000, replace=False)
    o, d = (pair // net.n).astype(np.int32), (pair % net.n).astype(np.int32)
    o, d = o[o != d], d[o != d]
    trips = rng.uniform(0.1, 5.0, o.size)
    ref_y, ref_stop, code = orc.aon(net, cost, *orc.demand_legs(o, d, trips), float("inf"), rule=1)[:3]
    assert code == orc.WARN_ABSORB
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, o, d, trips, float("inf"))
        y = torch.empty(net.m, dtype=torch.int64, device="cuda")
        stop = torch.empty(o.size, dtype=torch.int32, device="cuda")
        rc = ctx.aon(q.default_opts(sssp_kernel=kernel, tree_waves=tree_waves), dev(cost), y, stop)
        assert rc == q.WABSORB
        assert np.array_equal(y.cpu().numpy(), ref_y)
        assert np.array_equal(stop.cpu().numpy(), ref_stop)


@pytest.mark.parametrize("kernel", [0, 1, 4])
def test_trees_with_costs_that_are_none(q, kernel):
    """Costs no assignment has: a negative one off every cycle counts like any other while the sum is not negative, a
    sum below zero and NaN are never taken; and on a negative cycle the trees still end."""
    import torch
    # 0 is the destination; 1 -> 0, 2 -> 1, 3 -> 1, 4 -> 0 and 4 -> 2, 5 -> 4, and 6 <-> 7 with 6 -> 0
    tail, head = np.array([1, 2, 3, 4, 4, 5, 6, 6, 7, 7]), np.array([0, 1, 1, 0, 2, 4, 0, 7, 6, 0])
    cost = np.array([10.0, -3.0, -20.0, 9.0, 1.0, np.nan, 10.0, 1.0, 2.0, 50.0], np.float32)
    row = np.zeros(9, np.int32)
    np.cumsum(np.bincount(tail, minlength=8), out=row[1:])
    net = Network(8, row, head.astype(np.int32), np.ones(10, np.float32), np.full(10, 900.0, np.float32))
    inf = np.inf
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], inf)
        dist = torch.empty((1, 8), dtype=torch.float32, device="cuda")
        succ = torch.empty((1, 8), dtype=torch.int32, device="cuda")
        o = q.default_opts(sssp_kernel=kernel)
        ctx.trees(o, 0, dev(cost), dev(np.zeros(1, np.int32)), dist, succ)
        assert dist[0].cpu().tolist() == [0.0, 10.0, 7.0, inf, 8.0, inf, 10.0, 12.0]
        cost[7] = -2.5                                     # 6 -> 7 -> 6 costs -0.5
        ctx.trees(o, 0, dev(cost), dev(np.zeros(1, np.int32)), dist, succ)
        d = dist[0].cpu().tolist()
        assert d[:6] == [0.0, 10.0, 7.0, inf, 8.0, inf] and 0.0 <= d[6] <= 10.0 and 0.0 <= d[7] <= 50.0


def test_line_search_sums_of_millions_of_large_terms(q, orc):
    """2^22 links and more, every term beyond 2^66 with its low 42 bits well filled, on the one copy of the sums that
    the call without allocations has: m times the oracle's term."""
    import torch
    m = (1 << 22) + 4097
    one = np.ones(1, np.float32)
    low = (1 << 42) - 1
    for x in range(1000 * FX, 1001 * FX):
        f, y = np.array([x], np.int64), np.array([3 * x], np.int64)
        C, D, _ = orc.ls_eval(f, y, one, one, 0.15, 4, 900.0, np.array([0.0]))
        if min(C[0], D[0]) > 1 << 66 and min(C[0] & low, D[0] & low) * m > 1.05 * (1 << 63):
            break
    else:
        raise AssertionError("no such flow")
    net = Network(2, np.array([0, m, m], np.int32), np.ones(m, np.int32), np.ones(m, np.float32),
                  np.ones(m, np.float32))
    F, Y = (torch.full((m,), v, dtype=torch.int64, device="cuda") for v in (x, 3 * x))
    alphas = dev(np.zeros(1))
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [], [], [], 900.0)
        ctx.layout()
        for call in (ctx.ls_eval, ctx.ls_eval_noalloc):
            sums = torch.zeros(4, dtype=torch.int64, device="cuda")
            call(q.default_opts(), F, Y, alphas, sums)
            s = sums.cpu().numpy().reshape(2, 2)
            assert i128(*s[0]) == m * C[0], call
            assert i128(*s[1]) == m * D[0], call


@pytest.mark.parametrize("m", [2, 257, 5000])
@pytest.mark.parametrize("stop_rule,objective", [(0, 0), (1, 0), (1, 1)])
def test_gap_and_objective_of_large_terms(q, orc, m, stop_rule, objective):
    """All demand on one link far beyond its capacity at first: its terms of the gap and the objective are beyond 2^66
    while the others are ordinary.  Gap, objective, flows and why the solve stopped, against the oracle."""
    import torch
    rng = np.random.default_rng(m)
    net = parallel_links(m, rng, 10.0)
    o, d, w = orc.demand_legs(np.array([0], np.int32), np.array([1], np.int32), np.array([1e6]))
    kw = dict(stop_rule=stop_rule, tol=1e-9, max_iter=5, objective=objective)
    ref = orc.fw_solve(net, o, d, w, keep_history=False, **kw)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, [0], [1], [1e6], float("inf"))
        st, _ = ctx.solve(q.default_opts(**kw))
        f = torch.empty(m, dtype=torch.int64, device="cuda")
        ctx.get_flows(f)
    assert np.array_equal(f.cpu().numpy(), ref.f)
    assert (st[0]["iters"], st[0]["stopped_by"]) == (ref.iters, ref.stopped_by)
    assert st[0]["gap"] == ref.gap and st[0]["objective"] == ref.objective
    assert 1e6 * 0.15 * (1e6 / net.cap[np.argmin(net.fftt)]) ** 4 * net.fftt.min() * 2.0 ** 16 > 2.0 ** 66

"""Calls made between others on one context: what one call reports or keeps is not changed by the next."""
from __future__ import annotations

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


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


def demand(rng, n, legs):
    return rng.integers(0, n, legs), rng.integers(0, n, legs), rng.uniform(1, 10, legs)


def test_trees_between_steps_leave_the_solves_absorption(q):
    """A solve that met FP32 absorption still says so after trees without any, and one without does not report that of
    the trees grown in between."""
    import torch
    opts = q.default_opts(fixed_iters=1)
    met = clean = 0
    for seed in range(30):
        rng = np.random.default_rng(seed)
        net = synth.tiny_network(8, 10, rng, costs="huge")
        plain = dev(rng.uniform(1.0, 2.0, net.m).astype(np.float32))
        dem = demand(rng, 8, 30)
        dests = dev(np.arange(8, dtype=np.int32))
        dist = torch.empty((8, 8), dtype=torch.float32, device="cuda")
        succ = torch.empty((8, 8), dtype=torch.int32, device="cuda")

        def steps(fftt, between):
            mid = []
            with q.Context() as ctx:
                ctx.add(synth.networks.Network(net.n, net.row_ptr, net.col, fftt, net.cap))
                ctx.set_demand(0, *dem, float("inf"))
                ctx.fw_begin(opts)
                live, out = True, []
                while live:
                    mid.append(ctx.trees(opts, 0, between, dests, dist, succ))
                    st, live = ctx.fw_step(opts)
                    out.append(st[0]["absorb"])
                mid.append(ctx.trees(opts, 0, between, dests, dist, succ))
                out.append(ctx.fw_step(opts)[0][0]["absorb"])   # nothing runs any more: what the solve has recorded
            return out, mid

        huge = net.fftt.astype(np.float32)
        out, mid = steps(huge, plain)
        if out[0]:
            assert mid == [q.OK] * len(mid) and all(out), seed
            met += 1
        out, mid = steps(rng.uniform(1.0, 2.0, net.m).astype(np.float32), dev(huge))
        if mid[0] == q.WABSORB:
            assert mid == [q.WABSORB] * len(mid) and not any(out), seed
            clean += 1
    assert met and clean


@pytest.mark.parametrize("workspace", [False, True])
@pytest.mark.parametrize("tree_waves", [0, 1])
def test_autotune_before_the_first_solve_leaves_it_its_queues(q, workspace, tree_waves):
    """The autotuner times both tree forms on queues as large as a solve of either form takes: none of them allocates
    any more afterwards, and inside a workspace of the queried size the solve still fits."""
    import torch
    rng = np.random.default_rng(5)
    net = synth.grid_network(71, rng)
    dem = demand(rng, net.n, 2000)
    opts = q.default_opts(fixed_iters=2, tree_waves=tree_waves)
    ref = torch.empty(net.m, dtype=torch.int64, device="cuda")
    got = torch.empty_like(ref)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, *dem, 900.0)
        ctx.solve(opts)
        ctx.get_flows(ref)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, *dem, 900.0)
        if workspace:
            ws = torch.empty(ctx.workspace_query(opts), dtype=torch.uint8, device="cuda")
            ctx.bind_workspace(ws)
        ctx.autotune(q.default_opts(fixed_iters=2, tree_waves=tree_waves), 2.0)
        before = ctx.alloc_count()
        for tw in (4, 1):
            ctx.solve(q.default_opts(fixed_iters=2, tree_waves=tw))
            ctx.get_flows(got)
            assert torch.equal(got, ref)
        assert ctx.alloc_count() == before


def test_autotune_on_a_small_network_keeps_the_path_record(q):
    """Trees of a small network need no contraction, so the autotuner builds none and a recorded interval stays
    usable; its choice is a configuration a solve takes."""
    import torch
    rng = np.random.default_rng(6)
    net = synth.grid_network(12, rng)
    o, d, trips = demand(rng, net.n, 300)
    opts = q.default_opts(fixed_iters=2, keep_history=1)
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, o, d, trips, 900.0)
        ctx.solve(opts)
        ctx.adjoint_record(opts)
        legs = ctx.legs()[2].astype(np.float64) / (1 << 20)
        f0, f1 = (torch.empty(net.m, dtype=torch.float64, device="cuda") for _ in range(2))
        ctx.model_forward(opts, dev(legs), None, f0)
        before = ctx.alloc_count()
        for tw in (0, 1, 4):
            tuned, ms = ctx.autotune(q.default_opts(fixed_iters=2, tree_waves=tw), 5.0)
            assert tuned.tree_waves in (1, 4) and 1 <= tuned.sssp_shape <= 6 and ms > 0.0
        assert ctx.alloc_count() == before
        ctx.model_forward(opts, dev(legs), None, f1)
        assert torch.equal(f0, f1)


@pytest.mark.parametrize("k", [12, 70])
def test_other_calls_keep_the_path_record(q, k):
    """A recorded interval is usable until the next solve, demand or network, whatever other calls allocate: explicit
    search kernels, other tree counts, line searches."""
    import torch
    rng = np.random.default_rng(k)
    net = synth.grid_network(k, rng)
    o, d, trips = demand(rng, net.n, 300)
    opts = q.default_opts(fixed_iters=2, keep_history=1)
    nq = 320
    dist = torch.empty((nq, net.n), dtype=torch.float32, device="cuda")
    succ = torch.empty((nq, net.n), dtype=torch.int32, device="cuda")
    with q.Context() as ctx:
        ctx.add(net)
        ctx.set_demand(0, o, d, trips, 900.0)
        ctx.solve(opts)
        ctx.adjoint_record(opts)
        legs = ctx.legs()[2].astype(np.float64) / (1 << 20)
        f0, f1 = (torch.empty(net.m, dtype=torch.float64, device="cuda") for _ in range(2))
        fbar = dev(rng.uniform(-1.0, 1.0, net.m))
        grads = []
        ctx.model_forward(opts, dev(legs), None, f0)
        y = torch.empty(net.m, dtype=torch.int64, device="cuda")
        cost = dev(net.fftt.astype(np.float32))
        calls = [lambda: None,
                 lambda: ctx.aon(q.default_opts(sssp_kernel=4), cost, y),
                 lambda: ctx.aon(q.default_opts(tree_waves=1), cost, y),
                 lambda: ctx.trees(q.default_opts(), 0, cost, dev(rng.integers(0, net.n, nq).astype(np.int32)), dist,
                                   succ),
                 lambda: ctx.autotune(q.default_opts(), 1.0)]
        for call in calls:
            call()
            fid = ctx.model_forward(opts, dev(legs), None, f1)
            assert torch.equal(f0, f1)
            call()
            dbar = torch.empty(legs.size, dtype=torch.float64, device="cuda")
            cbar = torch.empty(net.m, dtype=torch.float64, device="cuda")
            ctx.model_backward(fid, fbar, dbar, cbar)
            torch.cuda.synchronize()
            grads.append((dbar, cbar))
        for g in grads[1:]:
            assert torch.equal(g[0], grads[0][0]) and torch.equal(g[1], grads[0][1])
        ctx.set_demand(0, o, d, trips, 900.0)
        with pytest.raises(q.QdtaError):
            ctx.model_forward(opts, dev(legs), None, f1)

"""Dataflow sweeps (one launch per SP or reverse sweep, each column by one
team of workgroups): bit for bit the persistent schedule, which keeps a
barrier per level and a kernel of its own, and the FP64 oracle; at level
widths around a wave, below and beyond what a team's waves hold at once, and
column counts around one per XCD."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import SP_ABS, assert_grad_close, assert_power_close, oracle_column, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return api.Context(0)


def _run(d, nl, sched, B, mode, ste=False, fixed=None, S=0):
    ev = api.Eval(d, B, S, mode=mode, n_sim=64 * 20, seed=5,
                  beta_grad=L.DP_BETA_STE if ste else L.DP_BETA_LOCAL)
    ev.set_pi_prob(synth.pi_probs(nl.n_pi, 6, batch=B))
    ev.set_caps(synth.net_caps(nl.n_nets, 7))
    if S:
        ev.set_cell_sizes(synth.cell_sizes(nl.n_gates, 8, n_size=S))
    if fixed is not None:
        ev.set_pi_fixed(fixed)
    ev.set_schedule(sched)
    out = None
    for _ in range(3):  # the second and third sweep find the first one's values
        r = ev.forward(("sp", "power"))
        r.update(ev.backward(want=("dpi", "dcap")))
        r["lam"], r["score"] = ev.power_gradients()
        if out is not None:
            for k in r:
                np.testing.assert_array_equal(r[k], out[k], err_msg=f"{k}, again")
        out = r
    return out


# widths: 1, a wave less one, a wave, a wave and one, several waves, and one
# level wider than a team's waves hold at once (2 x 32 workgroups x 8 waves)
@pytest.mark.parametrize("gates,pis,depth,B", [
    (5, 3, 5, 1), (63, 4, 1, 1), (64 * 4, 70, 4, 2), (65 * 3, 9, 3, 9), (3000, 130, 12, 8),
    (3000, 130, 12, 17), (3000, 130, 12, 64), (40_000, 90, 1, 1), (70_000, 40_000, 2, 3)])
@pytest.mark.parametrize("mode,ste", [(L.DP_MODELED, False), (L.DP_HYBRID, True)])
def test_flow_is_bitwise_the_barrier_sweep(ctx, gates, pis, depth, B, mode, ste):
    say(f"dataflow sweep: {gates} gates, {pis} PIs, depth {depth}, B={B}, mode {mode}, ste {ste}")
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth), 11)
    d = api.Design(ctx, nl)
    fixed = (np.arange(pis) % 5 == 0).astype(np.uint8)
    ref = _run(d, nl, L.DP_SCHED_PERSISTENT, B, mode, ste, fixed)
    for sched in (L.DP_SCHED_AUTO, L.DP_SCHED_GRAPH):
        r = _run(d, nl, sched, B, mode, ste, fixed)
        for k in ref:
            np.testing.assert_array_equal(r[k], ref[k], err_msg=f"{k}, schedule {sched}")
    o = oracle.Netlist.of(nl)
    p, cap = synth.pi_probs(pis, 6, batch=B), synth.net_caps(nl.n_nets, 7)
    for b in {0, B - 1}:
        f, adj = oracle_column(o, p[b], cap, mode="hybrid" if mode == L.DP_HYBRID else "modeled",
                               n_words=20, seed=5, ste=ste)
        assert np.abs(r["sp"][b] - f["sp"]).max() <= SP_ABS
        assert_power_close(r["power"][b], f["power"], "power")
        assert_grad_close(r["dpi"][b], np.where(fixed, 0.0, adj["dpi"]), "dP/dp")


@pytest.mark.parametrize("readers", [32, 33, 64, 65, 256, 257, 600, 1300])
def test_flow_long_fanout_ranges(ctx, readers):
    """A net and a PI of many readers each (the whole-wave pull), beside nets
    of one to a few readers."""
    say(f"dataflow sweep: {readers} readers")
    gates = [(synth.AND2, [0, 1])]
    gates += [(synth.XOR2 if i % 2 else synth.OR2, [3, 0 if i % 3 else 2]) for i in range(readers)]
    gates += [(synth.MUX2, [4 + i, 3, 4 + (i * 7) % readers]) for i in range(readers)]
    nl = synth.from_gates(3, gates)
    d = api.Design(ctx, nl)
    ref = _run(d, nl, L.DP_SCHED_PERSISTENT, 2, L.DP_MODELED)
    r = _run(d, nl, L.DP_SCHED_AUTO, 2, L.DP_MODELED)
    for k in ref:
        np.testing.assert_array_equal(r[k], ref[k], err_msg=k)


def test_flow_sizes_and_weights(ctx):
    say("dataflow sweep: sizes and upstream weights")
    nl = synth.random_dag(synth.DagSpec(2500, 100, 14), 12)
    d = api.Design(ctx, nl)
    B, S = 4, 3
    w = np.random.default_rng(1).uniform(-2, 2, (B, S)).astype(np.float32)
    res = []
    for sched in (L.DP_SCHED_PERSISTENT, L.DP_SCHED_AUTO):
        ev = api.Eval(d, B, S)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 6, batch=B))
        ev.set_caps(synth.net_caps(nl.n_nets, 7))
        ev.set_cell_sizes(synth.cell_sizes(nl.n_gates, 8, n_size=S))
        ev.set_schedule(sched)
        r = ev.forward(("power",))
        r.update(ev.backward(w, want=("dpi", "dcap", "dsize")))
        r["cols"] = ev.backward_columns()
        res.append(r)
    for k in res[0]:
        np.testing.assert_array_equal(res[1][k], res[0][k], err_msg=k)


def test_flow_on_several_streams(ctx):
    """Sweeps of several evals in flight on streams of their own keep their
    results."""
    import torch
    say("dataflow sweeps on several streams")
    nl = synth.random_dag(synth.DagSpec(30_000, 600, 25), 13)
    cap = torch.from_numpy(synth.net_caps(nl.n_nets, 7)).cuda()
    runs = []
    for i in range(4):
        s = torch.cuda.Stream()
        c = api.Context(0, s.cuda_stream)
        B = 1 + 3 * i
        ev = api.Eval(api.Design(c, nl), B)
        ev.set_pi_prob(torch.from_numpy(synth.pi_probs(nl.n_pi, 20 + i, batch=B)).cuda())
        ev.set_caps(cap)
        runs.append((s, c, ev))

    def sweep(s, ev):
        with torch.cuda.stream(s):
            r = ev.forward(("power",), device=True)
            r.update(ev.backward(want=("dpi",), device=True))
            return r
    ref = []
    for s, c, ev in runs:
        ref.append(sweep(s, ev))
        torch.cuda.synchronize()
    for _ in range(10):
        got = [sweep(s, ev) for s, c, ev in runs]
        torch.cuda.synchronize()
        for g, r in zip(got, ref):
            for k in r:
                assert torch.equal(g[k], r[k]), k


def test_flow_library_cells(ctx):
    """Fixed and library cells in one sweep, launched and replayed from a graph,
    against the oracle (test_gpu_reuse.py has the bits against level launches)."""
    say("dataflow sweep: library cells")
    ops = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(synth.LIBRARY)))
    nl = synth.random_dag(synth.DagSpec(5000, 100, 15, ops=ops, cells=synth.LIBRARY), 14)
    d = api.Design(ctx, nl)
    r = _run(d, nl, L.DP_SCHED_AUTO, 3, L.DP_MODELED)
    g = _run(d, nl, L.DP_SCHED_GRAPH, 3, L.DP_MODELED)
    for k in r:
        np.testing.assert_array_equal(r[k], g[k], err_msg=k)
    o = oracle.Netlist.of(nl)
    p, cap = synth.pi_probs(nl.n_pi, 6, batch=3), synth.net_caps(nl.n_nets, 7)
    for b in range(3):
        f, adj = oracle_column(o, p[b], cap)
        assert np.abs(r["sp"][b] - f["sp"]).max() <= SP_ABS
        assert_grad_close(r["dpi"][b], adj["dpi"], "dP/dp")


@pytest.mark.parametrize("budget", [100_000, 200_000, 1 << 26])
def test_server_with_and_without_room_for_flow_buffers(ctx, budget):
    """Lanes whose dataflow buffers fit the budget, and lanes that run merged
    level launches for want of them, give the same bits."""
    say(f"server budget {budget}")
    nls = [synth.random_dag(synth.DagSpec(3000, 64, 12), 41),
           synth.random_dag(synth.DagSpec(1500, 40, 9), 42)]
    caps = [synth.net_caps(nl.n_nets, 43) for nl in nls]
    srv = api.Server(ctx, budget, max_batch=8, max_inflight=4)
    ids = [srv.add_design(api.Design(ctx, nl), c, mode=L.DP_MODELED) for nl, c in zip(nls, caps)]
    tickets = []
    for k in range(24):
        i = k % 2
        p = synth.pi_probs(nls[i].n_pi, 50 + k)[0]
        size = synth.cell_sizes(nls[i].n_gates, 80 + k)[0]
        tickets.append((i, p, size, srv.submit(ids[i], p, size, backward=k % 3 == 0)))
    for i, p, size, t in tickets:
        power, dpi, _ = srv.wait(t)
        ev = api.Eval(api.Design(ctx, nls[i]), 1, 1)
        ev.set_pi_prob(p[None])
        ev.set_caps(caps[i])
        ev.set_cell_sizes(size[None])
        ev.set_schedule(L.DP_SCHED_PERSISTENT)
        ref = ev.forward(("power",))["power"][0, 0]
        assert abs(power - ref) <= 1e-6 * abs(ref)  # paired sizes sum in another order
        if dpi is not None:
            np.testing.assert_array_equal(dpi, ev.backward(want=("dpi",))["dpi"][0])
    srv.close()


def test_group_beyond_one_sweep(ctx):
    """A group of more (net, column) jobs than one dataflow sweep takes runs
    merged level launches; both match each eval alone."""
    say("groups of 40 and of 80 columns")
    nls = [synth.random_dag(synth.DagSpec(900 * (k + 1), 30 + k, 7 + 2 * k), 60 + k) for k in range(4)]
    for cols in (10, 20):
        evs = []
        for k, nl in enumerate(nls):
            ev = api.Eval(api.Design(ctx, nl), cols)
            ev.set_pi_prob(synth.pi_probs(nl.n_pi, 70 + k, batch=cols))
            ev.set_caps(synth.net_caps(nl.n_nets, 71))
            evs.append(ev)
        for graph in (True, False):
            g = api.Group(ctx, evs)
            g.configure(use_graph=graph)
            for backward in (False, True, True):
                res = g.run(("sp", "power"), backward=backward)
            for ev, r in zip(evs, res):
                ev.set_schedule(L.DP_SCHED_PERSISTENT)
                ref = ev.forward(("sp", "power"))
                ref.update(ev.backward(want=("dpi",)))
                ev.set_schedule(L.DP_SCHED_AUTO)
                for k in r:
                    np.testing.assert_array_equal(r[k], ref[k], err_msg=k)
            g.close()


@pytest.mark.parametrize("graph", [True, False])
def test_group_of_evals_with_the_persistent_schedule(ctx, graph):
    """A group does not use its evals' own schedules: with the persistent one set
    its results are those of the evals alone."""
    say(f"group of evals with the persistent schedule, graph {graph}")
    evs, want = [], []
    for k, mode in enumerate((L.DP_HYBRID, L.DP_MODELED, L.DP_HYBRID)):
        nl = synth.random_dag(synth.DagSpec(900 * (k + 1), 30 + k, 7 + 2 * k), 60 + k)
        ev = api.Eval(api.Design(ctx, nl), 2, mode=mode, n_sim=64 * 20, seed=3)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 70 + k, batch=2))
        ev.set_caps(synth.net_caps(nl.n_nets, 71))
        r = ev.forward(("sp", "power"))
        r.update(ev.backward(want=("dpi",)))
        want.append(r)
        fresh = api.Eval(api.Design(ctx, nl), 2, mode=mode, n_sim=64 * 20, seed=3)
        fresh.set_pi_prob(synth.pi_probs(nl.n_pi, 70 + k, batch=2))
        fresh.set_caps(synth.net_caps(nl.n_nets, 71))
        fresh.set_schedule(L.DP_SCHED_PERSISTENT)
        evs.append(fresh)
    g = api.Group(ctx, evs)
    g.configure(use_graph=graph)
    for r, ref in zip(g.run(("sp", "power"), backward=True), want):
        for k in ref:
            np.testing.assert_array_equal(r[k], ref[k], err_msg=k)
    g.close()


def _with_chain(nl, levels):
    """The netlist with a chain of inverters from its last gate: designs of few
    levels take level launches."""
    ptr, fan = nl.fanin_ptr, nl.fanin
    gates = [(int(nl.op[g]), fan[ptr[g]:ptr[g + 1]].tolist()) for g in range(nl.n_gates)]
    last = nl.n_nets - 1
    gates += [(synth.INV, [last + i]) for i in range(levels)]
    return synth.from_gates(nl.n_pi, gates)


@pytest.mark.parametrize("gates,pis,depth,B", [
    (5, 3, 5, 1), (63, 4, 1, 1), (64 * 4, 70, 4, 2), (65 * 3, 9, 3, 9), (40_000, 90, 1, 1),
    (70_000, 40_000, 2, 3), (20_000, 500, 2, 40)])
@pytest.mark.parametrize("mode,ste", [(L.DP_MODELED, False), (L.DP_HYBRID, True)])
def test_flow_of_wide_levels_in_deep_designs(ctx, gates, pis, depth, B, mode, ste):
    say(f"dataflow sweep, deep: {gates} gates, {pis} PIs, depth {depth}, B={B}, mode {mode}, ste {ste}")
    nl = _with_chain(synth.random_dag(synth.DagSpec(gates, pis, depth), 11), 200)
    d = api.Design(ctx, nl)
    fixed = (np.arange(pis) % 5 == 0).astype(np.uint8)
    ref = _run(d, nl, L.DP_SCHED_PERSISTENT, B, mode, ste, fixed)
    for sched in (L.DP_SCHED_AUTO, L.DP_SCHED_GRAPH):
        r = _run(d, nl, sched, B, mode, ste, fixed)
        for k in ref:
            np.testing.assert_array_equal(r[k], ref[k], err_msg=f"{k}, schedule {sched}")


@pytest.mark.parametrize("readers", [32, 33, 64, 65, 256, 257, 600, 1300])
def test_flow_long_fanout_ranges_in_deep_designs(ctx, readers):
    say(f"dataflow sweep, deep: {readers} readers")
    gates = [(synth.AND2, [0, 1])]
    gates += [(synth.XOR2 if i % 2 else synth.OR2, [3, 0 if i % 3 else 2]) for i in range(readers)]
    gates += [(synth.MUX2, [4 + i, 3, 4 + (i * 7) % readers]) for i in range(readers)]
    nl = _with_chain(synth.from_gates(3, gates), 200)
    d = api.Design(ctx, nl)
    ref = _run(d, nl, L.DP_SCHED_PERSISTENT, 2, L.DP_MODELED)
    r = _run(d, nl, L.DP_SCHED_AUTO, 2, L.DP_MODELED)
    for k in ref:
        np.testing.assert_array_equal(r[k], ref[k], err_msg=k)

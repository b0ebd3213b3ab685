"""Host-logic scenarios run against the CPU stand-in runtime.

    python -m tests.hoststub.scenarios <libdp_stub.so> <scenario>

Prints one JSON line of results.  The library's host code runs for real
(compile and levelization, validation, schedules and graph capture
bookkeeping, merged level tables, the serving scheduler); the stand-in
launchers check each launch's extents and compute nothing, so numerical
outputs are placeholders and only flows, status codes and host-computed
structure are checked."""
from __future__ import annotations

import dataclasses
import json
import sys

import numpy as np

from paper_2608_03778_amd import _lib

_lib._settle_hip_runtime = lambda: None  # the stand-in runtime only, never a real one
_lib.load(sys.argv[1])

import oracle  # noqa: E402
from paper_2608_03778_amd import _lib as L, api, synth  # noqa: E402


def status_of(fn, *a, **kw):
    """Status name and message of a call ("OK" when it succeeds)."""
    try:
        fn(*a, **kw)
        return "OK", ""
    except L.DiffPowerError as e:
        return L.STATUS_NAMES.get(e.status, str(e.status)), str(e)


def mixed_spec(n_gates, n_pi, depth):
    ops = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(synth.LIBRARY)))
    return synth.DagSpec(n_gates=n_gates, n_pi=n_pi, depth=depth, ops=ops, cells=synth.LIBRARY)


def scenario_compile(ctx):
    out = {}
    nets = {
        "fixed": synth.random_dag(synth.SPECS["dag2k"], 3),
        "library": synth.random_dag(mixed_spec(3000, 64, 18), 4),
        "flop_cut": synth.cut_flops(synth.random_seq_dag(synth.DagSpec(n_gates=1500, n_pi=20,
                                                                       depth=12), 30, 5)).netlist,
        "tree": synth.random_tree(40, 6, cells=synth.LIBRARY,
                                  ops=tuple(range(9)) + (synth.CELL_BASE, synth.CELL_BASE + 4)),
    }
    for name, nl in nets.items():
        d = api.Design(ctx, nl)
        lv = d.levels()
        ref = oracle.Netlist.of(nl).levels()
        out[f"{name}_levels_match"] = bool(np.array_equal(lv, ref))
        out[f"{name}_depth_match"] = int(d.depth) == int(ref.max())
        d.close()
    # fixed cells written as expressions compile to the same levels
    nl = synth.random_dag(synth.DagSpec(n_gates=800, n_pi=32, depth=10, ops=tuple(range(8))), 7)
    expr = dataclasses.replace(nl, op=(nl.op.astype(np.int32) + synth.CELL_BASE).astype(np.uint8),
                               cells=("!A", "A", "A&B", "A|B", "!(A&B)", "!(A|B)", "A^B",
                                      "!(A&B|C)"))
    out["expressions_levels_match"] = bool(np.array_equal(api.Design(ctx, nl).levels(),
                                                          api.Design(ctx, expr).levels()))
    # errors
    cyc = synth.from_gates(2, [(synth.AND2, [0, 3]), (synth.INV, [2])])
    out["cycle"] = status_of(api.Design, ctx, cyc)[0]
    bad_arity = synth.from_gates(2, [(synth.AND2, [0])])
    out["bad_arity"] = status_of(api.Design, ctx, bad_arity)[0]
    bad_op = synth.from_gates(2, [(12, [0, 1])])
    out["bad_op"] = status_of(api.Design, ctx, bad_op)[0]
    bad_net = synth.from_gates(2, [(synth.AND2, [0, 7])])
    out["bad_net"] = status_of(api.Design, ctx, bad_net)[0]
    one = synth.from_gates(3, [(synth.CELL_BASE, [0, 1])], ("A&B",))
    msgs = {}
    for text in ("A&", "(A|B", "A $ B", "A B", "a&b&c&d&e&f&g", "&".join(["A"] * 20),
                 "A|(B|(C|(D|(E|(F|(A|(B|C)))))))", "1"):
        st, msg = status_of(api.Design, ctx, dataclasses.replace(one, cells=(text,)))
        msgs[text] = [st, msg]
    out["parse"] = msgs
    out["cell_arity"] = status_of(api.Design, ctx, dataclasses.replace(one, cells=("A&B&C",)))[0]
    out["cell_missing"] = status_of(api.Design, ctx, dataclasses.replace(one, cells=()))[0]
    return out


def scenario_flows(ctx):
    out = {}
    for name, nl in (("fixed", synth.random_dag(synth.SPECS["dag2k"], 8)),
                     ("library", synth.random_dag(mixed_spec(2500, 48, 14), 9))):
        d = api.Design(ctx, nl)
        cap = synth.net_caps(nl.n_nets, 1)
        runs = 0
        for mode in (L.DP_MODELED, L.DP_HYBRID, L.DP_FROZEN_BETA):
            for B, S in ((1, 0), (3, 2)):
                ev = api.Eval(d, B, S, mode=mode, n_sim=64 * 40, seed=2)
                ev.set_pi_prob(synth.pi_probs(nl.n_pi, 3, batch=B))
                ev.set_caps(cap)
                if S:
                    ev.set_cell_sizes(synth.cell_sizes(nl.n_gates, 4, n_size=S))
                if mode == L.DP_FROZEN_BETA:
                    ev.set_beta(np.ones((B, nl.n_nets), np.float32))
                scheds = [(L.DP_SCHED_LEVEL, 0, 0, 1), (L.DP_SCHED_GRAPH, 0, 0, 1)]
                if mode == L.DP_HYBRID:
                    scheds += [(L.DP_SCHED_LEVEL, 8, 2, 2), (L.DP_SCHED_LEVEL, 6, 1, 3)]
                    if B > 1:  # ragged column groups, alone and with chunks on streams
                        ev.set_sim_columns(2)
                        for chunk, lanes in ((0, 1), (8, 2)):
                            ev.set_schedule(L.DP_SCHED_LEVEL, chunk, 0)
                            ev.set_sim_streams(lanes)
                            ev.forward(("sp", "tr", "power"))
                            runs += 1
                        ev.set_sim_columns(0)
                if name == "fixed":
                    scheds += [(L.DP_SCHED_PERSISTENT, 0, 0, 1)]
                for sched, chunk, ppl, lanes in scheds:
                    ev.set_schedule(sched, chunk, ppl)
                    ev.set_sim_streams(lanes)
                    ev.forward(("sp", "tr", "power"))
                    ev.backward(want=("dpi", "dcap") + (("dsize",) if S else ()))
                    runs += 1
                # a sizing sweep's two sweeps in one call: one captured graph
                # (twice: the second replays it), then the plain calls
                for sched in (L.DP_SCHED_GRAPH, L.DP_SCHED_GRAPH, L.DP_SCHED_LEVEL):
                    ev.set_schedule(sched)
                    ev.set_sim_streams(1)
                    ev.forward_backward_columns()
                    runs += 1
                ev.set_schedule(L.DP_SCHED_LEVEL)
                ev.set_sim_streams(1)
                ev.power_gradients()
                if mode == L.DP_HYBRID and S == 0:
                    tau = np.full((B, nl.n_pi), 0.3, np.float32)
                    ev.set_pi_rates(tau)
                    ev.set_pi_streams((np.arange(nl.n_pi) // 2 * 2).astype(np.int32))
                    ev.set_pi_fixed(np.arange(nl.n_pi) % 5 == 0)
                    for sched, chunk in ((L.DP_SCHED_LEVEL, 0), (L.DP_SCHED_GRAPH, 0),
                                         (L.DP_SCHED_LEVEL, 8)):
                        ev.set_schedule(sched, chunk)
                        ev.forward(("power",))
                        ev.backward(want=("dpi",))
                        runs += 1
                    ev.set_pi_rates(None)
                    ev.set_pi_streams(None)
                    ev.set_pi_fixed(None)
                if mode == L.DP_MODELED and S == 0:
                    ev.power_virus(3, 1e-3)
                    runs += 1
                ev.close()
        out[f"{name}_runs"] = runs
        # validation and state errors
        ev = api.Eval(d, 2, mode=L.DP_HYBRID, n_sim=256)
        out[f"{name}_backward_first"] = status_of(ev.backward, want=("dpi",))[0]
        out[f"{name}_forward_no_inputs"] = status_of(ev.forward, ("power",))[0]
        bad_p = np.full((2, nl.n_pi), 0.5, np.float32)
        bad_p[1, 3] = 1.5
        out[f"{name}_p_range"] = status_of(ev.set_pi_prob, bad_p)[0]
        bad_c = cap.copy()
        bad_c[5] = -1.0
        out[f"{name}_cap_range"] = status_of(ev.set_caps, bad_c)[0]
        out[f"{name}_rates_range"] = status_of(ev.set_pi_rates,
                                               np.full((2, nl.n_pi), 1.5, np.float32))[0]
        out[f"{name}_streams_range"] = status_of(ev.set_pi_streams,
                                                 np.full(nl.n_pi, nl.n_pi, np.int32))[0]
        out[f"{name}_schedule_bad"] = status_of(ev.set_schedule, 9)[0]
        out[f"{name}_persistent"] = status_of(ev.set_schedule, L.DP_SCHED_PERSISTENT)[0]
        ev.set_pi_prob(np.full((2, nl.n_pi), 0.5, np.float32))
        ev.set_caps(cap)
        out[f"{name}_virus_hybrid"] = status_of(ev.power_virus, 2, 0.1)[0]
        ev.close()
        d.close()
    return out


def scenario_group_serving(ctx):
    out = {}
    nls = [synth.random_dag(mixed_spec(2000, 40, 12), 11),
           synth.random_dag(synth.SPECS["dag2k"], 12),
           synth.random_dag(synth.DagSpec(n_gates=5000, n_pi=80, depth=25), 13)]
    designs = [api.Design(ctx, nl) for nl in nls]
    caps = [synth.net_caps(nl.n_nets, 20 + i) for i, nl in enumerate(nls)]
    evs = []
    for i, (nl, d) in enumerate(zip(nls, designs)):
        mode = L.DP_HYBRID if i == 2 else L.DP_MODELED
        ev = api.Eval(d, 2, mode=mode, n_sim=64 * 20, seed=i)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 30 + i, batch=2))
        ev.set_caps(caps[i])
        evs.append(ev)
    grp = api.Group(ctx, evs)
    for use_graph, branches in ((True, 0), (False, 1), (False, 0), (True, 2)):
        grp.configure(use_graph=use_graph, max_branches=branches)
        for backward in (False, True):
            res = grp.run(("sp", "power"), backward=backward)
    out["group_results"] = len(res)
    grp.close()
    srv = api.Server(ctx, hbm_budget_bytes=64 << 20, max_batch=8, max_inflight=3)
    ids = [srv.add_design(d, c, mode=L.DP_MODELED, n_sim=128, seed=5)
           for d, c in zip(designs, caps)]
    rng = np.random.default_rng(1)
    tickets = []
    for k in range(60):
        i = int(rng.integers(0, 3))
        size = None if k % 3 else np.ones(nls[i].n_gates, np.float32)
        tickets.append(srv.submit(ids[i], rng.uniform(0.1, 0.9, nls[i].n_pi).astype(np.float32),
                                  size, bool(k % 2)))
    done = sum(1 for t in tickets if srv.wait(t) is not None)
    st = srv.stats()
    out["served"] = done
    out["completed"] = st["completed"]
    out["batched"] = st["device_steps"] < 60
    bad = np.ones(nls[0].n_gates, np.float32)
    bad[3] = np.nan
    t_bad = srv.submit(ids[0], np.full(nls[0].n_pi, 0.5, np.float32), bad)
    out["nan_size"] = status_of(srv.wait, t_bad)[0]
    out["bad_p"] = status_of(srv.submit, ids[0], np.full(nls[0].n_pi, 2.0, np.float32))[0]
    out["unknown_ticket"] = status_of(srv.wait, 123456)[0]
    srv.close()
    tiny = api.Server(ctx, hbm_budget_bytes=4096)
    tid = tiny.add_design(designs[2], caps[2])
    out["budget"] = status_of(tiny.submit, tid, np.full(nls[2].n_pi, 0.5, np.float32))[0]
    tiny.close()
    return out


def scenario_capture_order(ctx):
    """The order in which a host crash was once seen on the GPU: design
    groups and serving, then the autotuner (graph candidates, several
    simulation streams) on a hybrid eval, in one process; then graph
    captures of multi-column hybrid sweeps and of a hybrid design group.
    The stand-in runtime checks every capture's forks and joins, the calls
    a capturing thread may not make, event reuse across captures, and that
    each graph launch touches only live allocations."""
    out = scenario_group_serving(ctx)
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    cap = synth.net_caps(nl.n_nets, 14)
    for B in (1, 2, 3):
        ev = api.Eval(d, B, mode=L.DP_HYBRID, n_sim=64 * 512, seed=8)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13, batch=B))
        ev.set_caps(cap)
        ev.forward(("sp", "ones", "toggles", "power"))
        ev.autotune(2, with_backward=True)
        ev.forward(("sp", "ones", "toggles", "power"))
        ev.backward(want=("dpi",))
        for chunk, lanes in ((128, 2), (0, 1), (128, 3)):
            ev.set_schedule(L.DP_SCHED_GRAPH, chunk, 0)
            ev.set_sim_streams(lanes)
            ev.forward(("power",))
            ev.backward(want=("dpi",))
        ev.close()
    evs = []
    for i in range(3):
        e = api.Eval(d, 2, mode=L.DP_HYBRID if i else L.DP_MODELED, n_sim=64 * 16, seed=i)
        e.set_pi_prob(synth.pi_probs(nl.n_pi, 40 + i, batch=2))
        e.set_caps(cap)
        evs.append(e)
    grp = api.Group(ctx, evs)
    for use_graph in (True, False, True):
        grp.configure(use_graph=use_graph)
        grp.run(("power",), backward=True)
    grp.close()
    out["capture_order_done"] = True
    import ctypes
    counts = (ctypes.c_long * 3)()
    ctypes.CDLL(sys.argv[1]).stub_capture_counts(counts)
    out["captures"], out["forks"], out["graph_launches"] = counts[0], counts[1], counts[2]
    return out


def scenario_group_persistent(ctx):
    """Groups of evals whose own schedule is the persistent one, which the group
    does not use."""
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    evs = []
    for mode in (L.DP_HYBRID, L.DP_MODELED, L.DP_HYBRID):
        ev = api.Eval(d, 2, mode=mode, n_sim=64 * 20, seed=3)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 30, batch=2))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        ev.set_schedule(L.DP_SCHED_PERSISTENT)
        evs.append(ev)
    grp = api.Group(ctx, evs)
    for use_graph in (True, False):
        grp.configure(use_graph=use_graph)
        res = grp.run(("sp", "power"), backward=True)
    return {"results": len(res), "schedules": [ev.get_schedule()["schedule"] for ev in evs]}


def scenario_group_after_columns(ctx):
    """Groups of evals whose reverse sweep alone goes by level launches: one
    that has made the smaller scratch of a sweep over (b, s) columns before,
    beside a fresh one, and each by itself."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 5)()
    n_pi = 1500  # two levels, up to four readers a net
    first = [(synth.AND2, [i, (i * 7 + 1) % n_pi]) for i in range(n_pi)]
    nl = synth.from_gates(n_pi, first + [(synth.MUX2, [n_pi + i, n_pi + (i * 5 + 2) % n_pi, i])
                                         for i in range(n_pi)])
    d = api.Design(ctx, nl)

    def make(S):
        ev = api.Eval(d, 4, S)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 30, batch=4))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        ev.set_cell_sizes(synth.cell_sizes(nl.n_gates, 3, n_size=S))
        return ev
    used, fresh = make(64), make(2)
    used.forward(("power",))
    used.backward_columns()
    stub.stub_sweep_counts(counts)
    n, wide = 0, counts[4] > 0
    for evs in ([used], [used, fresh], [fresh], [used, make(64)]):
        grp = api.Group(ctx, evs)
        for use_graph in (True, False):
            grp.configure(use_graph=use_graph)
            n += len(grp.run(("power",), backward=True))
        grp.close()
        used.backward_columns()
    return {"results": n, "wide": wide}


def scenario_group_routes(ctx):
    """Which way groups' forward and reverse sweeps go: [forward, reverse], "flow"
    or "levels", launched as they are and recorded into a graph."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    f, b = (ctypes.c_long * 2)(), (ctypes.c_long * 2)()

    def counts():
        stub.stub_multi_counts(f)
        stub.stub_multi_reverse_counts(b)
        return list(f), list(b)
    out = {}
    lib = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(3))
    for name, gates, depth, n, B, cells in (
            ("deep", 2000, 40, 3, 2, False), ("shallow", 20_000, 2, 4, 8, False),
            ("middle", 20_000, 4, 2, 16, False), ("shallow, one column", 20_000, 2, 4, 1, False),
            ("shallow cells", 20_000, 2, 4, 16, True), ("deep cells", 2000, 20, 3, 4, True)):
        nl = synth.random_dag(synth.DagSpec(gates, 500, depth, ops=lib if cells else tuple(range(9)),
                                            cells=synth.LIBRARY[:3] if cells else ()), 13)
        d = api.Design(ctx, nl)
        evs = []
        for i in range(n):
            ev = api.Eval(d, B)
            ev.set_pi_prob(synth.pi_probs(nl.n_pi, 30 + i, batch=B))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            evs.append(ev)
        grp = api.Group(ctx, evs)
        for use_graph in (False, True):
            grp.configure(use_graph=use_graph)
            for backward in (True, False, True):
                f0, b0 = counts()
                grp.run(("power",), backward=backward)
                f1, b1 = counts()
                got = ["flow" if x1[0] > x0[0] else "levels" if x1[1] > x0[1] else "-"
                       for x0, x1 in ((f0, f1), (b0, b1))]
                out.setdefault(name, got if backward else None)
                want = out[name] if backward else [out[name][0], "-"]
                assert got == want, (name, use_graph, backward, got, want)
        grp.close()
        for ev in evs:
            ev.close()
    return out


def scenario_deep_graphs(ctx):
    """Captures of the reverse sweep of chains whose level launches are about as
    many as a graph takes (1,024)."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 3)()
    out = {}
    for depth in (1021, 1022, 1023, 1024):
        nl = synth.from_gates(1, [(synth.INV, [i]) for i in range(depth)])
        ev = api.Eval(api.Design(ctx, nl), 1)
        ev.set_pi_prob(np.full((1, 1), 0.5, np.float32))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        ev.set_schedule(L.DP_SCHED_GRAPH)
        ev.forward(("power",))
        stub.stub_capture_counts(counts)
        before = counts[0]
        ev.backward(want=("dpi",))
        stub.stub_capture_counts(counts)
        out[str(depth)] = counts[0] - before
        ev.close()
    return out


def scenario_profile(ctx):
    """What the profile books a forward under (the stand-in's events are a
    microsecond apart)."""
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    out = {}
    for name, B, mode in (("modeled", 1, L.DP_MODELED), ("rides", 1, L.DP_HYBRID),
                          ("rides2", 2, L.DP_HYBRID), ("apart", 3, L.DP_HYBRID)):
        ev = api.Eval(d, B, mode=mode, n_sim=64 * 40, seed=8)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13, batch=B))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        ev.profile(True)
        ev.forward(("power",))
        out[name] = ev.get_profile()
        ev.close()
    return out


def scenario_tile_memory(ctx):
    """A short simulation on a device that holds the level launches' words and not
    the tiles', and a second after there is memory."""
    import ctypes
    import time
    stub = ctypes.CDLL(sys.argv[1])
    stub.stub_live_bytes.restype = ctypes.c_long
    counts = (ctypes.c_long * 2)()
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    out = {}

    def sims(ev):
        stub.stub_sim_counts(counts)
        before = list(counts)
        st = status_of(ev.forward, ("power",))[0]
        stub.stub_sim_counts(counts)
        return [st, counts[0] > before[0], counts[1] > before[1]]
    for sched in (L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH):
        def make():
            ev = api.Eval(d, 1, mode=L.DP_HYBRID, n_sim=64 * 1280, seed=8)
            ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            ev.set_schedule(sched)
            return ev
        ev = make()
        out[f"{sched} all"] = sims(ev)
        live = stub.stub_live_bytes()
        ev.close()
        ev = make()
        stub.stub_set_memory(live - 100_000)
        out[f"{sched} less"] = sims(ev)
        out[f"{sched} again"] = sims(ev)
        stub.stub_set_memory(0)
        time.sleep(1.1)
        out[f"{sched} later"] = sims(ev)
        ev.close()
    return out


def scenario_scratch_memory(ctx):
    """Reverse sweeps on a device that holds the level launches' buffers and not
    the dataflow sweep's, alone and in a group, and a second after there is
    memory."""
    import ctypes
    import time
    stub = ctypes.CDLL(sys.argv[1])
    stub.stub_live_bytes.restype = ctypes.c_long
    counts = (ctypes.c_long * 5)()
    multi = (ctypes.c_long * 2)()
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    out = {}

    def flows(call):
        stub.stub_sweep_counts(counts)
        before = counts[2]
        st = status_of(call)[0]
        stub.stub_sweep_counts(counts)
        return [st, counts[2] > before]
    for sched in (L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH):
        def make():
            ev = api.Eval(d, 16)
            ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13, batch=16))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            ev.set_schedule(sched)
            ev.forward(("power",))
            return ev
        ev = make()
        out[f"{sched} all"] = flows(ev.backward)
        live = stub.stub_live_bytes()
        ev.close()
        ev = make()
        stub.stub_set_memory(live - 100_000)
        out[f"{sched} less"] = flows(ev.backward)
        out[f"{sched} again"] = flows(ev.backward)
        stub.stub_set_memory(0)
        time.sleep(1.1)
        out[f"{sched} later"] = flows(ev.backward)
        ev.close()
    evs = []
    for i in range(2):
        ev = api.Eval(d, 16)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13 + i, batch=16))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        evs.append(ev)
    grp = api.Group(ctx, evs)
    grp.configure(use_graph=False)
    grp.run(("power",))

    def group():
        stub.stub_multi_reverse_counts(multi)
        before = list(multi)
        st = status_of(grp.run, ("power",), True)[0]
        stub.stub_multi_reverse_counts(multi)
        return [st, multi[0] > before[0], multi[1] > before[1]]
    live = stub.stub_live_bytes()
    edges = len(nl.fanin)
    stub.stub_set_memory(live + 2 * 16 * 4 * (edges + nl.n_pi) + 150_000)  # the contributions
    out["group less"] = group()
    stub.stub_set_memory(0)
    time.sleep(1.1)
    out["group later"] = group()
    return out


def scenario_autotune(ctx):
    """What the autotuner times (launches of word tiles and of simulation levels),
    entered with each schedule."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 2)()
    nl = synth.random_dag(synth.SPECS["dag2k"], 13)
    d = api.Design(ctx, nl)
    out = {}
    for name, sched in (("level", L.DP_SCHED_LEVEL), ("persistent", L.DP_SCHED_PERSISTENT)):
        ev = api.Eval(d, 1, mode=L.DP_HYBRID, n_sim=64 * 300, seed=8)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 13))
        ev.set_caps(synth.net_caps(nl.n_nets, 14))
        ev.set_schedule(sched)
        stub.stub_sim_counts(counts)
        before = list(counts)
        ev.autotune(2)
        stub.stub_sim_counts(counts)
        out[name] = [counts[0] - before[0], counts[1] - before[1]]
        ev.close()
    return out


def scenario_server_give_up(ctx):
    """A serving step whose sweep gives up, and the steps after it."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    nls = [synth.random_dag(synth.SPECS["dag2k"], 12), synth.random_dag(synth.DagSpec(900, 30, 9), 13)]
    srv = api.Server(ctx, hbm_budget_bytes=64 << 20, max_batch=8, max_inflight=1)
    ids = [srv.add_design(api.Design(ctx, nl), synth.net_caps(nl.n_nets, 20)) for nl in nls]

    def query(i):
        return status_of(srv.wait, srv.submit(ids[i], np.full(nls[i].n_pi, 0.5, np.float32), None, True))
    out = {"before": [query(i)[0] for i in (0, 1)]}
    stub.stub_fail_flows(1)
    out["failed"] = query(0)
    out["after"] = [query(i)[0] for i in (0, 1, 0)]
    srv.close()
    return out


def scenario_sweep_routes(ctx):
    """Whether the SP and the reverse sweep of a shape go out as dataflow launches."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 5)()
    out = {}
    lib = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(synth.LIBRARY)))
    for gates, pis, depth, ops, cells in ((2000, 64, 20, tuple(range(9)), ()), (20_000, 500, 2, tuple(range(9)), ()),
                                          (20_000, 500, 60, tuple(range(9)), ()),
                                          (117_000, 2000, 3, tuple(range(9)), ()),
                                          (117_000, 2000, 60, tuple(range(9)), ()),
                                          (20_000, 500, 2, lib, synth.LIBRARY),
                                          (20_000, 500, 60, lib, synth.LIBRARY)):
        nl = synth.random_dag(synth.DagSpec(gates, pis, depth, ops=ops, cells=cells), 13)
        d = api.Design(ctx, nl)
        for B in (1, 16, 64):
            ev = api.Eval(d, B)
            ev.set_pi_prob(np.full((B, nl.n_pi), 0.5, np.float32))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            stub.stub_sweep_counts(counts)
            c0 = list(counts)
            ev.forward(("power",))
            ev.backward(want=("dpi",))
            stub.stub_sweep_counts(counts)
            got = [counts[k] - c0[k] for k in range(5)]
            assert (got[0] > 0) != (got[1] > 0) and (got[2] > 0) != (got[3] > 0), got
            out[f"{gates} {depth} {'cells' if cells else 'fixed'} {B}"] = [got[0] > 0, got[2] > 0]
            ev.close()
    return out


def scenario_tile_routes(ctx):
    """Whether the simulation of a shape goes out in word tiles."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 2)()
    out = {}
    for gates, pis, depth in ((2000, 64, 20), (20_000, 500, 30), (117_000, 2000, 3), (117_000, 2000, 60)):
        nl = synth.random_dag(synth.DagSpec(gates, pis, depth), 13)
        d = api.Design(ctx, nl)
        for B, T in ((1, 16), (1, 1024), (4, 96)):
            ev = api.Eval(d, B, mode=L.DP_HYBRID, n_sim=64 * T, seed=8)
            ev.set_pi_prob(np.full((B, nl.n_pi), 0.5, np.float32))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            stub.stub_sim_counts(counts)
            c0 = list(counts)
            ev.forward(("power",))
            stub.stub_sim_counts(counts)
            out[f"{gates} {depth} {B}x{T}"] = counts[0] > c0[0]
            ev.close()
    return out


def scenario_wide_routes(ctx):
    """Whether a sizing sweep's gradients go in adjoints: gates times columns at
    and below 130,000 a strand, from the design's own fan-out."""
    import ctypes
    stub = ctypes.CDLL(sys.argv[1])
    counts = (ctypes.c_long * 5)()
    out = {}
    lib = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(synth.LIBRARY)))
    for name, spec in (("fixed", synth.DagSpec(3000, 90, 9)), ("far", synth.DagSpec(3000, 90, 9, fo_mean=3.0, fo_cap=256)),
                       ("cells", synth.DagSpec(3000, 90, 9, ops=lib, cells=synth.LIBRARY))):
        nl = synth.random_dag(spec, 22)
        lv = oracle.Netlist.of(nl).levels()
        longest = np.zeros(int(lv.max()) + 1, np.int64)
        np.maximum.at(longest, lv, np.bincount(nl.fanin, minlength=nl.n_nets))
        line = int(130_000 * (-(-longest // 8)).sum() / nl.n_gates)  # columns
        d = api.Design(ctx, nl)
        for what, B, S in (("below", line // 32 - 1, 32), ("above", line // 32 + 2, 32), ("few sizes", 2 * line // 15, 15),
                           ("small", 5, 16)):
            ev = api.Eval(d, B, S)
            ev.set_pi_prob(np.full((B, nl.n_pi), 0.5, np.float32))
            ev.set_caps(synth.net_caps(nl.n_nets, 14))
            ev.set_cell_sizes(np.ones((S, nl.n_gates), np.float32))
            ev.forward(("power",))
            stub.stub_sweep_counts(counts)
            c0 = list(counts)
            ev.backward_columns()
            stub.stub_sweep_counts(counts)
            got = [counts[k] - c0[k] for k in range(5)]
            assert sum(x > 0 for x in got[2:]) == 1, got
            out[f"{name} {what}"] = got[4] > 0
            ev.close()
    return out


def scenario_lane_memory(ctx):
    """Serving with a device that has less memory than the budget says: enough
    for a lane, and not for its dataflow sweeps' buffers."""
    import ctypes
    import time
    stub = ctypes.CDLL(sys.argv[1])
    stub.stub_live_bytes.restype = ctypes.c_long
    counts = (ctypes.c_long * 2)()
    nl = synth.random_dag(synth.SPECS["dag2k"], 12)
    d = api.Design(ctx, nl)
    out = {}

    def serve(limit, later=False):
        srv = api.Server(ctx, hbm_budget_bytes=64 << 20, max_batch=8, max_inflight=2)
        did = srv.add_design(d, synth.net_caps(nl.n_nets, 20))
        stub.stub_set_memory(limit)
        stub.stub_multi_counts(counts)
        before = list(counts)
        t = srv.submit(did, np.full(nl.n_pi, 0.5, np.float32), None, True)
        end = time.time() + 5
        while not srv.poll(t) and time.time() < end:
            time.sleep(0.01)
        done = srv.poll(t)
        stub.stub_multi_counts(counts)
        stub.stub_set_memory(0)
        live = stub.stub_live_bytes()
        if done and later:  # the same lane, once there is memory and a second has passed
            first = list(counts)
            time.sleep(1.1)
            srv.wait(srv.submit(did, np.full(nl.n_pi, 0.5, np.float32), None, True))
            stub.stub_multi_counts(counts)
            out["later"] = [counts[0] > first[0], counts[1] > first[1]]
            out["lanes"] = srv.stats()["lanes_created"]
            counts[0], counts[1] = first
        if done:
            srv.wait(t)
        srv.close()
        return [done, counts[0] > before[0], counts[1] > before[1], live]
    out["all"] = serve(0)
    out["less"] = serve(out["all"][3] - 100_000, later=True)
    return out


def scenario_large_faces(ctx):
    """Forward sweeps whose (b, s) results times slabs of nets are beyond 2^31
    and 2^32 (the stand-in touches the last partial that the contraction
    writes), and the device memory they take beside their inputs and powers."""
    import ctypes
    live = ctypes.CDLL(sys.argv[1]).stub_live_bytes
    live.restype = ctypes.c_long
    out = {}
    for gates, B, S in ((16_384, 4096, 4096), (16_384, 2048, 4100)):
        nl = synth.random_dag(synth.DagSpec(gates, 64, 8), 15)
        ev = api.Eval(api.Design(ctx, nl), B, S)
        ev.set_pi_prob(np.full((B, nl.n_pi), 0.5, np.float32))
        ev.set_caps(synth.net_caps(nl.n_nets, 1))
        ev.set_cell_sizes(np.ones((S, nl.n_gates), np.float32))
        before = live()
        out[f"{B}x{S}"] = status_of(ev.forward, ("power",))[0]
        out[f"{B}x{S} bytes"] = live() - before - 4 * B * S
        ev.close()
    return out


if __name__ == "__main__":
    context = api.Context(0)
    result = {"compile": scenario_compile, "flows": scenario_flows,
              "group_serving": scenario_group_serving,
              "capture_order": scenario_capture_order,
              "group_persistent": scenario_group_persistent,
              "scratch_memory": scenario_scratch_memory,
              "group_routes": scenario_group_routes,
              "group_after_columns": scenario_group_after_columns,
              "deep_graphs": scenario_deep_graphs,
              "profile": scenario_profile,
              "tile_memory": scenario_tile_memory,
              "autotune": scenario_autotune,
              "server_give_up": scenario_server_give_up,
              "sweep_routes": scenario_sweep_routes,
              "tile_routes": scenario_tile_routes,
              "wide_routes": scenario_wide_routes,
              "lane_memory": scenario_lane_memory,
              "large_faces": scenario_large_faces}[sys.argv[2]](context)
    print(json.dumps(result), flush=True)

"""The (b, s) contraction and the size vectors' layout at the edges of their
tiles: B and S around 16 and 32 (one or two matrix tiles a side), nets around
a slab, against the FP64 oracle; and a column's power and gradients the same
bits whatever else shares the call."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import assert_grad_close, assert_power_close, oracle_column, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gates,pis,B,S,mode", [
    (60, 4, 1, 1, "modeled"), (60, 4, 15, 17, "hybrid"), (61, 4, 16, 16, "frozen"),
    (300, 20, 17, 33, "modeled"), (2000, 64, 32, 31, "hybrid"), (2000, 64, 3, 65, "modeled"),
    (17_000, 200, 2, 3, "modeled"), (4, 2, 5, 40, "modeled")])
def test_many_size_vectors(gates, pis, B, S, mode):
    say(f"contraction: {gates} gates, B={B}, S={S}, {mode}")
    nl = synth.random_dag(synth.DagSpec(gates, pis, min(gates, 8)), 21)
    p, cap = synth.pi_probs(pis, 1, batch=B), synth.net_caps(nl.n_nets, 2)
    size = synth.cell_sizes(nl.n_gates, 3, n_size=S)
    beta = np.random.default_rng(4).uniform(0.2, 3.0, (B, nl.n_nets)).astype(np.float32)
    modes = {"modeled": L.DP_MODELED, "hybrid": L.DP_HYBRID, "frozen": L.DP_FROZEN_BETA}

    def run(bs, ss):
        ev = api.Eval(api.Design(api.Context(0), nl), len(bs), len(ss), mode=modes[mode],
                      n_sim=64 * 12, seed=9)
        ev.set_pi_prob(p[bs])
        ev.set_caps(cap)
        ev.set_cell_sizes(size[ss])
        if mode == "frozen":
            ev.set_beta(beta[bs])
        return ev.forward(("power",))["power"], ev.backward_columns()
    power, dpi = run(list(range(B)), list(range(S)))
    bs, ss = [B - 1], [0, S - 1] if S > 1 else [0]
    sub_power, sub_dpi = run(bs, ss)
    np.testing.assert_array_equal(sub_power, power[np.ix_(bs, ss)])
    np.testing.assert_array_equal(sub_dpi, dpi[np.ix_(bs, ss)])
    o = oracle.Netlist.of(nl)
    for b, s in {(0, 0), (B - 1, S - 1), (B // 2, S // 2)}:
        f, adj = oracle_column(o, p[b], cap, size[s], mode=mode, n_words=12, seed=9,
                               beta=beta[b] if mode == "frozen" else None)
        assert_power_close(power[b, s], f["power"], f"power {b} {s}")
        assert_grad_close(dpi[b, s], oracle_adjoint(o, f, cap, size[s], beta[b], mode, adj),
                          f"dP/dp {b} {s}")


# 257 slabs of nets: faces whose partials take two pieces of columns, of size
# vectors, and of both with a remainder in each
@pytest.mark.parametrize("B,S", [(130, 300), (20, 2000), (97, 1100)])
def test_size_contraction_in_pieces(B, S):
    say(f"contraction in pieces: B={B}, S={S}")
    nl = synth.random_dag(synth.DagSpec(16_384, 64, 8), 23)
    p, cap = synth.pi_probs(nl.n_pi, 1, batch=B), synth.net_caps(nl.n_nets, 2)
    size = np.random.default_rng(3).uniform(0.3, 4.0, (S, nl.n_gates)).astype(np.float32)
    d = api.Design(api.Context(0), nl)

    def run(bs, ss):
        ev = api.Eval(d, len(bs), len(ss))
        ev.set_pi_prob(p[bs])
        ev.set_caps(cap)
        ev.set_cell_sizes(size[ss])
        return ev.forward(("power",))["power"]
    power = run(np.arange(B), np.arange(S))
    for bs in (np.arange(0, B, 2), np.arange(1, B, 2)):  # each small enough for one piece
        for k in range(4):
            ss = np.arange(k, S, 4)
            np.testing.assert_array_equal(run(bs, ss), power[np.ix_(bs, ss)])
    o = oracle.Netlist.of(nl)
    for b, s in {(0, 0), (B - 1, S - 1), (B // 2, S // 2)}:
        f, _ = oracle_column(o, p[b], cap, size[s])
        assert_power_close(power[b, s], f["power"], f"power {b} {s}")


def oracle_adjoint(o, f, cap, size, beta, mode, adj):
    """The adjoint with the beta in force (oracle_column's own for modeled and
    hybrid columns)."""
    if mode != "frozen":
        return adj["dpi"]
    return o.adjoint(f["sp"], beta, cap, size)["dpi"]


# column counts that take one and four columns a lane, b crossing a lane's
# and a wave's columns; nets of more than 32 readers among them
@pytest.mark.parametrize("gates,pis,depth,B,S,mode,cells,ste", [
    (3000, 90, 9, 8, 64, "modeled", False, False), (3000, 90, 9, 5, 100, "hybrid", False, True),
    (3000, 90, 9, 3, 33, "hybrid", True, False), (12_000, 300, 6, 3, 256, "modeled", False, False),
    (300, 70, 3, 16, 17, "modeled", False, False)])
def test_reverse_of_many_size_vectors(gates, pis, depth, B, S, mode, cells, ste):
    """The sweep in adjoints is bit for bit the one in contributions (the
    persistent schedule's), alone and in one graph with the forward, and a
    column's gradient does not depend on the others."""
    say(f"many sizes, reverse: {gates} gates, B={B}, S={S}, {mode}, cells {cells}, ste {ste}")
    ops = tuple(range(9)) + (tuple(synth.CELL_BASE + c for c in range(9)) if cells else ())
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth, ops=ops, fo_mean=3.0, fo_cap=256,
                                        cells=synth.LIBRARY if cells else ()), 22)
    d = api.Design(api.Context(0), nl)
    p, cap = synth.pi_probs(pis, 1, batch=B), synth.net_caps(nl.n_nets, 2)
    size = np.random.default_rng(3).uniform(0.3, 4.0, (S, nl.n_gates)).astype(np.float32)
    fixed = (np.arange(pis) % 7 == 0).astype(np.uint8)

    def make(bs, ss, sched):
        ev = api.Eval(d, len(bs), len(ss), n_sim=64 * 8, seed=2,
                      mode=L.DP_HYBRID if mode == "hybrid" else L.DP_MODELED,
                      beta_grad=L.DP_BETA_STE if ste else L.DP_BETA_LOCAL)
        ev.set_pi_prob(p[bs])
        ev.set_caps(cap)
        ev.set_cell_sizes(size[ss])
        ev.set_pi_fixed(fixed)
        ev.set_schedule(sched)
        return ev
    every = (list(range(B)), list(range(S)))
    ev = make(*every, L.DP_SCHED_AUTO)
    ev.forward(("power",))
    dpi = ev.backward_columns()
    np.testing.assert_array_equal(ev.backward_columns(), dpi)
    ev = make(*every, L.DP_SCHED_GRAPH)
    for _ in range(3):
        _, g = ev.forward_backward_columns()
        np.testing.assert_array_equal(g, dpi)
    if not cells:
        ev = make(*every, L.DP_SCHED_PERSISTENT)
        ev.forward(("power",))
        np.testing.assert_array_equal(ev.backward_columns(), dpi)
    ev = make([0, B - 1], [1, S - 1], L.DP_SCHED_AUTO)
    ev.forward(("power",))
    np.testing.assert_array_equal(ev.backward_columns(), dpi[np.ix_([0, B - 1], [1, S - 1])])
    o = oracle.Netlist.of(nl)
    f, adj = oracle_column(o, p[B - 1], cap, size[S - 1], mode=mode, n_words=8, seed=2, ste=ste)
    assert_grad_close(dpi[B - 1, S - 1], np.where(fixed, 0.0, adj["dpi"]), "dP/dp")


# columns enough for the sweep in adjoints (the ones above are in contributions
# but for the library cells), four columns a lane and one, with hybrid beta, STE
# and library cells
@pytest.mark.parametrize("gates,pis,depth,B,S,mode,cells,ste", [
    (3000, 90, 9, 24, 256, "modeled", False, False), (3000, 90, 9, 40, 129, "hybrid", False, True),
    (12_000, 300, 6, 8, 256, "hybrid", False, False), (300, 70, 3, 64, 256, "modeled", False, False),
    (300, 70, 3, 150, 65, "modeled", False, False), (3000, 90, 9, 24, 256, "hybrid", True, True)])
def test_reverse_of_very_many_size_vectors(gates, pis, depth, B, S, mode, cells, ste):
    test_reverse_of_many_size_vectors(gates, pis, depth, B, S, mode, cells, ste)


def weighted_adjoints(o, p, cap, size, w, mode, ste):
    """dP/dp [B][n_pi] and dP/dC [nets] of sum over (b, s) of w power, in FP64."""
    dpi, dcap = [], 0.0
    for b in range(len(p)):
        adj = [oracle_column(o, p[b], cap, size[s], mode=mode, n_words=8, seed=2, ste=ste)[1]
               for s in range(len(size))]
        dpi.append(sum(w[b, s] * a["dpi"] for s, a in enumerate(adj)))
        dcap = dcap + sum(w[b, s] * a["dcap"] for s, a in enumerate(adj))
    return np.stack(dpi), dcap


# size vectors around a staged chunk (16) and the fewest that are staged (4);
# columns around the row kernel's fewest (16) and its tile (32); blocks of nets
# that end in the next column, and in the second next of a small design
@pytest.mark.parametrize("gates,pis,B,S,mode,cells,ste,weighted", [
    (700, 30, 3, 3, "modeled", False, False, True), (700, 30, 3, 4, "modeled", False, False, True),
    (60, 5, 9, 5, "modeled", False, False, True), (700, 30, 15, 16, "modeled", False, False, False),
    (700, 300, 16, 17, "hybrid", False, False, True), (226, 30, 33, 15, "hybrid", False, False, True),
    (700, 30, 2, 33, "modeled", True, False, True), (700, 30, 17, 48, "hybrid", True, True, False)])
def test_gradients_weighted_over_size_vectors(gates, pis, B, S, mode, cells, ste, weighted):
    say(f"gradients over sizes: {gates} gates, B={B}, S={S}, {mode}, cells {cells}")
    ops = tuple(range(9)) + (tuple(synth.CELL_BASE + c for c in range(9)) if cells else ())
    nl = synth.random_dag(synth.DagSpec(gates, pis, 6, ops=ops, fo_mean=3.0, fo_cap=64,
                                        cells=synth.LIBRARY if cells else ()), 25)
    ctx = api.Context(0)
    d = api.Design(ctx, nl)
    p, cap = synth.pi_probs(pis, 1, batch=B), synth.net_caps(nl.n_nets, 2)
    rng = np.random.default_rng(3)
    size = rng.uniform(0.3, 4.0, (S, nl.n_gates)).astype(np.float32)
    w = rng.uniform(0.2, 1.8, (B, S)).astype(np.float32) if weighted else None

    def make(bs, sched):
        ev = api.Eval(d, len(bs), S, n_sim=64 * 8, seed=2,
                      mode=L.DP_HYBRID if mode == "hybrid" else L.DP_MODELED,
                      beta_grad=L.DP_BETA_STE if ste else L.DP_BETA_LOCAL)
        ev.set_pi_prob(p[bs])
        ev.set_caps(cap)
        ev.set_cell_sizes(size)
        ev.set_schedule(sched)
        return ev

    def run(bs, sched):
        ev = make(bs, sched)
        ev.forward(("power",))
        return ev.backward(None if w is None else w[bs], want=("dpi", "dcap"))
    every = list(range(B))
    g = run(every, L.DP_SCHED_AUTO)
    for sched in (L.DP_SCHED_LEVEL,) if cells else (L.DP_SCHED_LEVEL, L.DP_SCHED_PERSISTENT):
        ref = run(every, sched)
        for k in ref:
            np.testing.assert_array_equal(g[k], ref[k], err_msg=f"{k}, schedule {sched}")
    np.testing.assert_array_equal(run([B - 1], L.DP_SCHED_AUTO)["dpi"][0], g["dpi"][B - 1])
    dpi, dcap = weighted_adjoints(oracle.Netlist.of(nl), p, cap, size,
                                  np.ones((B, S)) if w is None else w, mode, ste)
    for b in (0, B - 1):
        assert_grad_close(g["dpi"][b], dpi[b], f"dP/dp {b}")
    assert_grad_close(g["dcap"], dcap, "dP/dC")
    if w is None:  # (a group's gradients are of the sum)
        evs = [make(every, L.DP_SCHED_AUTO), make([0], L.DP_SCHED_AUTO)]
        grp = api.Group(ctx, evs)
        for _ in range(2):
            r = grp.run(("power",), backward=True)
            np.testing.assert_array_equal(r[0]["dpi"], g["dpi"])
            np.testing.assert_array_equal(r[1]["dpi"][0], g["dpi"][0])


# gates that end within a block, vectors around one block's 32; two vectors,
# and faces just below and above the size from which whole runs are written
@pytest.mark.parametrize("gates,S", [(400_001, 2), (50_003, 15), (50_003, 16), (25_027, 33),
                                     (12_700, 65), (800_000, 1)])
def test_order_of_large_size_arrays(gates, S):
    say(f"size arrays: {gates} gates x {S}")
    import torch
    nl = synth.random_dag(synth.DagSpec(gates, 500, 6), 26)
    d = api.Design(api.Context(0, torch.cuda.current_stream().cuda_stream), nl)
    size = np.random.default_rng(5).uniform(0.3, 4.0, (S, gates)).astype(np.float32)
    cap = synth.net_caps(nl.n_nets, 2)

    def power(sizes):
        ev = api.Eval(d, 1, len(sizes))
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 1, batch=1))
        ev.set_caps(cap)
        ev.set_cell_sizes(sizes)
        return ev.forward(("power", "sp"))
    r = power(size)
    np.testing.assert_array_equal(power(torch.from_numpy(size).cuda())["power"], r["power"])
    for s in range(S):  # a vector by itself is gathered below 800K gates
        np.testing.assert_array_equal(power(size[s:s + 1])["power"][0, 0], r["power"][0, s])
    p = r["sp"][0].astype(np.float64)
    term = 0.5 * cap.astype(np.float64) * 2 * p * (1 - p)
    ref = term[:nl.n_pi].sum() + size.astype(np.float64) @ term[nl.n_pi:]
    assert_power_close(r["power"][0], ref, "power")

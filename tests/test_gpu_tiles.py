"""The simulation in word tiles (all levels in one launch, each tile by one
team of workgroups): counts bit for bit the level launches' and the oracle's,
at words around the pitches (16, 32, 64) and the tile limits, level widths
below and beyond a team's turn, each form of stimulus, and library cells."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import SP_ABS, say

pytestmark = pytest.mark.gpu
FIELDS = ("ones", "toggles", "sp", "beta", "power")


@pytest.fixture(scope="module")
def ctx():
    return api.Context(0)


def _eval(d, nl, B, T, stim=None, tau=None, stream=None):
    ev = api.Eval(d, B, mode=L.DP_HYBRID, n_sim=64 * T, seed=9)
    ev.set_pi_prob(synth.pi_probs(nl.n_pi, 41, batch=B))
    ev.set_caps(synth.net_caps(nl.n_nets, 42))
    if stim is not None:
        ev.set_stimulus(stim)
    if tau is not None:
        ev.set_pi_rates(tau)
    if stream is not None:
        ev.set_pi_streams(stream)
    return ev


def _same(a, b, msg):
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=f"{k}, {msg}")


@pytest.mark.parametrize("gates,pis,depth,B,T", [
    (5, 3, 5, 1, 2), (64, 9, 1, 2, 3), (700, 33, 7, 1, 15), (700, 33, 7, 3, 16), (700, 33, 7, 1, 17),
    (700, 33, 7, 1, 384), (700, 33, 7, 1, 385), (700, 33, 7, 24, 7), (700, 33, 7, 25, 7),
    (700, 33, 7, 1, 769), (700, 33, 7, 2, 1024), (700, 33, 7, 1, 2049), (6500, 2100, 3, 1, 33),
    (9000, 50, 1, 1, 250), (9000, 50, 1, 1, 100), (3000, 40, 900, 1, 40)])
def test_tiles_are_the_level_launches(ctx, gates, pis, depth, B, T):
    say(f"word tiles: {gates} gates, {pis} PIs, depth {depth}, B={B}, T={T}")
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth), 43)
    d = api.Design(ctx, nl)
    ref = _eval(d, nl, B, T)
    ref.set_schedule(L.DP_SCHED_LEVEL, T)  # a chunk that is set: level launches
    want = ref.forward(FIELDS)
    ev = _eval(d, nl, B, T)
    for _ in range(2):
        _same(ev.forward(FIELDS), want, "tiles")
    ev.set_schedule(L.DP_SCHED_GRAPH)
    for k in range(3):
        _same(ev.forward(FIELDS), want, f"graph replay {k}")
    p, cap = synth.pi_probs(pis, 41, batch=B), synth.net_caps(nl.n_nets, 42)
    f = oracle.Netlist.of(nl).forward(p[B - 1], cap, hybrid=True, n_words=T,
                                      pi_words=oracle.stimulus_model(p[B - 1], 9, T))
    np.testing.assert_array_equal(want["ones"][B - 1].astype(np.uint64), f["ones"])
    np.testing.assert_array_equal(want["toggles"][B - 1].astype(np.uint64), f["toggles"])


@pytest.mark.parametrize("form", ["explicit", "markov", "streams"])
@pytest.mark.parametrize("B,T", [(1, 21), (3, 130)])
def test_tiles_with_each_stimulus(ctx, form, B, T):
    say(f"word tiles: {form}, B={B}, T={T}")
    nl = synth.random_dag(synth.DagSpec(900, 31, 9), 44)
    d = api.Design(ctx, nl)
    rng = np.random.default_rng(45)
    kw = {}
    if form == "explicit":
        kw["stim"] = rng.integers(0, 2 ** 64, size=(B, nl.n_pi, T), dtype=np.uint64)
    elif form == "markov":
        p = synth.pi_probs(nl.n_pi, 41, batch=B)
        kw["tau"] = (p * (1 - p) * 0.7).astype(np.float32)
    else:
        kw["stream"] = np.where(np.arange(nl.n_pi) % 4 == 1, 0, np.arange(nl.n_pi)).astype(np.int32)
    ref = _eval(d, nl, B, T, **kw)
    ref.set_schedule(L.DP_SCHED_LEVEL, T)
    want = ref.forward(FIELDS)
    _same(_eval(d, nl, B, T, **kw).forward(FIELDS), want, form)


# NOTs of inputs, constants, results and NOTs; chains that wait two deep and
# deeper; each input count
ODD_CELLS = ("!(!A)", "1^A", "!(0|A)", "A&!B", "!(!A&!B)", "A^(B|!C)", "A&(B|(C^!D))",
             "!(A&B)^(C|D)&E", "A|(B&(C|(D&(E|F))))", "(A^B)&(C^D)|!(E^F)")


@pytest.mark.parametrize("pis,gates,depth,B,T", [(40, 900, 1, 1, 16), (30, 4000, 12, 2, 70),
                                                 (30, 2000, 9, 1, 700)])
def test_tiles_of_library_cells(ctx, pis, gates, depth, B, T):
    say(f"word tiles of library cells: {gates} gates, depth {depth}, B={B}, T={T}")
    ops = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(ODD_CELLS)))
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth, ops=ops, cells=ODD_CELLS), 46)
    d = api.Design(ctx, nl)
    ref = _eval(d, nl, B, T)
    ref.set_schedule(L.DP_SCHED_LEVEL, T)
    want = ref.forward(FIELDS)
    _same(_eval(d, nl, B, T).forward(FIELDS), want, "tiles")
    p, cap = synth.pi_probs(pis, 41, batch=B), synth.net_caps(nl.n_nets, 42)
    for b in range(B):
        f = oracle.Netlist.of(nl).forward(p[b], cap, hybrid=True, n_words=T,
                                          pi_words=oracle.stimulus_model(p[b], 9, T))
        np.testing.assert_array_equal(want["ones"][b].astype(np.uint64), f["ones"])
        np.testing.assert_array_equal(want["toggles"][b].astype(np.uint64), f["toggles"])
        np.testing.assert_allclose(want["sp"][b], f["sp"], atol=SP_ABS, rtol=0)


def _with_chain(nl, levels):
    """The netlist with a chain of inverters from its last gate: designs of few
    levels take level launches."""
    ptr, fan = nl.fanin_ptr, nl.fanin
    gates = [(int(nl.op[g]), fan[ptr[g]:ptr[g + 1]].tolist()) for g in range(nl.n_gates)]
    gates += [(synth.INV, [nl.n_nets - 1 + i]) for i in range(levels)]
    return synth.from_gates(nl.n_pi, gates, cells=nl.cells) if nl.cells else synth.from_gates(nl.n_pi, gates)


@pytest.mark.parametrize("gates,pis,depth,B,T,cells", [
    (5, 3, 5, 1, 2, False), (64, 9, 1, 2, 3, False), (700, 33, 7, 3, 16, False), (700, 33, 7, 25, 7, False),
    (6500, 2100, 3, 1, 33, False), (9000, 50, 1, 1, 250, False), (9000, 50, 1, 1, 2000, False),
    (900, 40, 1, 1, 16, True), (4000, 30, 12, 2, 70, True)])
def test_tiles_of_wide_levels_in_deep_designs(ctx, gates, pis, depth, B, T, cells):
    say(f"word tiles, deep: {gates} gates, {pis} PIs, depth {depth}, B={B}, T={T}, library cells {cells}")
    ops = tuple(range(9)) + (tuple(synth.CELL_BASE + c for c in range(len(ODD_CELLS))) if cells else ())
    nl = _with_chain(synth.random_dag(synth.DagSpec(gates, pis, depth, ops=ops,
                                                    cells=ODD_CELLS if cells else ()), 43), 60)
    d = api.Design(ctx, nl)
    ref = _eval(d, nl, B, T)
    ref.set_schedule(L.DP_SCHED_LEVEL, T)  # a chunk that is set: level launches
    want = ref.forward(FIELDS)
    ev = _eval(d, nl, B, T)
    for _ in range(2):
        _same(ev.forward(FIELDS), want, "tiles")
    p, cap = synth.pi_probs(pis, 41, batch=B), synth.net_caps(nl.n_nets, 42)
    f = oracle.Netlist.of(nl).forward(p[B - 1], cap, hybrid=True, n_words=T,
                                      pi_words=oracle.stimulus_model(p[B - 1], 9, T))
    np.testing.assert_array_equal(want["ones"][B - 1].astype(np.uint64), f["ones"])
    np.testing.assert_array_equal(want["toggles"][B - 1].astype(np.uint64), f["toggles"])

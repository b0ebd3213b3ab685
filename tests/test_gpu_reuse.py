"""The launches whose data are their signals, on buffers that hold an earlier
pass with other inputs: a slot that was not armed again, a stale line, a claim
or a flag left over would show that pass's values.  Each pass against kernels
that keep a barrier or a launch per level, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return api.Context(0)


def _inputs(ev, nl, k):
    ev.set_pi_prob(synth.pi_probs(nl.n_pi, 100 + k, batch=ev.B))
    ev.set_caps(synth.net_caps(nl.n_nets, 200 + k))


def _eval(d, nl, B, mode, k=0, T=40):
    ev = api.Eval(d, B, mode=mode, n_sim=64 * T, seed=5)
    _inputs(ev, nl, k)
    return ev


def _pass(ev, w, mode):
    r = ev.forward(("sp", "power") + (("ones", "toggles", "beta") if mode == L.DP_HYBRID else ()))
    r.update(ev.backward(w, want=("dpi", "dcap")))
    r["lam"], _ = ev.power_gradients()
    return r


def _same(got, want, msg):
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=f"{k}, {msg}")


ORDER = (0, 1, 2, 0, 3, 3, 1)  # inputs of each pass; a repeated one after others, and at once


@pytest.mark.parametrize("gates,pis,depth,B", [(300, 40, 30, 1), (6000, 300, 24, 3), (3000, 130, 12, 40),
                                               (40_000, 900, 6, 2)])
@pytest.mark.parametrize("mode", [L.DP_MODELED, L.DP_HYBRID])
@pytest.mark.parametrize("sched", [L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH])
def test_sweeps_with_new_inputs_each_pass(ctx, gates, pis, depth, B, mode, sched):
    say(f"new inputs each pass: {gates} gates, depth {depth}, B={B}, mode {mode}, schedule {sched}")
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth), 31)
    d = api.Design(ctx, nl)
    weights = [np.random.default_rng(k).uniform(-2, 2, (B, 1)).astype(np.float32) for k in range(4)]
    want = []
    for k in range(4):
        ref = _eval(d, nl, B, mode, k)
        ref.set_schedule(L.DP_SCHED_PERSISTENT)
        want.append(_pass(ref, weights[k], mode))
    ev = _eval(d, nl, B, mode)
    ev.set_schedule(sched)
    for n, k in enumerate(ORDER):
        _inputs(ev, nl, k)
        _same(_pass(ev, weights[k], mode), want[k], f"pass {n}, inputs {k}")


@pytest.mark.parametrize("sched", [L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH])
@pytest.mark.parametrize("gates,B,T", [(900, 1, 21), (900, 3, 130), (4000, 1, 384), (4000, 2, 1000)])
def test_tiles_with_a_new_stimulus_each_pass(ctx, sched, gates, B, T):
    say(f"new stimulus each pass: {gates} gates, B={B}, T={T}, schedule {sched}")
    nl = synth.random_dag(synth.DagSpec(gates, 60, 9), 32)
    d = api.Design(ctx, nl)
    # (an odd one: mostly zeros, so that rows of another pass would stand out)
    stim = [np.random.default_rng(k).integers(0, 2 ** 64, size=(B, nl.n_pi, T), dtype=np.uint64)
            for k in range(3)] + [np.zeros((B, nl.n_pi, T), np.uint64)]
    fields = ("ones", "toggles", "sp", "beta", "power")
    want = []
    for k in range(4):
        ref = _eval(d, nl, B, L.DP_HYBRID, k, T)
        ref.set_stimulus(stim[k])
        ref.set_schedule(L.DP_SCHED_LEVEL, T)  # a chunk that is set: level launches
        want.append(ref.forward(fields))
    ev = _eval(d, nl, B, L.DP_HYBRID, 0, T)
    ev.set_schedule(sched)
    for n, k in enumerate(ORDER):
        _inputs(ev, nl, k)
        ev.set_stimulus(stim[k])
        _same(ev.forward(fields), want[k], f"pass {n}, stimulus {k}")


@pytest.mark.parametrize("graph", [True, False])
def test_groups_with_new_inputs_each_run(ctx, graph):
    say(f"groups, new inputs each run, graph {graph}")
    nls = [synth.random_dag(synth.DagSpec(900 * (k + 1), 30 + k, 7 + 2 * k), 60 + k) for k in range(4)]
    modes = (L.DP_MODELED, L.DP_HYBRID, L.DP_MODELED, L.DP_MODELED)
    ds = [api.Design(ctx, nl) for nl in nls]
    evs = [_eval(d, nl, 3, m) for d, nl, m in zip(ds, nls, modes)]
    want = []
    for k in range(4):
        want.append([])
        for d, nl, m in zip(ds, nls, modes):
            ref = _eval(d, nl, 3, m, k)
            ref.set_schedule(L.DP_SCHED_PERSISTENT)
            r = ref.forward(("sp", "power"))
            r.update(ref.backward(want=("dpi",)))
            want[k].append(r)
    g = api.Group(ctx, evs)
    g.configure(use_graph=graph)
    for n, k in enumerate(ORDER):
        for ev, nl in zip(evs, nls):
            _inputs(ev, nl, k)
        for i, r in enumerate(g.run(("sp", "power"), backward=True)):
            _same(r, want[k][i], f"run {n}, inputs {k}, eval {i}")
    g.close()


def test_several_streams_with_new_inputs_each_pass(ctx):
    """Evals on streams of their own, in flight together, each pass with other
    inputs, outputs read after all of them."""
    import torch
    say("several streams, new inputs each pass")
    nl = synth.random_dag(synth.DagSpec(30_000, 600, 25), 33)
    runs = []
    for i in range(4):
        s = torch.cuda.Stream()
        c = api.Context(0, s.cuda_stream)
        B = 1 + 3 * i
        d = api.Design(c, nl)
        ins = [(torch.from_numpy(synth.pi_probs(nl.n_pi, 100 + 10 * i + k, batch=B)).cuda(),
                torch.from_numpy(synth.net_caps(nl.n_nets, 200 + k)).cuda()) for k in range(4)]
        want = []
        for p, cap in ins:
            ref = api.Eval(d, B)
            ref.set_pi_prob(p)
            ref.set_caps(cap)
            ref.set_schedule(L.DP_SCHED_PERSISTENT)
            r = ref.forward(("sp", "power"))
            r.update(ref.backward(want=("dpi",)))
            want.append(r)
        runs.append((s, c, api.Eval(d, B), ins, want))
    torch.cuda.synchronize()
    outs = []
    for n, k in enumerate(ORDER):
        for i, (s, c, ev, ins, want) in enumerate(runs):
            with torch.cuda.stream(s):
                ev.set_pi_prob(ins[(k + i) % 4][0])
                ev.set_caps(ins[(k + i) % 4][1])
                r = ev.forward(("sp", "power"), device=True)
                r.update(ev.backward(want=("dpi",), device=True))
                outs.append((n, i, r, want[(k + i) % 4]))
    torch.cuda.synchronize()
    for n, i, r, want in outs:
        _same({key: v.cpu().numpy() for key, v in r.items()}, want, f"pass {n}, stream {i}")


@pytest.mark.parametrize("mode,ste", [(L.DP_MODELED, False), (L.DP_HYBRID, False), (L.DP_HYBRID, True)])
def test_library_cells_against_level_launches(ctx, mode, ste):
    """Library cells in the dataflow sweeps against the level launches of more
    columns than those take: a column does not depend on the others."""
    say(f"library cells against level launches: mode {mode}, ste {ste}")
    ops = tuple(range(9)) + tuple(synth.CELL_BASE + c for c in range(len(synth.LIBRARY)))
    nl = synth.random_dag(synth.DagSpec(5000, 100, 15, ops=ops, cells=synth.LIBRARY), 14)
    d = api.Design(ctx, nl)
    p, cap = synth.pi_probs(nl.n_pi, 6, batch=70), synth.net_caps(nl.n_nets, 7)
    fixed = (np.arange(nl.n_pi) % 5 == 0).astype(np.uint8)

    def run(cols):
        ev = api.Eval(d, len(cols), mode=mode, n_sim=64 * 20, seed=5,
                      beta_grad=L.DP_BETA_STE if ste else L.DP_BETA_LOCAL)
        ev.set_pi_prob(p[cols])
        ev.set_caps(cap)
        ev.set_pi_fixed(fixed)
        r = ev.forward(("sp", "power"))
        r.update(ev.backward(want=("dpi",)))
        r["lam"], r["score"] = ev.power_gradients()
        return r
    want = run(list(range(70)))
    for cols in ([0], [3, 69], list(range(5, 69))):
        got = run(cols)
        _same(got, {k: v[cols] for k, v in want.items()}, f"{len(cols)} columns")

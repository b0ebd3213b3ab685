"""The bounded waits of the dataflow sweeps and word tiles, forced from the
host: at a limit of 0 a wait whose first look finds nothing gives up, the
launch's other waits stop at once (every kernel exits normally), the failure
is reported, and the next sweeps are whole again."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu
OFF, ON = 0.0, 1000.0


@pytest.fixture(scope="module")
def ctx():
    return api.Context(0)


def _net(seed=17):
    """Levels of several waves each, narrow and wide in turn: waves wait."""
    return synth.random_dag(synth.DagSpec(6000, 300, 24), seed)


def _eval(d, nl, B=2, mode=L.DP_MODELED, T=40, sched=L.DP_SCHED_AUTO):
    ev = api.Eval(d, B, mode=mode, n_sim=64 * T, seed=5)
    ev.set_pi_prob(synth.pi_probs(nl.n_pi, 6, batch=B))
    ev.set_caps(synth.net_caps(nl.n_nets, 7))
    ev.set_schedule(sched)
    return ev


def _pass(ev):
    r = ev.forward(("sp", "beta", "power"))
    r.update(ev.backward(want=("dpi", "dcap")))
    return r


@pytest.mark.parametrize("sched", [L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH])
@pytest.mark.parametrize("mode", [L.DP_MODELED, L.DP_HYBRID])
def test_give_up_is_reported_once(ctx, sched, mode):
    say(f"give-up: schedule {sched}, mode {mode}")
    nl = _net()
    d = api.Design(ctx, nl)
    want = _pass(_eval(d, nl, mode=mode))
    ev = _eval(d, nl, mode=mode, sched=sched)
    _pass(ev)  # (a captured graph of the default limit)
    ev.set_barrier_timeout(OFF)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.forward(("sp", "power"))
    ev.forward(("power",), device=True)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.synchronize()
    ev.synchronize()  # reported once
    ev.set_barrier_timeout(ON)
    ev.forward(("power",))
    ev.set_barrier_timeout(OFF)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.backward(want=("dpi",))
    ev.set_barrier_timeout(ON)
    got = _pass(ev)
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


@pytest.mark.parametrize("sched", [L.DP_SCHED_LEVEL, L.DP_SCHED_GRAPH])
def test_no_gradient_of_an_earlier_sweep_is_left(ctx, sched):
    """What a reverse sweep that gives up does not reach is NaN, not what its
    output held before: each gradient is NaN or the right one."""
    import torch
    say(f"give-up: gradients, schedule {sched}")
    nl = _net()
    B = 40
    ev = _eval(api.Design(ctx, nl), nl, B, sched=sched)
    ev.forward(("power",))
    want = ev.backward(want=("dpi",))["dpi"]
    out = torch.empty((B, nl.n_pi), dtype=torch.float32, device="cuda")
    for _ in range(3):
        out.fill_(7.0)
        torch.cuda.synchronize()
        ev.set_barrier_timeout(OFF)
        api.check(ev.lib.dp_backward(ev.handle, None, out.data_ptr(), None, None, 1))
        with pytest.raises(L.DiffPowerError, match="gave up"):
            ev.synchronize()
        ev.set_barrier_timeout(ON)
        got = out.cpu().numpy()
        bad = np.isnan(got)
        assert bad.any()
        np.testing.assert_array_equal(got[~bad], want[~bad])
    np.testing.assert_array_equal(ev.backward(want=("dpi",))["dpi"], want)


@pytest.mark.parametrize("cells", [False, True])
def test_reverse_sweep_after_a_forward_that_gave_up(ctx, cells):
    """It has nothing to wait for: NaN go through it as values do."""
    import torch
    say(f"give-up: the reverse sweep after it, library cells {cells}")
    ops = tuple(range(9)) + (tuple(synth.CELL_BASE + c for c in range(9)) if cells else ())
    nl = synth.random_dag(synth.DagSpec(6000, 300, 24, ops=ops, cells=synth.LIBRARY if cells else ()), 18)
    ev = _eval(api.Design(ctx, nl), nl, 3)
    ev.set_barrier_timeout(OFF)
    ev.forward(("power",), device=True)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.synchronize()
    ev.set_barrier_timeout(ON)
    dpi = ev.backward(want=("dpi",), device=True)["dpi"]
    ev.synchronize()  # no wait of this sweep gave up
    assert torch.isnan(dpi).any()


@pytest.mark.parametrize("B,sched", [(1, L.DP_SCHED_LEVEL), (3, L.DP_SCHED_LEVEL), (3, L.DP_SCHED_GRAPH)])
def test_simulation_that_gave_up(ctx, B, sched):
    """Word tiles: no count, rate, beta or power of it can be taken for a result,
    and its inputs are what they were."""
    say(f"give-up: word tiles, B={B}, schedule {sched}")
    nl = _net(19)
    d = api.Design(ctx, nl)
    names = ("sp", "tr", "sp_acc", "tr_acc", "beta", "tr_hyb", "ones", "toggles", "power")
    want = _eval(d, nl, B, L.DP_HYBRID).forward(names)
    ev = _eval(d, nl, B, L.DP_HYBRID, sched=sched)
    ev.set_barrier_timeout(OFF)
    r = ev.forward(names, device=True)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.synchronize()
    r = {k: v.cpu().numpy() for k, v in r.items()}
    pi = np.arange(nl.n_nets) < nl.n_pi
    for k in ("ones", "toggles"):
        assert (r[k].view(np.uint32) == 0xFFFFFFFF).all(), k
    for k in ("sp_acc", "tr_acc", "beta", "tr_hyb", "power"):
        assert np.isnan(r[k]).all(), k
    for k in ("sp", "tr"):
        assert np.isnan(r[k][:, ~pi]).all(), k
        np.testing.assert_array_equal(r[k][:, pi], want[k][:, pi])
    ev.set_barrier_timeout(ON)
    got = ev.forward(names)
    for k in names:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


def test_virus_ascent_that_gave_up(ctx):
    """Its last probabilities are no start for anything: they have to be set
    again."""
    say("give-up: virus ascent")
    nl = _net(20)
    d = api.Design(ctx, nl)
    want = _eval(d, nl).power_virus(5, 1e-3)
    ev = _eval(d, nl)
    ev.set_barrier_timeout(OFF)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        ev.power_virus(5, 1e-3)
    ev.set_barrier_timeout(ON)
    with pytest.raises(L.DiffPowerError, match="probabilities not set"):
        ev.forward(("power",))
    ev.set_pi_prob(synth.pi_probs(nl.n_pi, 6, batch=2))
    for a, b in zip(ev.power_virus(5, 1e-3), want):
        np.testing.assert_array_equal(a, b)


@pytest.fixture(scope="module")
def group_evals(ctx):
    """Two modeled evals (merged sweeps) and two hybrid ones (on branches)."""
    made = []
    for k, mode in enumerate((L.DP_MODELED, L.DP_HYBRID, L.DP_MODELED, L.DP_HYBRID)):
        nl = _net(21 + k)
        d = api.Design(ctx, nl)
        made.append((_eval(d, nl, mode=mode), _pass(_eval(d, nl, mode=mode))))
    return made


def _limits(evs, off):
    for i, ev in enumerate(evs):
        ev.set_barrier_timeout(OFF if i in off else ON)


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("off", [(0, 2), (2,), (1,), (3,), (0, 1, 2, 3)])
def test_group_with_a_sweep_that_gave_up(ctx, group_evals, graph, off):
    """Host outputs: the run fails, whichever eval it was, and nothing is left to
    report.  Device outputs: each eval whose outputs it concerns reports it,
    once: all that share the merged sweeps, or the hybrid one."""
    say(f"give-up: group, graph {graph}, evals {off}")
    evs, want = [e for e, _ in group_evals], [w for _, w in group_evals]
    g = api.Group(ctx, evs)
    g.configure(use_graph=graph)
    _limits(evs, off)
    with pytest.raises(L.DiffPowerError, match="gave up"):
        g.run(("power",), backward=True)
    for ev in evs:
        ev.synchronize()
    g.run(("power",), backward=True, device=True)
    hit = set(off) | ({0, 2} if {0, 2} & set(off) else set())
    for again in (False, True):
        for i, ev in enumerate(evs):
            if i in hit and not again:
                with pytest.raises(L.DiffPowerError, match="gave up"):
                    ev.synchronize()
            else:
                ev.synchronize()
    # a group that is gone when its evals look
    g.run(("power",), device=True)
    g.close()
    g = api.Group(ctx, evs)
    for i, ev in enumerate(evs):
        if i in hit:
            with pytest.raises(L.DiffPowerError, match="gave up"):
                ev.synchronize()
        ev.synchronize()
    _limits(evs, ())
    for r, w in zip(g.run(("sp", "power"), backward=True), want):
        for k in r:
            np.testing.assert_array_equal(r[k], w[k], err_msg=k)
    g.close()

"""Levels of many columns, four a lane (from 400,000 (gate, column) pairs of a
level on): each column bit for bit what it is in a launch of few columns, for
nets of every fan-out, and at column counts that are and are not multiples of
four."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _run(d, nl, p, fixed, **kw):
    ev = api.Eval(d, p.shape[0], n_sim=64 * 5, seed=3, **kw)
    ev.set_pi_prob(p)
    ev.set_caps(synth.net_caps(nl.n_nets, 92))
    ev.set_pi_fixed(fixed)
    r = ev.forward(("sp", "power"))
    r["dpi"] = ev.backward(want=("dpi",))["dpi"]
    r["lam"], _ = ev.power_gradients()
    return r


@pytest.mark.parametrize("gates,pis,depth,B", [(6500, 300, 2, 128), (6500, 300, 2, 126),
                                               (13000, 40, 8, 252), (110_000, 2000, 1, 4)])
@pytest.mark.parametrize("mode,ste", [(L.DP_MODELED, False), (L.DP_HYBRID, True)])
def test_columns_are_independent(gates, pis, depth, B, mode, ste):
    say(f"many columns: {gates} gates, depth {depth}, B={B}, mode {mode}, ste {ste}")
    nl = synth.random_dag(synth.DagSpec(gates, pis, depth, fo_mean=6.0, fo_cap=200), 91)
    d = api.Design(api.Context(0), nl)
    p = synth.pi_probs(pis, 93, batch=B)
    fixed = (np.arange(pis) % 7 == 2).astype(np.uint8)
    kw = dict(mode=mode, beta_grad=L.DP_BETA_STE if ste else L.DP_BETA_LOCAL)
    all_ = _run(d, nl, p, fixed, **kw)
    for b0 in (0, B // 2, B - 3):
        part = _run(d, nl, p[b0:b0 + 3], fixed, **kw)
        for k, v in part.items():
            np.testing.assert_array_equal(all_[k][b0:b0 + 3], v, err_msg=f"{k}, columns {b0}..")

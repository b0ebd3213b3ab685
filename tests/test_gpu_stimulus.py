"""Stimulus words drawn once for several query columns: PI counts bit-exact
against the oracle's words at column counts around the group sizes (1, 2, 4,
8), ragged rows and chunks, shared streams, and probabilities 0 and 1."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,chunk,shared", [
    (1, 2, 0, False), (2, 3, 0, False), (3, 127, 0, True), (4, 128, 0, False), (5, 129, 0, False),
    (7, 300, 64, False), (8, 257, 0, True), (9, 64, 0, False), (17, 131, 6, False),
    (1, 1025, 0, False)])
def test_columns_share_their_draws(B, T, chunk, shared):
    say(f"stimulus: B={B}, T={T}, chunk {chunk}, shared streams {shared}")
    nl = synth.random_dag(synth.DagSpec(400, 37, 6), 31)
    p = synth.pi_probs(nl.n_pi, 32, batch=B)
    p[:, 0], p[:, 1] = 0.0, 1.0  # thresholds 0 and 2^32
    cap = synth.net_caps(nl.n_nets, 33)
    ev = api.Eval(api.Design(api.Context(0), nl), B, mode=L.DP_HYBRID, n_sim=64 * T, seed=2 ** 40 + 7)
    ev.set_pi_prob(p)
    ev.set_caps(cap)
    stream = np.arange(nl.n_pi, dtype=np.int32)
    if shared:
        stream[5] = stream[9] = 3
        ev.set_pi_streams(stream)
    ev.set_schedule(L.DP_SCHED_LEVEL, chunk)
    r = ev.forward(("ones", "toggles"))
    o = oracle.Netlist.of(nl)
    for b in {0, B // 2, B - 1}:
        words = oracle.stimulus_model(p[b], 2 ** 40 + 7, T, stream=stream)
        f = o.forward(p[b], cap, hybrid=True, n_words=T, pi_words=words)
        np.testing.assert_array_equal(r["ones"][b].astype(np.uint64), f["ones"])
        np.testing.assert_array_equal(r["toggles"][b].astype(np.uint64), f["toggles"])

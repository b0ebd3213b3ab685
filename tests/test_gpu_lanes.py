"""Serving steps and design groups in merged launches (staging, power,
gradients out): burst sizes around the power tile (16 columns), odd PI and
gate counts (ragged 16-byte pieces), lanes with and without sizes."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_03778_amd import _lib as L
from paper_2608_03778_amd import api, synth
from tests.gpu_helpers import assert_grad_close, assert_power_close, oracle_column, say

pytestmark = pytest.mark.gpu
SPECS = ((5, 3, 2), (1021, 37, 9), (4099, 130, 14))


@pytest.fixture(scope="module")
def setup():
    ctx = api.Context(0)
    nls = [synth.random_dag(synth.DagSpec(g, p, d), 60 + i) for i, (g, p, d) in enumerate(SPECS)]
    return ctx, nls, [synth.net_caps(nl.n_nets, 70 + i) for i, nl in enumerate(nls)]


@pytest.mark.parametrize("burst", [1, 3, 16, 17, 45])
@pytest.mark.parametrize("sizes", ["all", "some", "none"])
def test_bursts_of_odd_designs(setup, burst, sizes):
    ctx, nls, caps = setup
    say(f"serving burst of {burst}, sizes: {sizes}")
    srv = api.Server(ctx, hbm_budget_bytes=64 << 20, max_batch=32, max_inflight=2)
    ids = [srv.add_design(api.Design(ctx, nl), c, mode=L.DP_MODELED) for nl, c in zip(nls, caps)]
    rng = np.random.default_rng(burst)
    qs = []
    for k in range(burst):
        i = k % len(nls)
        with_size = sizes == "all" or (sizes == "some" and k % 4 < 2)
        qs.append((i, rng.uniform(0.1, 0.9, nls[i].n_pi).astype(np.float32),
                   rng.choice([0.5, 1, 2, 4], nls[i].n_gates).astype(np.float32) if with_size else None,
                   k % 5 != 1))
    alone = [srv.wait(srv.submit(ids[i], p, s, b)) for i, p, s, b in qs]
    tickets = [srv.submit(ids[i], p, s, b) for i, p, s, b in qs]
    orc = [oracle.Netlist.of(nl) for nl in nls]
    for k, t in enumerate(tickets):
        i, p, s, b = qs[k]
        r = srv.wait(t)
        f, adj = oracle_column(orc[i], p, caps[i], np.ones(nls[i].n_gates, np.float32) if s is None else s)
        assert_power_close(r[0], f["power"], f"query {k}")
        assert r[0] == alone[k][0], k
        if b:
            assert_grad_close(r[1], adj["dpi"], f"query {k}")
            np.testing.assert_array_equal(r[1], alone[k][1])
    srv.close()


@pytest.mark.parametrize("cols", [(1, 16, 17), (40, 2, 64)])
@pytest.mark.parametrize("S", [0, 3])
def test_group_power_is_each_evals_own(setup, cols, S):
    ctx, nls, caps = setup
    say(f"group of {cols} columns, {S} size vectors")
    evs, want = [], []
    for nl, cap, B in zip(nls, caps, cols):
        ev = api.Eval(api.Design(ctx, nl), B, S)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 80, batch=B))
        ev.set_caps(cap)
        if S:
            ev.set_cell_sizes(synth.cell_sizes(nl.n_gates, 81, n_size=S))
        want.append(ev.forward(("power",))["power"])
        evs.append(ev)
    group = api.Group(ctx, evs)
    for _ in range(3):
        for r, w in zip(group.run(("power",)), want):
            np.testing.assert_array_equal(r["power"], w)


def test_group_outputs_on_the_device(setup):
    """More outputs than one list of copies holds (17 evals, power and
    gradients), the arrays unaligned and of odd lengths."""
    ctx, nls, caps = setup
    say("group outputs on the device")
    torch = pytest.importorskip("torch")
    ctx = api.Context.for_torch(0)
    evs = []
    for k in range(17):
        nl, cap = nls[k % 3], caps[k % 3]
        ev = api.Eval(api.Design(ctx, nl), 1 + k % 4)
        ev.set_pi_prob(synth.pi_probs(nl.n_pi, 90 + k, batch=1 + k % 4))
        ev.set_caps(cap)
        evs.append(ev)
    group = api.Group(ctx, evs)
    want = group.run(("power",), backward=True)
    got = group.run(("power",), backward=True, device=True)
    torch.cuda.synchronize()
    for k, (r, w) in enumerate(zip(got, want)):
        for f in ("power", "dpi"):
            np.testing.assert_array_equal(r[f].cpu().numpy(), w[f], err_msg=f"eval {k}, {f}")

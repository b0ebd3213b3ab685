"""The library's host code without a GPU: its C++ sources built with g++
against a CPU stand-in for the HIP runtime (tests/hoststub), whose launchers
check every launch's extents and compute nothing.  Covered here: compile and
levelization (levels against the oracle's) for fixed cells, library cells,
trees and flop-cut sequential netlists; every compile and parse error; the
setters' validation and state errors; every schedule's host path (graph
capture bookkeeping, chunks, concurrent simulation streams, the persistent
schedule and its refusal for library cells); the stimulus model's setters;
design groups' merged tables and branches; the serving scheduler's batching,
errors and budget.  Each scenario runs in a process of its own, which loads
only the stand-in runtime."""
from __future__ import annotations

import json
import os
import subprocess
import sys

import pytest

from tests.hoststub import build as stub_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def stub_lib(tmp_path_factory):
    if not stub_build.available():
        pytest.skip("g++ or the HIP headers are missing")
    return stub_build.build(str(tmp_path_factory.mktemp("hoststub")))


def _run(lib, scenario):
    p = subprocess.run([sys.executable, "-m", "tests.hoststub.scenarios", lib, scenario],
                       cwd=ROOT, capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stderr[-4000:]
    return json.loads(p.stdout.strip().splitlines()[-1])


def test_compile_and_levelization(stub_lib):
    r = _run(stub_lib, "compile")
    for name in ("fixed", "library", "flop_cut", "tree"):
        assert r[f"{name}_levels_match"] and r[f"{name}_depth_match"], name
    assert r["expressions_levels_match"]
    assert r["cycle"] == "DP_E_CYCLE"
    for k in ("bad_arity", "bad_op", "bad_net", "cell_arity", "cell_missing"):
        assert r[k] == "DP_E_INVALID", k
    want = {"A&": "operand", "(A|B": "')'", "A $ B": "character", "A B": "after",
            "a&b&c&d&e&f&g": "6 inputs", "&".join(["A"] * 20): "32 operations",
            "A|(B|(C|(D|(E|(F|(A|(B|C)))))))": "8 stack", "1": "no inputs"}
    for text, what in want.items():
        st, msg = r["parse"][text]
        assert st == "DP_E_INVALID" and what in msg, (text, msg)


def test_eval_flows_and_validation(stub_lib):
    r = _run(stub_lib, "flows")
    assert r["fixed_runs"] == 46 and r["library_runs"] == 40
    for name in ("fixed", "library"):
        assert r[f"{name}_backward_first"] == "DP_E_STATE"
        assert r[f"{name}_forward_no_inputs"] == "DP_E_STATE"
        for k in ("p_range", "cap_range", "rates_range", "streams_range", "schedule_bad"):
            assert r[f"{name}_{k}"] == "DP_E_INVALID", (name, k)
        assert r[f"{name}_virus_hybrid"] == "DP_E_UNSUPPORTED"
    assert r["fixed_persistent"] == "OK"
    assert r["library_persistent"] == "DP_E_UNSUPPORTED"


def test_groups_and_serving(stub_lib):
    r = _run(stub_lib, "group_serving")
    assert r["group_results"] == 3
    assert r["served"] == 60 and r["completed"] >= 60 and r["batched"]
    assert r["nan_size"] == "DP_E_INVALID" and r["bad_p"] == "DP_E_INVALID"
    assert r["unknown_ticket"] == "DP_E_NOTFOUND" and r["budget"] == "DP_E_BUDGET"


def test_group_of_persistent_evals(stub_lib):
    r = _run(stub_lib, "group_persistent")
    assert r["results"] == 3 and len(set(r["schedules"])) == 1


def test_groups_of_evals_with_other_scratch(stub_lib):
    assert _run(stub_lib, "group_after_columns") == {"results": 12, "wide": True}


def test_routes_of_groups(stub_lib):
    """Few levels of many pairs go level by level, forward and reverse by
    themselves; a reverse sweep of one column does not."""
    assert _run(stub_lib, "group_routes") == {
        "deep": ["flow", "flow"], "shallow": ["levels", "levels"], "middle": ["levels", "flow"],
        "shallow, one column": ["flow", "flow"], "shallow cells": ["levels", "levels"],
        "deep cells": ["flow", "flow"]}


def test_reverse_graphs_of_deep_designs(stub_lib):
    assert _run(stub_lib, "deep_graphs") == {"1021": 1, "1022": 1, "1023": 1, "1024": 0}


def test_profile_books_a_joint_launch_as_simulation(stub_lib):
    r = _run(stub_lib, "profile")
    assert r["modeled"]["sp_launches"] == 1 and r["modeled"]["sim_launches"] == 0
    for k in ("rides", "rides2"):  # the SP sweep goes out with the tiles
        assert r[k]["sp_launches"] == 0 and r[k]["sp_ms"] == 0 and r[k]["sp_bytes"] == 0, k
        assert r[k]["sim_launches"] == 1
    assert r["apart"]["sp_launches"] == 1 and r["apart"]["sim_launches"] == 1
    # a column of SP bytes went to the simulation's
    sim1, sim2, sim3 = (r[k]["sim_bytes"] for k in ("rides", "rides2", "apart"))
    assert r["modeled"]["sp_bytes"] > 0
    assert sim1 + sim2 > sim3 and sim2 > sim1


def test_reverse_without_memory_for_its_scratch(stub_lib):
    r = _run(stub_lib, "scratch_memory")
    for sched in (1, 2):  # status, a dataflow sweep (a replayed graph makes none)
        assert r[f"{sched} all"] == ["OK", True]
        assert r[f"{sched} less"] == r[f"{sched} again"] == ["OK", False]
        assert r[f"{sched} later"] == ["OK", True]
    assert r["group less"] == ["OK", False, True]  # status, dataflow, level launches
    assert r["group later"] == ["OK", True, False]


def test_simulation_without_memory_for_tiles(stub_lib):
    r = _run(stub_lib, "tile_memory")
    for sched in (1, 2):  # status, tiles, level launches (a replayed graph makes none)
        assert r[f"{sched} all"] == ["OK", True, False]
        assert r[f"{sched} less"] == ["OK", False, True]
        assert r[f"{sched} again"] == ["OK", False, sched == 1]
        assert r[f"{sched} later"] == ["OK", True, False]


def test_autotuner_times_the_same_from_any_schedule(stub_lib):
    r = _run(stub_lib, "autotune")
    assert r["level"][0] > 0 and r["persistent"] == r["level"]


def test_server_step_that_gave_up(stub_lib):
    r = _run(stub_lib, "server_give_up")
    assert r["before"] == ["OK"] * 2 and r["after"] == ["OK"] * 3
    assert r["failed"][0] == "DP_E_HIP" and "gave up" in r["failed"][1]


def test_dataflow_sweeps_where_they_pay(stub_lib):
    """Forward and reverse of shapes measured well on either side of the line."""
    r = _run(stub_lib, "sweep_routes")
    want = {"2000 20 fixed": {1: [True, True], 16: [True, True], 64: [True, True]},
            "20000 2 fixed": {1: [False, True], 16: [False, False], 64: [False, False]},
            "20000 60 fixed": {1: [True, True], 16: [True, True], 64: [True, True]},
            "117000 3 fixed": {1: [False, True], 16: [False, False], 64: [False, False]},
            "117000 60 fixed": {1: [True, True], 16: [True, True], 64: [False, False]},
            "20000 2 cells": {64: [False, False]},
            "20000 60 cells": {1: [True, True], 16: [True, True], 64: [True, True]}}
    for shape, by_columns in want.items():
        for columns, route in by_columns.items():
            assert r[f"{shape} {columns}"] == route, (shape, columns)


def test_word_tiles_where_they_pay(stub_lib):
    r = _run(stub_lib, "tile_routes")
    for shape in ("2000 20", "20000 30", "117000 60"):
        assert all(r[f"{shape} {k}"] for k in ("1x16", "1x1024", "4x96")), shape
    assert not r["117000 3 1x16"] and not r["117000 3 1x1024"] and r["117000 3 4x96"]


def test_reverse_sweep_in_adjoints_where_it_pays(stub_lib):
    r = _run(stub_lib, "wide_routes")
    for name in ("fixed", "far"):
        assert not r[f"{name} below"] and r[f"{name} above"], name
    assert r["cells below"] and r["cells above"] and r["cells small"]
    assert not any(r[f"{name} few sizes"] for name in ("fixed", "far", "cells"))
    assert not r["fixed small"] and not r["far small"]


def test_lane_without_memory_for_its_dataflow_buffers(stub_lib):
    r = _run(stub_lib, "lane_memory")
    assert r["all"][:3] == [True, True, False]   # done, dataflow, merged levels
    assert r["less"][:3] == [True, False, True]
    assert r["later"] == [True, False] and r["lanes"] == 1


def test_contraction_scratch_of_large_faces(stub_lib):
    r = _run(stub_lib, "large_faces")
    for B, S in ((4096, 4096), (2048, 4100)):
        assert r[f"{B}x{S}"] == "OK"
        # the partials of slabs of 2,048 nets, and the evals' control words
        assert r[f"{B}x{S} bytes"] <= 9 * 8 * B * S + (1 << 20)


def test_capture_order_under_the_capture_model(stub_lib):
    """Groups and serving, then the autotuner and graph-captured multi-column
    hybrid sweeps and a captured hybrid design group, in one process, under
    the stand-in's capture model (forks and joins, calls a capturing thread
    may not make, event reuse across captures, graph launches touching only
    live allocations).  Captures record one stream, so nothing forks."""
    r = _run(stub_lib, "capture_order")
    assert r["capture_order_done"] and r["served"] == 60
    assert r["captures"] > 20 and r["graph_launches"] > 100
    assert r["forks"] == 0

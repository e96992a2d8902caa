"""The host side of the library on a stand-in for the HIP runtime (fake_hip.cpp): which launches a call makes, what it
waits for and what it gives back.  No GPU; the library is the one that was built."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so],
                   check=True)

    def run(name, cases):
        """the probe's result for every list of arguments, from one process"""
        out = subprocess.run([sys.executable, os.path.join(HERE, "host_probe.py"), so, name], check=True,
                             input=json.dumps(cases), capture_output=True, text=True)
        return json.loads(out.stdout)
    return run


def fixed(**kw):
    return dict(omega=1.7, theta_target=1e-300, max_sweeps=60, fixed_links=1, bulk_format=3, finish_format=3, **kw)


LINK = dict(omega=1.7, theta_target=1e-300, max_sweeps=60)
# name: (gauge fixings on one handle, theta from one measurement to the next, graphs that are needed)
GRAPH_RUNS = {
    # the partial sums' buffer is first needed by the measurement after the first chunk
    "fixed, separate passes": ([("landau", fixed(separate_measure=1))], 1.0, 1),
    "fixed, FP32-12, separate passes": ([("landau", {**fixed(separate_measure=1), "bulk_format": 2, "finish_format": 2})], 1.0, 1),
    # the finish measures in passes of its own right after the switch
    "fixed, switch at the target": ([("landau", {**fixed(), "bulk_format": 2, "theta_switch": 1e-8, "theta_target": 0.5})], 0.3, 1),
    "fixed, switch": ([("landau", {**fixed(), "bulk_format": 2, "theta_switch": 0.5})], 0.3, 2),
    "fixed, fused and separate": ([("landau", fixed()), ("landau", fixed(separate_measure=1))], 1.0, 2),
    "fixed, separate and fused": ([("landau", fixed(separate_measure=1)), ("landau", fixed())], 1.0, 2),
    "fixed coulomb": ([("coulomb", fixed())], 1.0, 1),
    "link": ([("landau", LINK)], 1.0, 1),
    "link, separate passes": ([("landau", {**LINK, "separate_measure": 1})], 1.0, 1),
    "link, switch": ([("landau", {**LINK, "bulk_format": 2, "finish_format": 3, "theta_switch": 0.5})], 0.3, 2),
    # more graphs than are kept: 60 sweeps in chunks of 14 to 24 with the rests
    "eleven lengths": ([("landau", fixed(check_every=n)) for n in range(14, 25)], 1.0, 22),
}


@pytest.fixture(scope="module")
def graph_logs(probe):
    cases = [((24, 24, 24, 24), 0, calls, factor) for calls, factor, _ in GRAPH_RUNS.values()]
    return dict(zip(GRAPH_RUNS, probe("fix_log", cases)))


@pytest.mark.parametrize("name", GRAPH_RUNS)
def test_graphs_outlive_their_launches(graph_logs, name):
    """A captured graph is destroyed only once the stream has been waited for since its last launch, and the chunks of
    one length replay one graph."""
    log, needed = graph_logs[name], GRAPH_RUNS[name][2]
    launched, made = {}, 0
    for i, words in enumerate(log):
        if words[0] == "graph_new":
            made += 1
        elif words[0] == "graph_launch":
            launched[words[1]] = i
        elif words[0] == "wait":
            launched.clear()
        elif words[0] == "graph_destroy":
            assert words[1] not in launched, f"graph {words[1]} destroyed while it may run: {log[launched[words[1]]:i + 1]}"
    assert 0 < made <= needed


def cube(L, n):
    return [[L, L, L, L]] * n


# configurations, format, tile, what, whether the tiles go in ranges per XCD: both sides of every line of the rule
ENSEMBLE_LISTS = [
    (cube(2, 1), 2, 64, "sweep", True), ([[4, 4, 6, 10], [2, 2, 2, 2], [6, 2, 4, 14]], 2, 64, "sweep", True),
    (cube(8, 5) + [[4, 4, 6, 10]], 0, 128, "measure", True), (cube(8, 3), 3, 256, "fixed", True),
    # link sweeps: 113 and 201 MB; 2^18 sites each
    (cube(8, 48), 0, 128, "sweep", True), (cube(16, 16), 2, 128, "sweep", False),
    ([[16, 16, 32, 30]] * 3, 3, 128, "sweep", False), ([[16, 16, 32, 32]] * 3, 3, 128, "sweep", True),
    # fixed-link sweeps: links and g of 377 and 403 MB; configurations of 160000, 331776 and 1048576 sites
    (cube(14, 20) + cube(8, 4), 3, 128, "fixed", True), (cube(20, 6), 3, 128, "fixed", True),
    (cube(20, 6), 0, 128, "fixed", False), (cube(24, 6), 3, 128, "fixed", False), (cube(32, 2), 3, 128, "fixed", True),
    (cube(32, 2), 0, 128, "fixed", True), (cube(32, 2), 2, 128, "fixed", False),
    # measurement: 302 and 369 MB; 127 and 191 MB each
    (cube(16, 8), 0, 128, "measure", True), (cube(20, 12), 2, 128, "measure", False),
    (cube(24, 4), 3, 128, "measure", False), (cube(24, 4), 0, 128, "measure", True),
]


@pytest.fixture(scope="module")
def ensemble_lists(probe):
    return probe("ensemble_work", [case[:4] for case in ENSEMBLE_LISTS])


@pytest.mark.parametrize("k", range(len(ENSEMBLE_LISTS)))
def test_ensemble_tile_list(ensemble_lists, k):
    """Every tile of every configuration once, consecutive ones on one XCD (workgroup b runs on XCD b % 8) where the rule
    says so, else in the order of dispatch; and no copy of the list on the heap of each call."""
    dims, _, tile, what, ranges = ENSEMBLE_LISTS[k]
    got, sites = ensemble_lists[k], tile // 2 if what == "fixed" else tile
    want = []
    for i, d in enumerate(dims):
        half, first = d[0] * d[1] * d[2] * d[3] // 2, len(want)
        want += [[i, h0, first + h0 // sites] for h0 in range(0, half, sites)]
    in_order = [t for x in range(8) for t in got["tiles"][x::8]] if ranges else got["tiles"]
    assert in_order == want
    assert got["heap"] <= 4096 + 64 * len(dims)


# fields of both formats' sizes between and beyond all lines of the choice (link form: 22, 48, 280, 420 MB and 1.6 GB;
# fixed-link form: 80000, 2^18 and 2 million sites, 400 MB)
LINK_DIMS = [(8, 8, 8, 8), (16, 16, 16, 16), (20, 20, 20, 20), (28, 28, 28, 28), (32, 32, 32, 32), (40, 40, 40, 40),
             (64, 64, 64, 64)]
FIXED_DIMS = [(8, 8, 8, 8), (20, 20, 20, 20), (24, 24, 24, 24), (32, 32, 32, 32), (48, 48, 48, 48)]


TUNING_CASES = [("link", d, f) for d in LINK_DIMS for f in range(4)] + [("fixed", d, f) for d in FIXED_DIMS for f in range(5)]
OTHER = {"link": (4, 256, 0, 1, 0, 2), "fixed": (4, 256, 0, 0)}


@pytest.fixture(scope="module")
def tuning_flows(probe):
    flows = probe("tuning_flows", [(d, f, form, OTHER[form], f"sweep_kernel<{f},_4,") for form, d, f in TUNING_CASES])
    return dict(zip(TUNING_CASES, flows))


@pytest.mark.parametrize("form,dims,fmt", TUNING_CASES)
def test_tunings_come_back_as_they_were_reported(tuning_flows, form, dims, fmt):
    """Setting what was reported changes no launch, on this handle or a new one: before any tuning, after the autotuner
    kept the default (launches chosen by size), after it found something else; and what is reported is within the
    documented values.  A start put back after another tuning is the start again."""
    got = tuning_flows[form, dims, fmt]
    for name in ("got and set", "put back", "tuned, default kept", "tuned, got and set", "kept, set on a new handle"):
        assert got[name] == got["fresh"], name
    assert got["other"][0] == list(OTHER[form]) and got["other"] != got["fresh"]
    assert f"sweep_kernel<{fmt},_4," in got["tuned, another"][1][0][0]
    for name in ("another, got and set", "another, set on a new handle"):
        assert got[name] == got["tuned, another"], name
    for t, _ in got.values():
        lanes, block, order = t[:3]
        assert lanes in (1, 2, 4) and block in (64, 128, 256)
        if form == "link":
            nt, schedule, sites = t[3:]
            assert order in (0, 1) and nt in (0, 1) and schedule in (0, 2) and sites in (1, 2, 4)
            assert nt or schedule != 2
        else:
            assert order in (0, 1, 2, 3) and t[3] in (0, 1)


def test_an_explicit_tuning_is_run_as_set(probe):
    """One lane per site, 128-lane workgroups, streamed, plain order, in place: what new handles once ran, still to be had
    at every size."""
    cases = [(d, f, (1, 128, 0, 1, 0, 1)) for d in LINK_DIMS for f in range(4)]
    for (dims, fmt, _), launch in zip(cases, probe("explicit_launch", cases)):
        half = dims[0] * dims[1] * dims[2] * dims[3] // 2
        for line in launch[:2]:
            assert line[0].startswith(f"sweep_kernel<{fmt},_1,_false,_1,_false"), line
            assert line[1:] == ["grid", str((half + 127) // 128), "1", "block", "128", "order", "0"], line


def test_the_transformation_has_a_lane_per_link_on_small_lattices(probe):
    cases = [((8, 8, 8, 8), 3), ((20, 20, 20, 10), 2), ((20, 20, 20, 12), 2)]
    ends = probe("session_end", cases)
    assert ends == [[["gauge_transform_link_kernel<0,_3,_0>", "grid", "8", "8", "block", "256"]],
                    [["gauge_transform_link_kernel<0,_2,_0>", "grid", "157", "8", "block", "256"]],
                    [["gauge_transform_kernel<0,_2,_0>", "grid", "376", "1", "block", "256"]]]


# dims, format: (what goes past the caches: 0 nothing, 1 all, 2 the stores; lanes of a workgroup; order of the parities)
ANNEAL_LAUNCHES = {
    ((8, 8, 8, 8), 0): (0, 64, "1 1"), ((16, 16, 16, 16), 3): (1, 64, "1 1"), ((24, 24, 24, 24), 0): (0, 64, "1 3"),
    ((40, 40, 40, 40), 0): (2, 64, "1 3"), ((42, 42, 42, 42), 3): (2, 64, "1 3"), ((44, 44, 44, 44), 3): (1, 64, "0 0"),
    ((44, 44, 44, 44), 0): (1, 256, "0 0"), ((48, 48, 48, 48), 3): (1, 128, "0 0"), ((64, 64, 64, 64), 0): (1, 256, "0 0"),
}


def test_annealing_launches_by_size(probe):
    for (dims, fmt), launches in zip(ANNEAL_LAUNCHES, probe("anneal_launches", list(ANNEAL_LAUNCHES))):
        nt, block, orders = ANNEAL_LAUNCHES[dims, fmt]
        assert len(launches) == 2
        for line, order in zip(launches, orders.split()):
            assert line[0].endswith(f"anneal_kernel<{fmt},_{nt},_{block}>"), (dims, fmt, line)
            assert line[4:] == ["block", str(block), "order", order], (dims, fmt, line)


def test_the_measurement_after_a_chunk_is_streamed_where_the_sweeps_are(probe):
    """Fields of 4, 38, 191, 604 MB and 2.4 GB."""
    cases = [((L, L, L, L), 0, [("landau", {**LINK, "max_sweeps": 20})], 1.0) for L in (8, 16, 24, 32, 48)]
    for (dims, *_), log, streamed in zip(cases, probe("fix_log", cases), ("false", "true", "false", "true", "true")):
        last = [line[1] for line in log if line[0] == "launch" and line[1].startswith("measure_kernel")][-1]
        assert last == f"measure_kernel<0,_{streamed}>", dims


def test_in_order_kernels_are_those_that_launches_choose(probe):
    """fixed_sweep_kernel<format, lanes, SR, post, mu0, records, in order, cached links>: two lanes per site in the order of
    one are chosen up to 80000 sites in FP32-12 only, on the cached link field."""
    names, = probe("kernels", [("fixed_sweep_kernel",)])
    in_order = [k for k in names if k.split("<")[1].strip(">").split(",_")[6] == "true"]
    assert len(in_order) == 10 and all(k.startswith("fixed_sweep_kernel<2,_2,") for k in in_order)
    assert all(k.endswith("_false,_true,_true>") for k in in_order)
    used, = probe("tuning_flows", [((8, 8, 8, 8), 2, "fixed", (4, 256, 0, 0), "sweep_kernel<2,_4,")])
    assert used["fresh"][1][0][0] in in_order

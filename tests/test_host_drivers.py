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

    def run(name, *args):
        out = subprocess.run([sys.executable, os.path.join(HERE, "host_probe.py"), so, name, json.dumps(args)],
                             check=True, capture_output=True, text=True)
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


@pytest.mark.parametrize("name", GRAPH_RUNS)
def test_graphs_outlive_their_launches(probe, name):
    """A captured graph is destroyed only once the stream has been waited for since its last launch, and the chunks of
    one length replay one graph."""
    calls, factor, needed = GRAPH_RUNS[name]
    log = probe("fix_log", (24, 24, 24, 24), 0, calls, factor)
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


@pytest.mark.parametrize("dims,tile", [([[2, 2, 2, 2]], 64), ([[4, 4, 6, 10], [2, 2, 2, 2], [6, 2, 4, 14]], 64),
                                       ([[8, 8, 8, 8]] * 5 + [[4, 4, 6, 10]], 128), ([[16, 16, 16, 16]] * 24, 64)])
def test_ensemble_tile_list(probe, dims, tile):
    """Every tile of every configuration once, consecutive ones on one XCD (workgroup b runs on XCD b % 8), and no
    copy of the list on the heap of each call."""
    got = probe("ensemble_work", dims, tile)
    want = []
    for i, d in enumerate(dims):
        half = d[0] * d[1] * d[2] * d[3] // 2
        want += [[i, h0, len(want) + h0 // tile] for h0 in range(0, half, tile)]
    # (len(want) is read before the extension)
    assert [t for x in range(8) for t in got["tiles"][x::8]] == want
    assert got["heap"] <= 4096 + 64 * len(dims)

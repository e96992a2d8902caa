"""The index arithmetic of csrc/lgf_device.hpp itself, compiled for the host (index_probe.cpp): the exact division that
site indices are decoded with, and the places that workgroups take on the lattice."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("probe") / "index_probe.so")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1305_3440_amd", "csrc"),
                    os.path.join(HERE, "index_probe.cpp"), "-o", so], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    lib.probe_items.argtypes = [ctypes.c_void_p] + [ctypes.c_uint32] * 4 + [ctypes.c_uint64]
    lib.probe_items.restype = ctypes.c_uint32
    return lib


def _at(a):
    return ctypes.c_void_p(a.ctypes.data)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 9, 12, 14, 18, 24, 31, 32, 33, 63, 64, 65, 96, 128, 510, 514, 1000,
                               4094, 65534, 65536, 65538, 1 << 20, (1 << 29) - 2, (1 << 30) - 2, 1 << 30, (1 << 31) - 1])
def test_quotients_are_exact(probe, d):
    """n / d for n < 2^31 at the values where a quotient changes."""
    rng = np.random.default_rng(d)
    q = np.concatenate([np.arange(200), rng.integers(0, (1 << 31) // d + 1, 20000), [((1 << 31) - 1) // d]])
    n = (q[:, None] * d + np.array([-1, 0, 1, d - 1])).reshape(-1)
    n = n[(n >= 0) & (n < 1 << 31)].astype(np.uint32)
    got = np.empty_like(n)
    probe.probe_div(_at(n), _at(got), len(n), d)
    assert np.array_equal(got, n // np.uint32(d))


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 64, 1000, 1001, 4096])
@pytest.mark.parametrize("order", [0, 1, 2, 3])
def test_every_workgroup_has_a_place_of_its_own(probe, n, order):
    """order 1: ranges per XCD (the grid a multiple of 8); 2: backwards, on the XCD that has it forwards where the grid
    is a multiple of 8; 3: both."""
    if order & 1:
        n = (n + 7) // 8 * 8
    places = np.empty(n, np.uint32)
    probe.probe_places(_at(places), n, order)
    assert np.array_equal(np.sort(places), np.arange(n))
    forwards = np.empty(n, np.uint32)
    probe.probe_places(_at(forwards), n, order & 1)
    if order & 1:
        for x in range(8):
            assert np.array_equal(forwards[x::8], np.arange(x * (n // 8), (x + 1) * (n // 8)))
    if order & 2 and n % 8 == 0:
        for x in range(8):
            assert np.array_equal(places[x::8], forwards[x::8][::-1])


@pytest.mark.parametrize("n,Lt,hs,site_bytes", [(1, 2, 4, 576), (2, 2, 4, 576), (31, 8, 256, 576), (32, 8, 256, 0),
                                                (16384, 32, 16384, 576), (65536, 64, 131072, 576), (65538, 64, 131072, 576),
                                                (1001, 6, 1 << 20, 576), (9, 64, 1 << 20, 192)])
def test_runs_cover_every_item_once(probe, n, Lt, hs, site_bytes):
    """Every item below n is one workgroup's, and what is left of the grid is at n and beyond; consecutive workgroups of
    an XCD take consecutive items within a run."""
    grid = probe.probe_items(None, 0, n, Lt, hs, site_bytes)
    items = np.empty(grid, np.uint32)
    assert probe.probe_items(_at(items), grid, n, Lt, hs, site_bytes) == grid
    assert np.array_equal(np.sort(items), np.arange(grid)) and grid >= n
    steps = np.diff(items[0::8].astype(np.int64))
    runs = 1 + np.count_nonzero(steps != 1)
    shared = 16 * hs * site_bytes > 200000000  # 8 t-slices of both parities beyond the last-level cache
    assert runs == 1 if not shared else runs <= Lt + 1

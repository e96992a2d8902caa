"""What the host side of liblgf.so does, seen without a GPU: runs the library on the stand-in for the HIP runtime of
fake_hip.cpp and prints the results of a probe, for one list of arguments after the other, as a JSON list.

    python host_probe.py <fake_hip.so> <probe> < <a JSON list of argument lists>

Run in a process of its own (test_host_drivers.py): the stand-in takes the place of the runtime for the whole process.
"""
import ctypes
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


class Fake:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
        self.lib.fake_log.restype = ctypes.c_char_p
        self.lib.fake_kernels.restype = ctypes.c_char_p
        self.lib.fake_result.argtypes = [ctypes.c_double] * 3
        self.lib.fake_memory.argtypes = [ctypes.c_uint64]
        self.lib.fake_fast.argtypes = [ctypes.c_char_p]
        self.lib.fake_new_bytes.restype = ctypes.c_size_t
        self.lib.fake_copied.argtypes = [ctypes.c_size_t]
        self.lib.fake_copied.restype = ctypes.c_void_p

    def lines(self, call):
        """the log of one call, a list of words per line"""
        self.lib.fake_clear()
        call()
        return [line.split() for line in self.lib.fake_log().decode().splitlines()]


def fix_log(fake, lgf, dims, fmt, calls, theta_factor):
    """the log of several gauge fixings on one handle; every measurement finds theta_factor times the last one's theta"""
    with lgf.Lattice(dims, fmt) as lat:
        fake.lib.fake_result(0.5, 1.0, theta_factor)
        def run():
            for gauge, kw in calls:
                (lat.gauge_fix if gauge == "landau" else lat.coulomb_gauge_fix)(**kw)
        return fake.lines(run)


def sweeps_of(fake, lat, form, fmt):
    """the sweep launches of one full sweep on the handle as it is tuned"""
    if form == "link":
        log = fake.lines(lambda: (lat.sweep(2, 1.7), lat.sweep_coulomb(2, 1.7)))
    else:
        lat.fix_begin(fmt)
        log = fake.lines(lambda: lat.fix_chunk(1, 1.7, use_graph=0))
    return [line[1:] for line in log if line[0] == "launch" and "sweep" in line[1]]


def tuning_flows(fake, lgf, dims, fmt, form, other, fast):
    """The sweep launches after several uses of the tuning calls (other: some set tuning, fast: text of the launches
    that the autotuner finds faster), and the tunings that were reported."""
    get, set_, tune = {"link": (lgf.lgf_get_tuning, lgf.lgf_set_tuning, lgf.lgf_autotune),
                       "fixed": (lgf.lgf_get_fixed_tuning, lgf.lgf_set_fixed_tuning, lgf.lgf_autotune_fixed)}[form]
    home = fmt if form == "link" else 0
    out = {}

    def note(name, lat):
        out[name] = [list(get(lat.h, fmt)), sweeps_of(fake, lat, form, fmt)]

    with lgf.Lattice(dims, home) as lat:
        note("fresh", lat)
        start = get(lat.h, fmt)
        set_(lat.h, fmt, *start)
        note("got and set", lat)
        set_(lat.h, fmt, *other)
        note("other", lat)
        set_(lat.h, fmt, *start)
        note("put back", lat)
        tune(lat.h, fmt, 1)
        note("tuned, default kept", lat)
        kept = get(lat.h, fmt)
        set_(lat.h, fmt, *kept)
        note("tuned, got and set", lat)
        fake.lib.fake_fast(fast.encode())
        tune(lat.h, fmt, 1)
        fake.lib.fake_fast(b"")
        note("tuned, another", lat)
        found = get(lat.h, fmt)
        set_(lat.h, fmt, *found)
        note("another, got and set", lat)
    for name, t in (("kept, set on a new handle", kept), ("another, set on a new handle", found)):
        with lgf.Lattice(dims, home) as lat:
            set_(lat.h, fmt, *t)
            note(name, lat)
    return out


def explicit_launch(fake, lgf, dims, fmt, tuning):
    """the sweep launches of a handle with this link-sweep tuning"""
    with lgf.Lattice(dims, fmt) as lat:
        lgf.lgf_set_tuning(lat.h, fmt, *tuning)
        return sweeps_of(fake, lat, "link", fmt)


def session_end(fake, lgf, dims, fmt):
    """the launches of a stepwise session's end"""
    with lgf.Lattice(dims, 0) as lat:
        lat.fix_begin(fmt)
        return [line[1:] for line in fake.lines(lat.fix_end) if line[0] == "launch"]


def anneal_launches(fake, lgf, dims, fmt):
    """the launches of one annealing sweep"""
    with lgf.Lattice(dims, fmt) as lat:
        log = fake.lines(lambda: lat.anneal_sweep(2, 0.5, 1, 2, False))
    return [line[1:] for line in log if line[0] == "launch"]


def kernels(fake, lgf, prefix):
    """the library's kernels whose names start so"""
    return sorted(k for k in fake.lib.fake_kernels().decode().splitlines() if k.startswith(prefix))


def ensemble_work(fake, lgf, dims, fmt, tile, what):
    """the tile list of a sweep, a fixed-link sweep or a measurement of the whole ensemble, and the bytes the call took
    from the C++ heap"""
    ens = lgf.Ensemble(dims, 0 if what == "fixed" else fmt)
    lgf.lgf_ensemble_set_tuning(ens.e, tile, 1, 1)
    sites = tile // 2 if what == "fixed" else tile
    n = sum((v // 2 + sites - 1) // sites for v in ens.V)
    fake.lib.fake_new_bytes()
    if what == "sweep":
        ens.sweep(2, 1.7)
    elif what == "measure":
        ens.measure()
    else:
        lgf.lgf_ensemble_time_fixed_sweeps(ens.e, fmt, 1, 1.7)
    heap = fake.lib.fake_new_bytes()
    tiles = (ctypes.c_uint32 * (4 * n)).from_address(fake.lib.fake_copied(16 * n))
    return {"tiles": [tiles[4 * k:4 * k + 3] for k in range(n)], "heap": heap}


def main():
    fake = Fake(sys.argv[1])
    import paper_1305_3440_amd as lgf
    lgf.load_library()
    print(json.dumps([globals()[sys.argv[2]](fake, lgf, *args) for args in json.load(sys.stdin)]))


if __name__ == "__main__":
    main()

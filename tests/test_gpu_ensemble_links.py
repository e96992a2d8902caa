"""Where the fixed-link sweeps of an ensemble read their links: the link fields through the caches up to 400 MB of links
and g, per-site records beyond.  Both give the bits of the single lattice, ragged tiles and XCD ranges included."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lgf():
    if not gpu_available():
        pytest.skip("no GPU visible")
    import paper_1305_3440_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("fmt", [2, 3, 4])
@pytest.mark.parametrize("p_sr", [0.0, 0.4])
@pytest.mark.parametrize("dims", [[(2, 2, 2, 2)], [(6, 4, 10, 14), (14, 10, 6, 18), (2, 2, 2, 2), (4, 4, 6, 10)],
                                  [(4, 4, 6, 10), (32, 30, 32, 30)]], ids=["one", "cached", "records"])
def test_ensemble_links_equal_single(lgf, dims, p_sr, fmt):
    print(f"[gpu-case] ensemble links {dims} {p_sr} {fmt}", flush=True)
    kw = dict(omega=1.7, p_sr=p_sr, seed=4, theta_target=1e-300, max_sweeps=4, check_every=2, fixed_links=1,
              bulk_format=fmt, finish_format=fmt)
    with lgf.Ensemble(dims, lgf.LGF_FP64_18) as ens:
        for i in range(len(dims)):
            ens.generate(i, 30 + i, 0.3)
        ens.gauge_fix(**kw)
        got = [ens.store(i) for i in range(len(dims))]
    for i, d in enumerate(dims):
        if p_sr and i:
            continue  # the coins of configuration i > 0 have their own counters
        with lgf.Lattice(d, lgf.LGF_FP64_18) as lat:
            lgf.lgf_set_fixed_tuning(lat.h, fmt, 2, 128, 0, 0)
            lat.generate(30 + i, 0.3)
            lat.gauge_fix(**kw)
            ref = lat.store()
        assert np.array_equal(ref, got[i]), (i, d)

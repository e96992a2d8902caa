"""Untuned launches choose lanes, workgroup, tile order and caching by the size of the lattice; the choice never
changes a bit.  Each rule's two sides, with the remainders of a tile, against the explicit tuning of one lane per site
(link form, FP32-12 fixed-link form) or two (FP64 fixed-link form)."""
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


# volumes on both sides of 40000 and 65536 sites, fields of 20, 24, 47, 49 MB (FP64-18 or FP64-12), around 380 and
# beyond 420 MB
LINK_CASES = [((2, 2, 2, 2), 0), ((4, 4, 6, 10), 1), ((4, 4, 6, 10), 2), ((6, 2, 4, 14), 3), ((14, 14, 14, 14), 0),
              ((14, 14, 14, 16), 0), ((16, 16, 16, 16), 2), ((16, 16, 18, 16), 2), ((18, 16, 20, 14), 0),
              ((18, 16, 20, 16), 0), ((22, 24, 22, 10), 3), ((28, 28, 28, 30), 3), ((28, 28, 28, 32), 0),
              ((34, 32, 32, 32), 2), ((34, 34, 34, 34), 1), ((34, 38, 34, 30), 1), ((34, 32, 38, 34), 3)]


@pytest.mark.parametrize("dims,fmt", LINK_CASES)
def test_link_sweeps_do_not_depend_on_the_choice(lgf, dims, fmt):
    import torch
    print(f"[gpu-case] choice link {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for tuned in (False, True):
        buf = torch.empty(V * 4 * lgf.lgf.LINK_BYTES[fmt] // 4, dtype=torch.float32, device="cuda")
        with lgf.Lattice(dims, fmt, device_buf=buf) as lat:
            if tuned:
                lgf.lgf_set_tuning(lat.h, fmt, 1, 128, 0, 1, 0, 1)
            lat.generate(5, 0.3)
            lat.sweep(0, 1.7)
            lat.sweep(1, 1.7, 0.5, 9, 3)
            lat.sweep(2, 1.6)
            lat.sweep_coulomb(2, 1.5, slice_active=[t % 3 != 1 for t in range(dims[0])])
            st, res, _ = lat.gauge_fix(omega=1.7, theta_target=1e-300, max_sweeps=3, check_every=2)
            lgf.lgf_synchronize(lat.h)
            out.append((buf.clone().view(torch.int32), res["F"], res["theta"]))
    assert torch.equal(out[0][0], out[1][0])
    assert abs(out[0][1] - out[1][1]) <= 1e-14 and abs(out[0][2] - out[1][2]) <= 1e-12 * out[1][2]


FIXED_CASES = [(dims, fmt) for dims in ((2, 2, 2, 2), (4, 4, 6, 10), (6, 2, 4, 14), (14, 14, 18, 22), (14, 14, 18, 24))
               for fmt in (2, 3, 4)] + [((4, 4, 6, 10), 0), ((4, 4, 6, 10), 1), ((16, 16, 32, 34), 3), ((28, 30, 32, 30), 4),
                                                           ((32, 30, 32, 34), 3), ((24, 24, 26, 28), 1)]


@pytest.mark.parametrize("gauge", ["landau", "coulomb"])
@pytest.mark.parametrize("dims,fmt", FIXED_CASES)
def test_fixed_sweeps_do_not_depend_on_the_choice(lgf, dims, fmt, gauge):
    import torch
    print(f"[gpu-case] choice fixed {gauge} {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for tuned in (False, True):
        buf = torch.empty(V * 4 * 18, dtype=torch.float64, device="cuda")
        with lgf.Lattice(dims, lgf.LGF_FP64_18, device_buf=buf) as lat:
            if tuned:
                lanes, _, _, layout = lgf.lgf_get_fixed_tuning(lat.h, fmt)
                lgf.lgf_set_fixed_tuning(lat.h, fmt, lanes, 128, 0, layout)
            lat.generate(6, 0.3)
            for p_sr in (0.0, 0.4):
                fix = lat.gauge_fix if gauge == "landau" else lat.coulomb_gauge_fix
                fix(omega=1.7, p_sr=p_sr, seed=4, theta_target=1e-300, max_sweeps=3, check_every=2, fixed_links=1,
                    bulk_format=fmt, finish_format=fmt)
            lgf.lgf_synchronize(lat.h)
            out.append(buf.clone().view(torch.int64))
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("scale", [1e-148, 1e-143, 1.0, 1e143, 1e148])
def test_normalisation_over_the_whole_range(lgf, scale):
    """|a|^2 of a subgroup block below 2^-960, beyond 2^960 and just inside: the update depends on K's direction only,
    so a sweep of scaled links is the scaled sweep of the links (the scales are rounded to powers of two: exactly)."""
    import oracle
    print(f"[gpu-case] scaled links {scale}", flush=True)
    dims = (4, 4, 6, 10)
    two = 2.0 ** round(np.log2(scale))
    U = oracle.generate_links(dims, 3, 0.3, True)
    got = []
    for s in (1.0, two):
        with lgf.Lattice(dims, lgf.LGF_FP64_18) as lat:
            lat.load(U * s)
            lat.sweep(2, 1.7)
            got.append(lat.store() / s)
    # one more rounding of 1 / |a| on either side of the estimate's range, amplified up to 40 times on
    # ill-conditioned sites, over two half-sweeps: 2 * 3 * 40 * 2^-52
    assert np.abs(got[1] - got[0]).max() <= 240 * 2.0 ** -52


@pytest.mark.parametrize("dims,fmt", [((2, 2, 2, 2), 0), ((4, 4, 6, 10), 3), ((16, 16, 16, 14), 0), ((22, 14, 14, 18), 3),
                                      ((34, 32, 30, 30), 0)])
def test_annealing_does_not_depend_on_the_choice(lgf, dims, fmt):
    """Untuned annealing launches (cached, streamed, stores streamed; XCD ranges; odd half-sweeps from the end) against
    streamed launches in the plain order: the same links and trials."""
    import torch
    print(f"[gpu-case] choice anneal {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for tuned in (False, True):
        buf = torch.empty(V * 4 * lgf.lgf.LINK_BYTES[fmt] // 4, dtype=torch.float32, device="cuda")
        with lgf.Lattice(dims, fmt, device_buf=buf) as lat:
            if tuned:
                lgf.lgf_set_tuning(lat.h, fmt, 1, 128, 0, 1, 0, 1)
            lat.generate(5, 0.3)
            trials = [lat.anneal_sweep(2, T, 8, 3) for T in (0.05, 3.0)]
            lgf.lgf_synchronize(lat.h)
            out.append((buf.clone().view(torch.int32), trials))
    assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1]

"""The sides of the launch choice that small lattices do not reach: link fields beyond 1.6 GB, fixed-link sweeps on more than
400 MB of links and g in each format, and more than 2 million sites.  The choice changes no bit."""
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


# 1.70 GB FP64-18, 1.66 GB FP32-18, 1.63 GB FP32-12, 1.64 GB FP64-12 (out of place)
@pytest.mark.parametrize("dims,fmt", [((40, 42, 42, 42), 0), ((48, 48, 50, 50), 1), ((54, 54, 54, 54), 2), ((44, 46, 46, 46), 3)])
def test_link_sweeps_of_large_fields(lgf, dims, fmt):
    import torch
    print(f"[gpu-case] large choice link {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for tune in (None, (1, 64, 0, 1, 0, 1)):
        buf = torch.empty(V * lgf.lgf.LINK_BYTES[fmt], dtype=torch.int32, device="cuda")
        with lgf.Lattice(dims, fmt, device_buf=buf) as lat:
            if tune:
                lgf.lgf_set_tuning(lat.h, fmt, *tune)
            lat.generate(5, 0.3)
            lat.sweep(2, 1.7, 0.5, 9, 3)
            lat.sweep_coulomb(2, 1.5, slice_active=[t % 3 != 1 for t in range(dims[0])])
            st, res, _ = lat.gauge_fix(omega=1.7, theta_target=1e-300, max_sweeps=3, check_every=2)
            lgf.lgf_synchronize(lat.h)
            out.append((buf, res["F"], res["theta"]))
    assert torch.equal(out[0][0], out[1][0])
    assert abs(out[0][1] - out[1][1]) <= 1e-14 and abs(out[0][2] - out[1][2]) <= 1e-12 * out[1][2]


# 440 MB FP64-18 and 403 MB FP32-12 (records) of links and g, then 2.09 million sites, each against the link field in
# workgroups of another size and the plain order
@pytest.mark.parametrize("gauge", ["landau", "coulomb"])
@pytest.mark.parametrize("dims,fmt,tune", [((26, 28, 28, 30), 0, (2, 128, 0, 0)), ((36, 36, 36, 36), 2, (1, 64, 0, 0)),
                                           ((38, 38, 38, 38), 0, (2, 128, 0, 0)), ((38, 38, 38, 38), 1, (2, 64, 0, 0)),
                                           ((38, 38, 38, 38), 2, (1, 64, 0, 0)), ((38, 38, 38, 38), 3, (2, 256, 0, 0)),
                                           ((38, 38, 38, 38), 4, (2, 256, 0, 0))])
def test_fixed_sweeps_of_large_lattices(lgf, dims, fmt, tune, gauge):
    import torch
    print(f"[gpu-case] large choice fixed {gauge} {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for t in (None, tune):
        buf = torch.empty(V * 144, dtype=torch.int32, device="cuda")
        with lgf.Lattice(dims, lgf.LGF_FP64_18, device_buf=buf) as lat:
            if t:
                lgf.lgf_set_fixed_tuning(lat.h, fmt, *t)
            lat.generate(6, 0.3)
            for p_sr in (0.0, 0.4):
                fix = lat.gauge_fix if gauge == "landau" else lat.coulomb_gauge_fix
                fix(omega=1.7, p_sr=p_sr, seed=4, theta_target=1e-300, max_sweeps=3, check_every=2, fixed_links=1,
                    bulk_format=fmt, finish_format=fmt)
            lgf.lgf_synchronize(lat.h)
            out.append(buf)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("dims", [(4, 4, 6, 10), (14, 14, 18, 22)])
def test_two_lanes_in_order_against_one_lane(lgf, dims):
    """FP32-12 up to 80000 sites in the fixed-link form: two lanes per site on the cached field, untuned, against one lane
    per site in another workgroup size."""
    import torch
    print(f"[gpu-case] in order {dims}", flush=True)
    out = []
    for t in (None, (1, 64, 0, 0)):
        buf = torch.empty(int(np.prod(dims)) * 144, dtype=torch.int32, device="cuda")
        with lgf.Lattice(dims, lgf.LGF_FP64_18, device_buf=buf) as lat:
            if t:
                lgf.lgf_set_fixed_tuning(lat.h, lgf.LGF_FP32_12, *t)
            lat.generate(6, 0.3)
            for p_sr in (0.0, 0.4):
                st, res, _ = lat.gauge_fix(omega=1.7, p_sr=p_sr, seed=4, theta_target=1e-300, max_sweeps=3, check_every=2,
                                           fixed_links=1, bulk_format=lgf.LGF_FP32_12, finish_format=lgf.LGF_FP32_12)
            lgf.lgf_synchronize(lat.h)
            out.append(buf)
    assert torch.equal(out[0], out[1])

"""Annealing launches of every workgroup size, streamed, give the links and trials of the untuned launch."""
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


# 16 and 480 sites, and 4032: whole and partial workgroups of 64, 128 and 256 lanes
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 10), (6, 8, 6, 14)])
@pytest.mark.parametrize("fmt", [0, 3])
def test_workgroup_size_changes_no_bit(lgf, dims, fmt):
    import torch
    print(f"[gpu-case] anneal workgroups {dims} {fmt}", flush=True)
    V = int(np.prod(dims))
    out = []
    for tune in (None, (1, 64, 0, 1, 0, 1), (1, 128, 0, 1, 0, 1), (1, 256, 0, 1, 0, 1), (1, 256, 1, 1, 0, 1)):
        buf = torch.empty(V * 4 * lgf.lgf.LINK_BYTES[fmt] // 4, dtype=torch.float32, device="cuda")
        with lgf.Lattice(dims, fmt, device_buf=buf) as lat:
            if tune:
                lgf.lgf_set_tuning(lat.h, fmt, *tune)
            lat.generate(7, 0.3)
            trials = [lat.anneal_sweep(2, T, 8, 3) for T in (0.05, 3.0)]
            lgf.lgf_synchronize(lat.h)
            out.append((buf.clone().view(torch.int32), trials))
    for links, trials in out[1:]:
        assert torch.equal(links, out[0][0]) and trials == out[0][1]

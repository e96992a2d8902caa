"""One launch measures both parities: F, theta and the plaquette against the oracle where the tiles of 256 sites per
parity end (a part of one, exactly one, one and a part, and more than eight XCD ranges)."""
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


@pytest.mark.parametrize("fmt", [0, 1, 2, 3])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 8), (2, 2, 10, 14), (6, 14, 10, 4), (4, 12, 18, 10)])
def test_observables_match_the_oracle(lgf, dims, fmt):
    import oracle as orc
    print(f"[gpu-case] observables {dims} {fmt}", flush=True)
    with lgf.Lattice(dims, fmt) as lat:
        lat.load(orc.generate_links(dims, 21, 0.4))
        U = lat.store()
        F, th = lat.measure()
        P = lat.plaquette()
    F_ref, th_ref = orc.measure(dims, U)
    # sums of O(1) terms in FP64; FP32 links come back as they are, up to the rounding of a rebuilt row 2
    tol = 2e-7 if fmt == 2 else 1e-14
    assert abs(F - F_ref) < tol and abs(th - th_ref) < 10 * tol * max(1.0, th_ref)
    assert abs(P - orc.plaquette(dims, U)) < tol

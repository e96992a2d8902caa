"""The final gauge transformation takes one lane per link on small lattices and one per site on larger ones."""
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


@pytest.mark.parametrize("home", [0, 3])
@pytest.mark.parametrize("fmt", [0, 1, 2, 3])
def test_transformation_does_not_depend_on_the_size(lgf, orc, home, fmt):
    """77616 sites (one lane per link, a partial last workgroup) against the same links twice over in t (155232 sites, one
    lane per site): two fixed-link sweeps and the transformation give each half the links of the small lattice."""
    print(f"[gpu-case] transform sizes home {home} g {fmt}", flush=True)
    dims = (14, 14, 18, 22)
    U = orc.generate_links(dims, 12, 0.3, True)
    got = []
    for n in (1, 2):
        with lgf.Lattice((n * dims[0],) + dims[1:], home) as lat:
            lat.load(np.concatenate([U] * n))
            lat.fix_begin(fmt)
            lat.fix_chunk(2, 1.7)
            lat.fix_end()
            got.append(lat.store())
    V = len(U)
    assert not np.array_equal(got[0], U)
    assert np.array_equal(got[1][:V], got[0]) and np.array_equal(got[1][V:], got[0])

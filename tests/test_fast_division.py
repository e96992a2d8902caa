"""The exact division by fixed extents that the kernels decode site indices with (csrc/lgf_device.hpp, FastDiv):
n / d = floor(2n m / 2^32) >> l for every n < 2^31, checked at the values where a quotient changes."""
import numpy as np
import pytest


def fast_div(n, d):
    l = 0
    while (1 << l) < d:
        l += 1
    m = (1 << (31 + l)) // d + 1
    assert m < 1 << 32
    return ((2 * n * np.uint64(m)) >> np.uint64(32)) >> np.uint64(l)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 9, 12, 14, 18, 24, 31, 32, 33, 63, 64, 65, 96, 128, 510, 514, 1000,
                               4094, 65534, 65536, 65538, 1 << 20, (1 << 29) - 2, (1 << 30) - 2, 1 << 30])
def test_quotients_are_exact(d):
    rng = np.random.default_rng(d)
    q = np.concatenate([np.arange(200), rng.integers(0, (1 << 31) // d + 1, 20000), [((1 << 31) - 1) // d]])
    n = (q[:, None] * d + np.array([-1, 0, 1, d - 1])).reshape(-1)
    n = n[(n >= 0) & (n < 1 << 31)].astype(np.uint64)
    assert np.array_equal(fast_div(n, d), n // np.uint64(d))

"""The con2prim bracket starts above zero exactly where sqrt(s2) - E is
positive in IEEE arithmetic: the pass takes that root only where s2 is not well
below E^2, and must not miss a case (values next to the boundary, extreme
scales, zeros, infinities, NaN)."""
import numpy as np


def test_root_skipped_only_below_the_energy():
    rng = np.random.default_rng(5)
    E = np.concatenate([10.0 ** rng.uniform(-300, 300, 20000), rng.uniform(0.5, 2, 20000)])
    ulps = rng.integers(-120, 121, E.size)
    with np.errstate(all="ignore"):
        s2 = E * E * (1.0 + ulps * 2.0**-53)
        special = np.array([0.0, -0.0, 5e-324, 1e-160, 1.0, -1.0, 1e154, 1e200, np.inf, -np.inf, np.nan])
        a, b = np.meshgrid(special, special)
        E, s2 = np.concatenate([E, a.ravel()]), np.concatenate([s2, b.ravel()])
        lo = np.sqrt(s2) - E
        full = np.where(lo > 0, lo, 0.0)
        takes = ~(E > 0) | (s2 >= E * E * (1.0 - 1e-14))
        np.testing.assert_array_equal(np.where(takes, full, 0.0), full)
    assert np.any(~takes) and np.any(full > 0)

"""Windows scale with the couplings, through powers of two that every step of
the recurrence and of the tridiagonal's root search carries exactly, down to
the documented width of 1e-8 that is padded."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [-10, 40, 200])
def test_windows_of_scaled_couplings(kpm, power):
    rng = np.random.default_rng(3)
    J = rng.uniform(0.5, 1.5, 12)

    def windows(scale):
        secs = []
        for n in (10, 12):
            c = W.ring(n)
            c = W.Cluster(n, c.bond_i, c.bond_j, J[:n] * scale)
            secs += [W.Sector(c, k, 0) for k in range(n // 2, n - 2)]
        return np.concatenate([kpm.spectral_bounds(secs, 30, 0.01, seed) for seed in range(20)])

    one = windows(1.0)
    assert (one[:, 1] > one[:, 0]).all()
    # 30 steps in sectors of at least 45 states: no step ends early, so the
    # scaled recurrence is the same bits times the power of two
    assert np.array_equal(windows(2.0**power), one * 2.0**power)

"""Windows of an 18-site sawtooth chain that don't hang on rounding.  The order
of summation moves an end of the window by about c omega^2 widths, c what the
extreme Ritz value moved over the last two steps and omega the orthogonality
that the Lanczos vectors have lost; here both are read off the oracle's own
recursion, omega from its vectors themselves.  Where c omega^2 is under 3e-15
the windows agree to rounding: 50 steps of sums of at most 48620 terms keep
1e-9 with room."""
import numpy as np
import pytest
import scipy.linalg as sla

import workloads as W
from oracle import ftlm, hamiltonian, moments, rng

pytestmark = pytest.mark.gpu


def settled(s, seed):
    H = hamiltonian.sector_hamiltonian(s.cluster, s.n_up)
    v0, _ = rng.box_muller(seed, s.cluster_id, s.n_up, rng.LANCZOS_STREAM, H.shape[0])
    a, b = ftlm.lanczos_coefficients(H, v0, 50)
    if a.size < 50:
        return False, H
    q = [np.zeros_like(v0), v0 / np.linalg.norm(v0)]
    for j in range(49):
        q.append((H @ q[-1] - a[j] * q[-1] - (b[j - 1] * q[-2] if j else 0.0)) / b[j])
    q = np.array(q[1:])
    omega = np.abs(q @ q.T - np.eye(50)).max()
    e = sla.eigh_tridiagonal(a, b, eigvals_only=True)
    e2 = sla.eigh_tridiagonal(a[:-2], b[:-2], eigvals_only=True)
    c = max(abs(e[0] - e2[0]), abs(e[-1] - e2[-1])) / (e[-1] - e[0])
    return c < 1e-13 or c * omega**2 < 3e-15, H


@pytest.mark.parametrize("seed", [3, 4])
def test_settled_windows_to_rounding(kpm, seed):
    secs = W.sectors(W.sawtooth(18))
    got = kpm.spectral_bounds(secs, 50, 0.01, seed)
    n = 0
    for p, s in enumerate(secs):
        yes, H = settled(s, seed)
        if yes:
            n += 1
            want = np.array(moments.spectral_bounds(s, 50, 0.01, seed, H=H))
            assert np.abs(got[p] - want).max() <= 1e-9, (s.dim, got[p], want)
    assert n >= 1

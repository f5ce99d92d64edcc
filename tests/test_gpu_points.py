"""The two-kernel thermodynamics at the edges of its splits: more sectors than
the 16 lanes of a point, a remainder of problems per cosine, odd and even node
counts, one point, a remainder of points, and more points than one chunk, with
temperatures that repeat in no order.

The Boltzmann sums have positive terms (Jackson weights), so both sides carry
the rounding of their exponents, at most beta (E_max - E_min) of 200 here times
2^-53 = 2e-14, and of the weights, 1e-14 of their largest; 1e-12 leaves room
for the C and chi of points where one level dominates."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import moments, thermo

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pts, Nt", [(1, 64), (17, 97), (16384 + 83, 64)])
def test_points_of_a_map(kpm, n_pts, Nt):
    rng = np.random.default_rng(n_pts)
    secs = W.sectors(W.ring(34)) + W.sectors(W.ring(9), cluster_id=1)
    assert len(secs) == 18 + 5
    M = 64
    mus = np.array([moments.exact_moments(np.sort(rng.uniform(-0.97, 0.97, 40)), M) for _ in secs])
    ab = np.array([(rng.uniform(2.0, 6.0), rng.uniform(-3.0, 1.0)) for _ in secs])
    T = rng.choice(W.log_temperatures(29, 0.1, 10.0), n_pts)
    h = rng.choice([0.0, 0.3, -0.8, 1.1], n_pts)
    out = kpm.thermo_field(torch.tensor(mus, device="cuda"), torch.tensor(ab, device="cuda"), secs, T, h,
                           "jackson", Nt)
    at = np.unique(np.concatenate([np.arange(min(n_pts, 20)), rng.integers(0, n_pts, 20),
                                   [n_pts - 1], np.arange(16380, 16390)]))
    at = at[at < n_pts]
    probs = [dict(cluster=s.cluster_id, n_sites=s.cluster.n_sites, n_up=s.n_up) for s in secs]
    ref = thermo.thermo_field(probs, mus, ab, T[at], h[at], "jackson", Nt)
    for q in ("lnZ", "E", "C", "chi", "M"):
        got = out[q].cpu().numpy()
        assert np.isfinite(got).all(), q
        scale = np.abs(ref[q]).max(axis=1, keepdims=True)
        assert (np.abs(got[:, at] - ref[q]) <= 1e-12 * np.maximum(scale, 1.0)).all(), q
    assert not out["z_nonpos"].any()

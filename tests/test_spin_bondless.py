"""Spin-s problems without bonds (H = 0): on the list kernel, since the records
of the split spin kernel are walked bond by bond."""
import ctypes

import numpy as np
import pytest

import workloads as W
from paper_2104_13218_amd import kpm as K


def _free(n, two_s):
    return W.spin_sectors(W.Cluster(n, [], [], []), two_s)


def _ring(n, two_s, cluster_id):
    return W.spin_sectors(W.Cluster(n, range(n), [(i + 1) % n for i in range(n)], np.ones(n)), two_s, cluster_id)


def _size(secs, R):
    ps = K.ProblemSet(secs, [(-1.0, 1.0)] * len(secs))
    return K.moments_workspace_size(ps, K.make_params(16, R, "rademacher", "fp64"))


@pytest.mark.parametrize("secs", [_free(8, 2)[:1], _free(9, 3)[:2], _ring(6, 3, 0) + _free(8, 2)],
                         ids=["8 sites of spin 1", "9 of spin 3/2", "with a ring"])
def test_bondless_problems_take_the_lists(monkeypatch, secs):
    """The plan, read off the workspace's size, is that of the list kernel."""
    monkeypatch.delenv("KPM_SPIN_SPLIT", raising=False)
    got = _size(secs, 8)
    monkeypatch.setenv("KPM_SPIN_SPLIT", "0")
    assert got == _size(secs, 8) > 0
    monkeypatch.setenv("KPM_SPIN_SPLIT", "1")
    assert got == _size(secs, 8)


@pytest.mark.gpu
@pytest.mark.parametrize("R", [1, 4, 8])
def test_moments_without_bonds(kpm, R):
    """H' = -b/a times the identity: mu_n = dim T_n(-b/a); M steps each pass on
    the rounding of those before, M^2 2^-52 in all."""
    lo, hi, M = -0.7, 1.3, 24
    secs = _free(8, 2)[:2]
    mu, ab = kpm.chebyshev_moments(secs, M, R, "rademacher", "fp64", 0.025, 3, bounds=[(lo, hi)] * len(secs))
    a, b = ab.cpu().numpy()[0]
    want = np.cos(np.arange(M) * np.arccos(-b / a))
    dims = np.array([[s.dim] for s in secs], dtype=float)
    assert np.abs(mu.cpu().numpy() / dims - want).max() <= M * M * 2.0 ** -52

"""The slice kernel as the default of sectors from 2^15 states on: its launch
shape by size and storage, the fall-back to 9 low bits, column blocks placed
on one XCD each, and the bounds run on it, against the oracle.

Tolerances relative to mu_0: float64 1e-10, float32 storage 1e-5 (as in
test_gpu_moments)."""
import numpy as np
import pytest

import workloads as W
from oracle import hamiltonian, moments

pytestmark = pytest.mark.gpu


def _mixed_graph(n, n_bonds, seed):
    rng = np.random.default_rng([seed, n, n_bonds])
    bi = rng.integers(0, n, n_bonds)
    bj = (bi + rng.integers(1, n, n_bonds)) % n
    return W.Cluster(n, bi, bj, rng.uniform(0.5, 1.5, n_bonds))


def _check(kpm, secs, M, R, kind, precision, seed, **kw):
    mu, ab = kpm.chebyshev_moments(secs, M, R, kind, precision, 0.025, seed, **kw)
    st = kpm.last_run_stats()
    mu, ab = mu.cpu().numpy(), ab.cpu().numpy()
    tol = 1e-10 if precision == "fp64" else 1e-5
    for p, s in enumerate(secs):
        H = hamiltonian.sector_hamiltonian(s.cluster, s.n_up)
        lo, hi = moments.spectral_bounds(s, 50, 0.01, seed, H=H)
        a, b = hamiltonian.scale_from_bounds(lo, hi, 0.025)
        assert np.abs(ab[p] - np.array([a, b])).max() <= 1e-9 * (hi - lo), (s.dim, ab[p], a, b)
        want = moments.sector_moments(s, ab[p, 0], ab[p, 1], M, R, kind, seed, H=H)
        assert np.abs(mu[p] - want).max() <= tol * want[0], (s.dim, np.abs(mu[p] - want).max() / want[0])
    return st, mu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,R", [("rademacher", 1), ("rademacher", 3), ("complex_gaussian", 2), ("gaussian", 9)])
def test_all_sectors_of_a_chain(kpm, precision, kind, R):
    """48620 states down to 1: full tiles, tiles of four small blocks, columns
    that fill the last block and that do not."""
    st, _ = _check(kpm, W.sectors(W.j1j2_chain(18, 1.0, 0.5)), 22, R, kind, precision, 5)
    assert st["kernel"] == 5, st


@pytest.mark.parametrize("n,n_up,n_bonds,kernel", [
    (17, 10, 20, 1),    # 19448 states (float32): row kernel
    (16, 8, 20, 1),     # 12870
    (18, 10, 24, 5),    # 43758 states, 64-byte word rows
    (18, 9, 90, 1),     # more bonds than a word row of any width holds
])
def test_route_by_size_and_bonds(kpm, n, n_up, n_bonds, kernel):
    st, _ = _check(kpm, [W.Sector(_mixed_graph(n, n_bonds, 2), n_up, 0)], 16, 2, "rademacher", "fp32", 3)
    assert st["kernel"] == kernel, st


def test_placement_of_column_blocks_does_not_change_results(kpm, monkeypatch):
    """Blocks on one XCD each (chosen where they balance), in 8 chunks, in
    contiguous ranges and in order: the same workgroups in another order."""
    secs = W.sectors(W.ladder(18))
    bl = [(-20.0, 20.0)] * len(secs)
    ref = None
    for remap in (None, "3", "2", "1", "0"):
        if remap is None:
            monkeypatch.delenv("KPM_XCD_REMAP", raising=False)
        else:
            monkeypatch.setenv("KPM_XCD_REMAP", remap)
        mu, _ = kpm.chebyshev_moments(secs, 40, 20, "rademacher", "fp64", 0.025, 4, bounds=bl)
        assert kpm.last_run_stats()["kernel"] == 5
        mu = mu.cpu().numpy()
        ref = mu if ref is None else ref
        assert np.array_equal(mu, ref), remap


def test_unstable_windows_of_larger_chains_are_the_reference_ones(kpm):
    """Sawtooth chain of 18 sites, all sectors in one call (the largest ones on
    the slice kernel): every window within 1e-5 of the oracle's, those that do
    not hang on rounding to 1e-9."""
    secs = W.sectors(W.sawtooth(18))
    got = kpm.spectral_bounds(secs, 50, 0.01, 3)
    for p, s in enumerate(secs):
        want = np.array(moments.spectral_bounds(s, 50, 0.01, 3))
        assert np.abs(got[p] - want).max() <= (1e-9 if s.dim > 20000 or s.dim < 20 else 1e-4), (s.dim, got[p], want)
        alone = kpm.spectral_bounds([s], 50, 0.01, 3)[0]
        assert np.abs(got[p] - alone).max() <= 1e-9, (s.dim, got[p], alone)

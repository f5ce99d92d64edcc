"""Resident recursions (every step of a column in one launch): moments and
Lanczos bounds against the oracle at the sizes where rows, index entries and
threads run out, and the calls that stay on the step kernels.

Tolerances: moments 1e-10 mu_0, bounds 1e-9 of the window, as for every other
float64 path (the arithmetic is the same float64 sums in another order)."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import hamiltonian, moments

pytestmark = pytest.mark.gpu

TOL = 1e-10


def _graph(n, n_bonds, seed):
    """n_bonds bonds on n sites (repeats allowed), J in [0.5, 1.5]."""
    rng = np.random.default_rng([seed, n, n_bonds])
    bi = rng.integers(0, n, n_bonds)
    bj = (bi + rng.integers(1, n, n_bonds)) % n
    return W.Cluster(n, bi, bj, rng.uniform(0.5, 1.5, n_bonds))


def _check(kpm, secs, M, R, kind, seed, kernel, eps=0.025, **kw):
    mu, ab = kpm.chebyshev_moments(secs, M, R, kind, "fp64", eps, seed, **kw)
    assert kpm.last_run_stats()["kernel"] == kernel
    mu, ab = mu.cpu().numpy(), ab.cpu().numpy()
    for p, s in enumerate(secs):
        H = hamiltonian.sector_hamiltonian(s.cluster, s.n_up)
        lo, hi = moments.spectral_bounds(s, 50, 0.01, seed, H=H)
        a, b = hamiltonian.scale_from_bounds(lo, hi, eps)
        assert np.abs(ab[p] - np.array([a, b])).max() <= 1e-9 * (hi - lo), (p, ab[p], a, b)
        want = moments.sector_moments(s, ab[p, 0], ab[p, 1], M, R, kind, seed, H=H)
        assert np.abs(mu[p] - want).max() <= TOL * want[0], (p, s.dim, np.abs(mu[p] - want).max() / want[0])


@pytest.mark.parametrize("n,n_up,n_bonds", [
    (2, 1, 1), (3, 3, 2), (4, 2, 6),          # a handful of states; one state
    (8, 4, 8), (9, 5, 9),                     # 70 and 126 states (2 waves); 8 and 9 bonds: 1 and 2 entries
    (14, 10, 16), (13, 8, 17),                # 1001 and 1287 states: 1 and 2 rows per thread
    (14, 8, 24), (16, 12, 25), (15, 10, 32),  # 3003, 1820, 3003: indices kept or read; 3 and 4 entries
    (16, 10, 9), (16, 9, 24), (16, 8, 32),    # 8008, 11440, 12870 states: 8 and 13 rows per thread
    (20, 15, 20), (17, 10, 32),               # 15504 and 19448 states: 19 rows per thread
])
def test_sizes(kpm, n, n_up, n_bonds):
    sec = W.Sector(_graph(n, n_bonds, 3), n_up, 0)
    _check(kpm, [sec], 41, 2, "rademacher", 7, 6)


@pytest.mark.parametrize("n,n_up,n_bonds,kernel", [(17, 9, 20, 1), (10, 5, 33, 1)])
def test_larger_sectors_stay_on_the_step_kernels(kpm, n, n_up, n_bonds, kernel):
    _check(kpm, [W.Sector(_graph(n, n_bonds, 4), n_up, 0)], 30, 2, "rademacher", 1, kernel)


@pytest.mark.parametrize("kind,R", [("rademacher", 3), ("gaussian", 2), ("complex_gaussian", 3), ("basis", 0)])
def test_vector_kinds_over_uneven_sectors(kpm, kind, R):
    """Sectors of 1 to 462 states of two clusters in one call, M even and odd,
    steps past one ring of dots."""
    secs = W.sectors(_graph(11, 15, 5), cluster_id=0) + W.sectors(W.ring(6), cluster_id=3)
    for M in (2, 3, 16, 17, 19, 120):
        _check(kpm, secs, M, R, kind, 11, 6)


def test_given_and_estimated_windows_mixed(kpm):
    secs = W.sectors(W.j1j2_chain(12, 1.0, 0.5))
    est = kpm.spectral_bounds(secs, 50, 0.01, 0)
    mu_e, ab_e = kpm.chebyshev_moments(secs, 60, 4)
    bl = [None if k % 2 else tuple(est[k]) for k in range(len(secs))]
    mu, ab = kpm.chebyshev_moments(secs, 60, 4, bounds=bl)
    assert kpm.last_run_stats()["kernel"] == 6
    assert np.abs(ab.cpu().numpy() - ab_e.cpu().numpy()).max() <= 1e-14 * np.abs(est).max()
    dims = np.array([s.dim for s in secs])[:, None]
    assert (np.abs(mu.cpu().numpy() - mu_e.cpu().numpy()) / dims).max() <= 1e-12


@pytest.mark.parametrize("steps,margin", [(1, 0.0), (2, 0.05), (256, 0.01), (257, 0.01)])
def test_bounds_steps(kpm, steps, margin):
    """From one step to the last that the coefficients' LDS holds, and past it."""
    secs = W.sectors(_graph(11, 22, 6))
    got = kpm.spectral_bounds(secs, steps, margin, 2)
    for p, s in enumerate(secs):
        want = np.array(moments.spectral_bounds(s, steps, margin, 2))
        assert np.abs(got[p] - want).max() <= 1e-9 * max(1.0, np.abs(want).max()), (p, s.dim)


def test_step_kernels_on_request(kpm, monkeypatch):
    """The same moments from the step kernels (KPM_RESIDENT=0, and a block width)."""
    secs = W.sectors(W.ladder(12))
    mu, _ = kpm.chebyshev_moments(secs, 80, 5, "gaussian", seed=9)
    mu_b, _ = kpm.chebyshev_moments(secs, 80, 5, "gaussian", seed=9, col_block=5)
    assert kpm.last_run_stats()["kernel"] != 6
    monkeypatch.setenv("KPM_RESIDENT", "0")
    mu_s, _ = kpm.chebyshev_moments(secs, 80, 5, "gaussian", seed=9)
    assert kpm.last_run_stats()["kernel"] != 6
    dims = np.array([math.comb(12, s.n_up) for s in secs])[:, None]
    for other in (mu_b, mu_s):
        assert (np.abs(mu.cpu().numpy() - other.cpu().numpy()) / dims).max() <= 1e-11


@pytest.mark.parametrize("n,seed", [(10, 2), (12, 9), (14, 1)])
def test_windows_that_hang_on_rounding_are_the_stepped_ones(kpm, monkeypatch, n, seed):
    """Sawtooth chains: the top of the spectrum converges long before the
    nearly flat bottom, the Lanczos vectors lose orthogonality, and E_min after
    50 steps depends on the order of every sum (by up to 1e-5).  Such windows
    come from the stepped recursion, bit for bit; the others agree to rounding."""
    secs = W.sectors(W.sawtooth(n))
    got = kpm.spectral_bounds(secs, 50, 0.01, seed)
    mu, ab = kpm.chebyshev_moments(secs, 60, 3, seed=seed)
    assert kpm.last_run_stats()["kernel"] == 6
    mu_n, ab_n = kpm.chebyshev_moments_noalloc(secs, 60, 3, seed=seed)
    monkeypatch.setenv("KPM_RESIDENT", "0")
    want = kpm.spectral_bounds(secs, 50, 0.01, seed)
    mu_s, ab_s = kpm.chebyshev_moments(secs, 60, 3, seed=seed)
    assert (got == want).all(axis=1).any()                       # at least one was taken over
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    assert np.abs((ab - ab_s).cpu().numpy()).max() <= 1e-12 * np.abs(want).max()
    dims = np.array([s.dim for s in secs])[:, None]
    assert (np.abs((mu - mu_s).cpu().numpy()) / dims).max() <= 1e-10
    assert np.array_equal(mu.cpu().numpy(), mu_n.cpu().numpy()) and np.array_equal(ab.cpu().numpy(), ab_n.cpu().numpy())


def test_window_too_narrow_is_reported(kpm):
    s = W.Sector(W.ring(10), 5, 0)
    with pytest.raises(kpm.KPMError) as ei:
        kpm.chebyshev_moments([s], 200, 2, bounds=[(-1.0, 1.0)])
    assert ei.value.code == kpm.KPM_EBOUNDS


def _gradient(kpm, sec, M, R, kind, ckpt, seed):
    """dL/dJ of one sector, from the resumed and from the single call, against the oracle."""
    import torch

    from oracle import adjoint
    ps = kpm.ProblemSet([sec])
    mu, ab, ws = kpm.moments_ckpt(None, M, R, kind, seed=seed, ckpt_every=ckpt, problems=ps)
    mu0, ab0 = kpm.chebyshev_moments([sec], M, R, kind, seed=seed)
    assert kpm.last_run_stats()["kernel"] == 6
    assert torch.equal(ab, ab0) and torch.equal(mu, mu0)
    lam = np.random.default_rng(M).normal(size=(1, M))
    lam_d = torch.tensor(lam, device="cuda")
    got = kpm.moments_vjp_resume(ps, M, R, ab, lam_d, ws, kind, seed=seed, ckpt_every=ckpt).cpu().numpy()
    once = kpm.moments_vjp([sec], M, R, ab, lam_d, kind, seed=seed, ckpt_every=ckpt).cpu().numpy()
    a, b = ab.cpu().numpy()[0]
    want = adjoint.sector_moments_vjp(sec, a, b, M, R, kind, seed, lam[0])
    assert np.abs(got - want).max() <= 1e-9 * np.abs(want).max(), (sec.dim, M, ckpt)
    assert np.array_equal(got, once)


@pytest.mark.parametrize("n,n_up,n_bonds", [
    (2, 1, 1), (4, 2, 6), (12, 8, 8), (12, 6, 16),      # 2, 6, 495, 924 states: 1 and 2 rows per thread
    (13, 7, 24), (14, 7, 17), (15, 8, 32), (16, 8, 9),  # 1716, 3432, 6435, 12870: 4, 8, 16, 26 rows
    (17, 10, 25),                                       # 19448: 38 rows
])
def test_gradient_sizes(kpm, n, n_up, n_bonds):
    sec = W.Sector(_graph(n, n_bonds, 8), n_up, 0)
    _gradient(kpm, sec, 15, 2, "rademacher", 64, 3)      # every vector kept
    _gradient(kpm, sec, 15, 2, "rademacher", 2, 3)       # checkpoints every second step


@pytest.mark.parametrize("kind,R", [("rademacher", 3), ("gaussian", 2), ("complex_gaussian", 2), ("basis", 0)])
@pytest.mark.parametrize("M,ckpt", [(2, 2), (3, 2), (17, 4), (18, 4), (40, 6), (41, 20), (42, 21), (64, 32)])
def test_gradient_kinds_and_checkpoints(kpm, kind, R, M, ckpt):
    """Moment counts even and odd, intervals that divide the steps or not, one
    short of the whole trajectory and the whole of it."""
    _gradient(kpm, W.Sector(_graph(9, 14, 9), 5, 2), M, R, kind, ckpt, 4)


def test_gradient_of_several_sectors_matches_the_step_kernels(kpm, monkeypatch):
    secs = W.sectors(_graph(10, 15, 10), cluster_id=0) + W.sectors(W.ring(7), cluster_id=1)
    T = W.log_temperatures(20, 0.5, 5.0)
    wC, wX = np.random.default_rng(1).uniform(0.5, 1.5, (2, 2, 20))
    out = []
    for env in ("1", "0"):
        monkeypatch.setenv("KPM_RESIDENT", env)
        L, dJ, ab = kpm.thermo_grad(secs, 60, 3, T, wC, wX, "complex_gaussian", kernel="jackson", ckpt_every=8, seed=5)
        out.append((float(L), dJ.cpu().numpy(), ab.cpu().numpy()))
    assert abs(out[0][0] - out[1][0]) <= 1e-10 * abs(out[1][0])
    assert np.abs(out[0][1] - out[1][1]).max() <= 1e-9 * np.abs(out[1][1]).max()


def test_gradient_refuses_an_unusable_map(kpm):
    import torch
    sec = W.Sector(W.ring(8), 4, 0)
    ab = torch.tensor([[0.0, 1.0]], dtype=torch.float64, device="cuda")
    lam = torch.ones((1, 8), dtype=torch.float64, device="cuda")
    with pytest.raises(kpm.KPMError) as ei:
        kpm.moments_vjp([sec], 8, 2, ab, lam, ckpt_every=4)
    assert ei.value.code == kpm.KPM_EINVAL

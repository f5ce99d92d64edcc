"""Which calls the float64 moments and gradients of small sectors run resident:
one column is one compute unit's work, so large sectors with few columns and many
steps stay on the step kernels (read off the workspace's size, which those
routes lay out differently; CPU), and both routes agree (GPU)."""
import ctypes

import numpy as np
import pytest

import workloads as W
from paper_2104_13218_amd import kpm as K


def _graph(n, n_bonds, seed=1):
    rng = np.random.default_rng([seed, n, n_bonds])
    bi = rng.integers(0, n, n_bonds)
    return W.Cluster(n, bi, (bi + rng.integers(1, n, n_bonds)) % n, rng.uniform(0.5, 1.5, n_bonds))


def _sizes(monkeypatch, secs, M, R, kind):
    """The call's size, and the step kernels' one."""
    ps = K.ProblemSet(secs, [(-60.0, 60.0)] * len(secs))
    q, out = K.make_params(M, R, "rademacher", "fp64"), []
    for env in (None, "0"):
        monkeypatch.delenv("KPM_RESIDENT", raising=False)
        if env is not None:
            monkeypatch.setenv("KPM_RESIDENT", env)
        out.append(K.moments_workspace_size(ps, q) if kind == "moments" else
                   int(K.load().chebyshev_moments_vjp_workspace_size(ps.arr, len(ps), ctypes.byref(q), 64)))
    return out


@pytest.mark.parametrize("n,n_up,M,R,resident", [
    (16, 8, 400, 1, True),                              # 12870 states
    (20, 15, 400, 2, False), (20, 15, 400, 3, True),    # 15504
    (17, 10, 400, 8, False), (17, 10, 400, 9, True),    # 19448
    (17, 10, 47, 1, True), (17, 10, 48, 1, False),      # 23 and 24 steps
])
def test_moments_by_columns(monkeypatch, n, n_up, M, R, resident):
    got, stepped = _sizes(monkeypatch, [W.Sector(_graph(n, 24), n_up, 0)], M, R, "moments")
    assert (got != stepped) == resident


@pytest.mark.parametrize("n,n_up,M,R,resident", [
    (23, 19, 400, 1, True),                             # 8855
    (16, 8, 400, 2, False), (16, 8, 400, 3, True),      # 12870
    (16, 8, 64, 1, True), (16, 8, 66, 1, False),        # 32 and 33 steps
    (17, 10, 400, 15, False), (17, 10, 400, 16, True),  # 19448
    (17, 10, 23, 1, True), (17, 10, 24, 1, False),      # 11 and 12 steps
])
def test_gradient_by_columns(monkeypatch, n, n_up, M, R, resident):
    got, stepped = _sizes(monkeypatch, [W.Sector(_graph(n, 24), n_up, 0)], M, R, "gradient")
    assert (got != stepped) == resident


def test_gradient_of_few_bonds_keeps_the_step_kernels(monkeypatch):
    for n_bonds, resident in ((15, False), (16, True)):
        got, stepped = _sizes(monkeypatch, [W.Sector(_graph(17, n_bonds), 10, 0)], 400, 16, "gradient")
        assert (got != stepped) == resident


@pytest.mark.parametrize("n,n_up,R,resident", [
    (23, 19, 2, False), (23, 19, 3, True),              # 8855
    (16, 8, 8, False), (16, 8, 9, True),                # 12870
])
def test_gradient_of_many_bonds(monkeypatch, n, n_up, R, resident):
    got, stepped = _sizes(monkeypatch, [W.Sector(_graph(n, 25), n_up, 0)], 400, R, "gradient")
    assert (got != stepped) == resident


def test_smaller_sectors_count_by_their_rows(monkeypatch):
    """The sectors of 17 sites that can be resident: the largest has 19448 of
    their 41226 rows."""
    secs = [s for s in W.sectors(_graph(17, 24)) if s.dim < 20000]
    rows = sum(s.dim for s in secs) / max(s.dim for s in secs)
    for kind, line in (("moments", 9), ("gradient", 16)):
        at = int(-(-line // rows))
        for R, resident in ((at - 1, False), (at, True)):
            got, stepped = _sizes(monkeypatch, secs, 400, R, kind)
            assert (got != stepped) == resident, (kind, R)


@pytest.mark.gpu
@pytest.mark.parametrize("R", [2, 8, 9])
def test_moments_on_either_side(kpm, R):
    from oracle import hamiltonian, moments
    sec = W.Sector(_graph(17, 24), 10, 0)
    mu, ab = kpm.chebyshev_moments([sec], 60, R, "rademacher", "fp64", seed=3, bounds=[(-40.0, 40.0)])
    assert (kpm.last_run_stats()["kernel"] == 6) == (R == 9)
    ab = ab.cpu().numpy()[0]
    want = moments.sector_moments(sec, ab[0], ab[1], 60, R, "rademacher", 3, H=hamiltonian.sector_hamiltonian(sec.cluster, 10))
    assert np.abs(mu.cpu().numpy()[0] - want).max() <= 1e-10 * want[0]


@pytest.mark.gpu
def test_checkpointed_gradient_beside_resident_moments(kpm):
    """16 sites, 28 bonds, four columns: the moments run resident, the gradient on the
    step kernels; forward, resumed and single call against the oracle."""
    import torch
    from oracle import adjoint
    sec, M, R = W.Sector(_graph(16, 28), 8, 0), 30, 4
    ps = kpm.ProblemSet([sec])
    mu, ab, ws = kpm.moments_ckpt(None, M, R, seed=2, ckpt_every=4, problems=ps)
    mu0, ab0 = kpm.chebyshev_moments([sec], M, R, seed=2)
    assert kpm.last_run_stats()["kernel"] == 6
    assert (ab - ab0).abs().max() <= 1e-13 * ab.abs().max()
    assert (mu - mu0).abs().max() <= 1e-11 * mu0[0, 0]
    lam = np.random.default_rng(1).normal(size=(1, M))
    lam_d = torch.tensor(lam, device="cuda")
    got = kpm.moments_vjp_resume(ps, M, R, ab, lam_d, ws, seed=2, ckpt_every=4).cpu().numpy()
    once = kpm.moments_vjp([sec], M, R, ab, lam_d, seed=2, ckpt_every=4).cpu().numpy()
    a, b = ab.cpu().numpy()[0]
    want = adjoint.sector_moments_vjp(sec, a, b, M, R, "rademacher", 2, lam[0])
    assert np.abs(got - want).max() <= 1e-9 * np.abs(want).max()
    assert np.abs(once - want).max() <= 1e-9 * np.abs(want).max()


@pytest.mark.gpu
@pytest.mark.parametrize("n,n_up,n_bonds,R", [
    (9, 5, 14, 2), (12, 6, 9, 2), (12, 6, 31, 2), (13, 7, 17, 2), (14, 7, 32, 2),   # 1 to 8 rows a thread
    (16, 10, 16, 2), (16, 10, 25, 2),                                               # 16 rows, two and four index entries
    (16, 8, 16, 9), (16, 8, 24, 9),                                                 # 26 rows, row sums
    (16, 8, 25, 9), (17, 10, 16, 16)])                                              # 26 and 38 rows, operands picked
def test_gradient_of_bonds_that_do_not_act(kpm, n, n_up, n_bonds, R):
    """Every number of rows a thread has, with and without the rows' own sums."""
    import torch
    from oracle import adjoint
    sec, M = W.Sector(_graph(n, n_bonds, 5), n_up, 0), 26
    a, b = 1.1 * n_bonds, 0.3
    ab = torch.tensor([[a, b]], dtype=torch.float64, device="cuda")
    lam = np.random.default_rng(2).normal(size=(1, M))
    got = kpm.moments_vjp([sec], M, R, ab, torch.tensor(lam, device="cuda"), seed=4, ckpt_every=4).cpu().numpy()
    want = adjoint.sector_moments_vjp(sec, a, b, M, R, "rademacher", 4, lam[0])
    assert np.abs(got - want).max() <= 1e-9 * np.abs(want).max()

"""Calls that estimate windows before their own work do it inside the memory
they were given, a second estimate of windows that hang on rounding included:
the windows are kpm_spectral_bounds' and nothing behind the queried size is
touched.  Sawtooth chains: such windows are common there."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
GUARD = 4 << 20


def _region(need):
    return torch.full((need + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")


def _scale(kpm, secs, seed, eps=0.025):
    e = kpm.spectral_bounds(secs, 50, 0.01, seed)
    return np.stack([(e[:, 1] - e[:, 0]) / (2.0 - eps), 0.5 * (e[:, 1] + e[:, 0])], axis=1)


@pytest.mark.parametrize("n,ups", [(12, range(6, 13)), (18, [9])])
@pytest.mark.parametrize("seed", [1, 3, 9])
def test_windows_of_checkpointed_moments(kpm, n, ups, seed):
    secs = [W.Sector(W.sawtooth(n), k, 0) for k in ups]
    ps, M, ck, lib = kpm.ProblemSet(secs), 12, 4, kpm.load()
    q = kpm.make_params(M, 2, "rademacher", seed=seed)
    need = int(lib.chebyshev_moments_ckpt_workspace_size(ps.arr, len(ps), ctypes.byref(q), ck))
    ws = _region(need)
    mu = torch.empty((len(ps), M), dtype=torch.float64, device="cuda")
    ab = torch.empty((len(ps), 2), dtype=torch.float64, device="cuda")
    r = lib.chebyshev_moments_ckpt(ps.arr, len(ps), ctypes.byref(q), ck, mu.data_ptr(), ab.data_ptr(), ws.data_ptr(),
                                   need, None)
    assert r == 0, kpm.strerror(r)
    assert np.abs(ab.cpu().numpy() - _scale(kpm, secs, seed)).max() <= 1e-14 * n
    lam = torch.ones((len(ps), M), dtype=torch.float64, device="cuda")
    dJ = kpm.moments_vjp_resume(ps, M, 2, ab, lam, ws[:need], seed=seed, ckpt_every=ck)
    want = kpm.moments_vjp(secs, M, 2, ab, lam, seed=seed, ckpt_every=ck)
    assert (dJ - want).abs().max() <= 1e-11 * want.abs().max()
    assert bool((ws[need:] == 0x5A).all())


@pytest.mark.parametrize("n,n_up", [(12, 7), (18, 9)])
@pytest.mark.parametrize("seed", [1, 3, 9])
def test_windows_of_vectors(kpm, n, n_up, seed):
    sec = W.Sector(W.sawtooth(n), n_up, 0)
    ps, lib = kpm.ProblemSet([sec]), kpm.load()
    q = kpm.make_params(6, 2, "rademacher", seed=seed)
    need = int(lib.chebyshev_vectors_workspace_size(ps.arr, ctypes.byref(q), 3))
    ws = _region(need)
    out = torch.empty((sec.dim, 2), dtype=torch.float64, device="cuda")
    ab = torch.empty(2, dtype=torch.float64, device="cuda")
    r = lib.chebyshev_vectors(ps.arr, ctypes.byref(q), 3, out.data_ptr(), ab.data_ptr(), ws.data_ptr(), need, None)
    assert r == 0, kpm.strerror(r)
    assert np.abs(ab.cpu().numpy() - _scale(kpm, [sec], seed)[0]).max() <= 1e-14 * n
    assert bool((ws[need:] == 0x5A).all())

"""The reverse sweep reads no window: chebyshev_moments_vjp_resume finds what
the forward call left whether its problems come with the windows that the forward
call estimated or without any."""
import ctypes

import numpy as np
import pytest

import workloads as W
from paper_2104_13218_amd import kpm as K


def _secs():
    return W.sectors(W.j1j2_chain(10, 1.0, 0.5))


@pytest.mark.parametrize("steps", [50, 256, 300])
@pytest.mark.parametrize("given", ["one", "all"])
def test_layout_does_not_depend_on_windows(steps, given):
    secs = _secs()
    q = K.make_params(24, 3, "rademacher", lanczos_steps=steps)
    size = lambda b: K.load().chebyshev_moments_vjp_workspace_size(  # noqa: E731
        K.ProblemSet(secs, b).arr, len(secs), ctypes.byref(q), 6)
    bounds = [(-9.0, 9.0) if given == "all" or k == 0 else None for k in range(len(secs))]
    assert size(bounds) == size([None] * len(secs)) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("ckpt", [4, 64])
def test_resume_with_the_windows_given(kpm, ckpt):
    secs, M = _secs(), 24
    mu, ab, ws = kpm.moments_ckpt(secs, M, 3, seed=2, ckpt_every=ckpt)
    a, b = ab.cpu().numpy().T
    half = 0.5 * a * (2.0 - 0.025)
    import torch
    lam = torch.tensor(np.random.default_rng(0).normal(size=(len(secs), M)), device="cuda")
    got = [kpm.moments_vjp_resume(kpm.ProblemSet(secs, w), M, 3, ab, lam, ws, seed=2, ckpt_every=ckpt).cpu().numpy()
           for w in ([None] * len(secs), list(zip(b - half, b + half)))]
    assert np.array_equal(got[0], got[1])

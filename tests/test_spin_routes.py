"""Which of the two spin-s kernels a plan takes (read off the workspace's size
on the CPU: the list kernel's lists and the split kernel's records differ), and
that the routes agree on the GPU."""
import numpy as np
import pytest

import workloads as W
from paper_2104_13218_amd import kpm as K


def _ring(n, two_s):
    return W.spin_sectors(W.Cluster(n, range(n), [(i + 1) % n for i in range(n)], np.ones(n)), two_s)


def _full(n, two_s):
    i, j = zip(*[(a, b) for a in range(n) for b in range(a)])
    return W.spin_sectors(W.Cluster(n, i, j, np.ones(len(i))), two_s)


def _size(secs, R, precision):
    ps = K.ProblemSet(secs, [(-90.0, 90.0)] * len(secs))
    return K.moments_workspace_size(ps, K.make_params(16, R, "rademacher", precision))


@pytest.mark.parametrize("secs,R,precision,split", [
    (_ring(9, 2)[:1], 16, "fp64", True), (_ring(9, 2)[:1], 17, "fp64", False),     # 8 and 9 lanes of two
    (_ring(9, 2), 32, "fp32", True), (_ring(9, 2), 33, "fp32", False),             # 8 and 9 lanes of four
    (_full(7, 2)[:1], 48, "fp64", True), (_ring(7, 2)[:1], 48, "fp64", False),     # 21 and 7 bonds
    (_ring(12, 3)[:1], 32, "fp64", True), (_ring(12, 3)[:1], 64, "fp64", False),   # lists of 177 MB: 16 and 32 lanes
])
def test_route(monkeypatch, secs, R, precision, split):
    got = _size(secs, R, precision)
    monkeypatch.setenv("KPM_SPIN_SPLIT", "2")
    forced = _size(secs, R, precision)
    monkeypatch.setenv("KPM_SPIN_SPLIT", "0")
    lists = _size(secs, R, precision)
    assert forced != lists and got == (forced if split else lists)


@pytest.mark.gpu
@pytest.mark.parametrize("secs,R,precision", [
    (_ring(9, 2), 24, "fp64"), (_ring(6, 5), 48, "fp64"), (_full(6, 3), 40, "fp32"), (_ring(8, 3), 37, "fp32"),
    (_ring(13, 2)[:1], 64, "fp32")])   # the last: a slot of 52 MB, eight columns per lane
def test_routes_agree(kpm, monkeypatch, secs, R, precision):
    """The same terms in the same order: the same bits, and with eight columns
    per lane another order of a dot's dim terms of at most one each."""
    got = {}
    for split in ("0", "1", "2"):
        monkeypatch.setenv("KPM_SPIN_SPLIT", split)
        mu, _ = kpm.chebyshev_moments(secs, 12, R, "rademacher", precision, 0.025, 6, bounds=[(-90.0, 90.0)] * len(secs))
        assert kpm.last_run_stats()["kernel"] == 4
        got[split] = mu.cpu().numpy()
    dims = np.array([[s.dim] for s in secs], dtype=float)
    for other in ("1", "2"):
        if secs[0].dim > 200000:
            assert (np.abs(got["0"] - got[other]) <= 2 * dims * dims * 2.0 ** -53).all()
        else:
            assert np.array_equal(got["0"], got[other])

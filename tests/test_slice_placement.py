"""Which calls of the slice kernel keep each column block on one XCD: those whose
XCDs' loads are even and whose slots are of up to 4 MB on average.  Read off the
workgroup records in the workspace's size: a queue per XCD is padded to the
longest, the plan that sweeps one block at a time pads block by block."""
import pytest

import workloads as W
from paper_2104_13218_amd import kpm as K


def _size(secs, R):
    ps = K.ProblemSet(secs, [(-90.0, 90.0)] * len(secs))
    return K.moments_workspace_size(ps, K.make_params(40, R, "rademacher", "fp64"))


@pytest.mark.parametrize("n,clusters,R,one_xcd", [
    (18, 1, 20, True), (20, 1, 16, True), (20, 8, 20, True),   # 0.5 and 1.7 MB
    (22, 1, 20, False), (22, 8, 20, False), (24, 1, 20, False),  # 6 and 23 MB
    (18, 1, 8, False),                                         # uneven
])
def test_placement(monkeypatch, n, clusters, R, one_xcd):
    secs = [s for c in range(clusters) for s in W.sectors(W.ring(n), cluster_id=c)]
    monkeypatch.delenv("KPM_XCD_REMAP", raising=False)
    got = _size(secs, R)
    monkeypatch.setenv("KPM_XCD_REMAP", "3")
    queues = _size(secs, R)
    monkeypatch.setenv("KPM_XCD_REMAP", "2")
    sweep = _size(secs, R)
    assert queues != sweep
    assert got == (queues if one_xcd else sweep)

"""The split spin kernel (neighbour ranks from the two halves of a digit
string) against the list kernel, which it replaces where its records are small:
both sum the same terms of a row in the same order, so the bounds (one float64
column, the same tiles) and every moment whose dots keep their order are the
same bits.  With eight columns per lane (float32, a multiple of eight columns)
only the order of a dot's dim terms differs: dim * 2^-53 of the moment's
largest, <v_0, v_0> = dim."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _sectors(n_sites, two_s, bonds):
    rng = np.random.default_rng(n_sites * 8 + two_s)
    i, j = zip(*bonds)
    return W.spin_sectors(W.Cluster(n_sites, i, j, rng.uniform(0.4, 1.6, len(bonds))), two_s)


RING = lambda n: [(i, (i + 1) % n) for i in range(n)]  # noqa: E731
GRAPHS = [
    (4, 5, RING(4)),                                          # four sites of spin 5/2
    (5, 3, RING(5) + [(0, 2), (1, 4)]),                       # halves of two and three sites, odd number of bonds
    (7, 2, [(6, 0), (3, 2), (5, 1), (4, 6), (2, 0), (1, 3)]),  # bonds given from either end
    (2, 7, [(1, 0)]),                                         # one site a half, one bond
    (8, 4, RING(8)),                                          # tiles with remainders, 38165 rows at most
]


@pytest.mark.parametrize("precision, R", [("fp64", 1), ("fp64", 5), ("fp32", 3), ("fp32", 16), ("fp32", 24)])
@pytest.mark.parametrize("graph", GRAPHS, ids=lambda g: f"{g[0]}x{g[1]}")
def test_split_against_lists(kpm, monkeypatch, graph, precision, R):
    secs = _sectors(*graph)
    got = {}
    for split in ("0", "1"):
        monkeypatch.setenv("KPM_SPIN_SPLIT", split)
        bounds = kpm.spectral_bounds(secs, seed=4)
        mu, ab = kpm.chebyshev_moments(secs, 24, R, "rademacher", precision, 0.025, 6)
        assert kpm.last_run_stats()["kernel"] == 4
        got[split] = bounds, mu.cpu().numpy(), ab.cpu().numpy()
    assert np.array_equal(got["0"][0], got["1"][0])
    assert np.array_equal(got["0"][2], got["1"][2])
    if precision == "fp32" and R % 8 == 0:
        dims = np.array([[s.dim] for s in secs], dtype=float)
        assert (np.abs(got["0"][1] - got["1"][1]) <= 2 * dims * dims * 2.0 ** -53).all()
    else:
        assert np.array_equal(got["0"][1], got["1"][1])

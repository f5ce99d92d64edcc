"""Householder reduction at the edges of its steps: sectors of two states (no
step), three (one step, its update in the last block), rows already zero (the
one-magnon chain is tridiagonal as it stands, up to the closing bond), and the
largest sector of a call beside the smallest.  Bound: the reduction and the
bisection each move an eigenvalue by at most D 2^-52 of the norm; 1e-12 covers
D = 1001 four times."""
import numpy as np
import pytest

import workloads as W
from oracle import ed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cl", [
    W.Cluster(2, [0], [1], [1.0]), W.Cluster(3, [0, 1], [1, 2], [1.0, 0.7]), W.Cluster(4, [0, 1, 2], [1, 2, 3], [1.0, 1.0, 1.0]),
    W.ring(7), W.Cluster(14, list(range(13)), list(range(1, 14)), np.linspace(0.6, 1.4, 13))], ids=lambda c: f"N{c.n_sites}")
def test_edges_of_the_reduction(kpm, cl):
    secs = [s for s in W.sectors(cl) if s.dim <= 1024]
    ev = kpm.sector_eigenvalues(secs, 1024).cpu().numpy()
    for row, s, (e, _, _) in zip(ev, secs, ed.sector_spectra(secs)):
        assert np.abs(row[:s.dim] - e).max() <= 1e-12 * max(1.0, np.abs(e).max()), s.dim

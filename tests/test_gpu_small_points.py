"""Small thermodynamics calls take a kernel of one pass, and few problems take a
wave each for the weights of a pair of nodes.  They form the same sums of the
same sectors in the same order as the kernels of large calls, so a point has
the same bits whichever takes it: a call of a few points against the same
points among many, on both sides of the line, with fields and without, with
KPM sectors and with exact levels, with fewer sectors than a workgroup's waves
and with more; a cluster alone against the same cluster among many."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import moments

pytestmark = pytest.mark.gpu


def inputs(sizes, M, seed):
    rng = np.random.default_rng(seed)
    secs = [s for c, n in enumerate(sizes) for s in W.sectors(W.ring(n), cluster_id=c)]
    mus = np.array([moments.exact_moments(np.sort(rng.uniform(-0.97, 0.97, 40)), M) for _ in secs])
    ab = np.array([(rng.uniform(2.0, 6.0), rng.uniform(-3.0, 1.0)) for _ in secs])
    return rng, secs, torch.tensor(mus, device="cuda"), torch.tensor(ab, device="cuda")


@pytest.mark.parametrize("sizes", [(3,), (8,), (34, 9, 5)])
@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("levels", [False, True])
def test_a_point_alone_and_among_many(kpm, sizes, field, levels):
    M = 64
    rng, secs, mu, ab = inputs(sizes, M, 7 * len(sizes) + field)
    line = (2000000 if field else 250000) // (len(secs) * M)
    many = line + 100
    T = rng.choice(W.log_temperatures(61, 0.1, 10.0), many)
    h = rng.choice([0.0, 0.3, -0.8], many) if field else None
    kw = {}
    if levels:
        exact = [s.dim <= 70 for s in secs]
        ev = np.full((len(secs), 70), np.nan)
        for e, s, x in zip(ev, secs, exact):
            if x:
                e[:s.dim] = np.sort(rng.uniform(-4.0, 3.0, s.dim))
        kw = dict(evals=torch.tensor(ev, device="cuda"), exact=exact)

    def run(n):
        hh = None if h is None else h[:n]
        if levels:
            return kpm.thermo_hybrid(mu, ab, secs, T=T[:n], h=hh, kernel="jackson", **kw)
        if field:
            return kpm.thermo_field(mu, ab, secs, T[:n], hh, "jackson")
        return kpm.thermo(mu, ab, secs, T[:n], "jackson")

    full = run(many)
    for n in (1, 5, line, line + 1):
        got = run(n)
        for q, x in got.items():
            assert torch.equal(x, full[q][..., :n]), (q, n)


@pytest.mark.parametrize("last", [(), (5,), (3,), (3, 5, 3, 7)])
def test_a_cluster_alone_and_among_many(kpm, last):
    """4 k, 4 k + 3, + 2 and + 3 problems with 97 nodes: past the line each wave
    takes four of them, below it one."""
    M = 97
    _, secs, mu, ab = inputs((7,) * 15 + last, M, 3)
    assert len(secs) >= 60 and (((M + 1) // 2 + 3) // 4) * len(secs) > 768
    T = W.log_temperatures(9, 0.1, 10.0)
    full = kpm.thermo(mu, ab, secs, T, "jackson")
    n = 0
    for c in range(15 + len(last)):
        one = W.sectors(W.ring(((7,) * 15 + last)[c]))
        got = kpm.thermo(mu[n:n + len(one)].contiguous(), ab[n:n + len(one)].contiguous(), one, T, "jackson")
        n += len(one)
        for q, x in got.items():
            assert torch.equal(x[0], full[q][c]), (q, c)

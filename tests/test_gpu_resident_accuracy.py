"""The resident kernels round no more than the step kernels that they replace:
the errors of both against the same recursion in 80 bits, over sets of moments
and gradients.  A row's sum has half its terms at the weight of a bond that
acts, as on the step kernels, so that the errors' geometric means agree to a
few tens of per cent (the order of the sums differs); 1.4 leaves room for 24 sets."""
import numpy as np
import pytest

import workloads as W
from oracle import hamiltonian, rng

pytestmark = pytest.mark.gpu
LD = np.longdouble


class Rows:
    """Bond terms of one sector: H_b v = diag_b v + amp_b v[partner_b]."""

    def __init__(self, cl, n_up):
        self.J, self.terms = cl.J, []
        for i, j in zip(cl.bond_i, cl.bond_j):
            H = hamiltonian.sector_hamiltonian(W.Cluster(cl.n_sites, [i], [j], [1.0]), n_up).tocoo()
            dim = H.shape[0]
            diag, part, amp, off = np.zeros(dim), np.arange(dim), np.zeros(dim), H.row != H.col
            diag[H.row[~off]] = H.data[~off]
            part[H.row[off]], amp[H.row[off]] = H.col[off], H.data[off]
            self.terms.append((diag.astype(LD)[:, None], part, amp.astype(LD)[:, None]))
        self.dim = dim

    def bond(self, q, v):
        d, p, a = self.terms[q]
        return d * v + a * v[p]

    def scaled(self, v, a, b):
        return (sum(LD(J) * self.bond(q, v) for q, J in enumerate(self.J)) - LD(b) * v) / LD(a)


def _vectors(rows, a, b, seed, n_up, R, K):
    V = np.stack([rng.rademacher(seed, 0, n_up, r, rows.dim) for r in range(R)], 1).astype(LD)
    vs = [V, rows.scaled(V, a, b)]
    for _ in range(1, K):
        vs.append(2 * rows.scaled(vs[-1], a, b) - vs[-2])
    return vs


def _moments(vs, M):
    al, be = [(v * v).sum(0) for v in vs], [(u * v).sum(0) for u, v in zip(vs, vs[1:])]
    t = [al[0], be[0]] + [2 * al[n // 2] - al[0] if n % 2 == 0 else 2 * be[n // 2] - be[0] for n in range(2, M)]
    return np.array([(x / al[0]).mean() for x in t]) * vs[0].shape[0]


def _gradient(rows, vs, a, b, lam):
    M, K, R = lam.size, len(vs) - 1, vs[0].shape[1]
    c = rows.dim / (R * (vs[0] * vs[0]).sum(0))
    lam = np.concatenate([lam, np.zeros(3)]).astype(LD)
    odd = sum(lam[2 * n + 1] for n in range(1, K + 1) if 2 * n + 1 < M)
    g_al = lambda n: 2 * lam[2 * n] * c if 2 * n < M else 0 * c  # noqa: E731
    g_be = lambda n: (lam[1] - odd) * c if n == 0 else (2 * lam[2 * n + 1] * c if 2 * n + 1 < M else 0 * c)  # noqa: E731
    dJ, w1, w2 = np.zeros(rows.J.size, LD), None, None
    for n in range(K, 0, -1):
        w = 2 * g_al(n) * vs[n] + g_be(n - 1) * vs[n - 1]
        if n < K:
            w = w + g_be(n) * vs[n + 1] + 2 * rows.scaled(w1, a, b)
        if w2 is not None:
            w = w - w2
        dJ += [(1 if n == 1 else 2) / LD(a) * (w * rows.bond(q, vs[n - 1])).sum() for q in range(rows.J.size)]
        w1, w2 = w, w1
    return dJ


@pytest.mark.parametrize("what", ["moments", "gradient"])
def test_errors_against_80_bits(kpm, monkeypatch, what):
    import torch
    M, R, logs = 128, 2, []
    for cl in (W.ring(10), W.j1j2_chain(11, 1.0, 0.5), W.sawtooth(12), W.ladder(10)):
        for n_up in ((cl.n_sites + 1) // 2, (cl.n_sites + 1) // 2 + 2):
            rows, sec = Rows(cl, n_up), W.Sector(cl, n_up, 0)
            e = np.linalg.eigvalsh(hamiltonian.sector_hamiltonian(cl, n_up).toarray())
            lo, hi = e[0] - 0.01, e[-1] + 0.01
            a, b = hamiltonian.scale_from_bounds(lo, hi, 0.025)
            for seed in range(3):
                vs = _vectors(rows, a, b, seed, n_up, R, M // 2)
                lam = np.random.default_rng(seed).normal(size=M) / (1 + np.arange(M))
                ref = _moments(vs, M) if what == "moments" else _gradient(rows, vs, a, b, lam)
                err = []
                for env in ("1", "0"):
                    monkeypatch.setenv("KPM_RESIDENT", env)
                    if what == "moments":
                        got = kpm.chebyshev_moments([sec], M, R, "rademacher", "fp64", 0.025, seed, bounds=[(lo, hi)])[0][0]
                    else:
                        ab = torch.tensor([[a, b]], dtype=torch.float64, device="cuda")
                        got = kpm.moments_vjp([sec], M, R, ab, torch.tensor(lam[None], device="cuda"), seed=seed, ckpt_every=16)
                    err.append(float(np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()))
                logs.append(np.log(max(err[0], 1e-17) / max(err[1], 1e-17)))
    assert np.exp(np.mean(logs)) <= 1.4, np.exp(np.mean(logs))

"""Calls that fit the allocation-free entry point's 64 MiB on the row and
block-table kernels keep fitting it: the slice kernel, the default of large
sectors, pads every column block to one width and leaves such calls to them."""
import numpy as np
import pytest

import workloads as W
from paper_2104_13218_amd import kpm

LIMIT = 64 << 20


def _need(R):
    return kpm.moments_workspace_size(kpm.ProblemSet(W.sectors(W.sawtooth(20))),
                                      kpm.make_params(500, R, "rademacher", "fp32", 0.025, 1))


def test_padded_blocks_do_not_pass_the_limit():
    """616666 rows: 11 columns take 62 MB in blocks as wide as they need, 84 MB in two of eight."""
    need = {R: _need(R) for R in (8, 11, 16)}
    assert need[8] <= LIMIT and need[11] <= LIMIT < need[16]


@pytest.mark.gpu
def test_call_at_the_limit_runs():
    secs = W.sectors(W.sawtooth(20))
    args = (secs, 12, 11, "rademacher", "fp32", 0.025, 3)
    mu, ab = kpm.chebyshev_moments(*args)
    assert kpm.last_run_stats()["kernel"] != 5
    mu_n, ab_n = kpm.chebyshev_moments_noalloc(*args)
    assert np.array_equal(mu.cpu().numpy(), mu_n.cpu().numpy())
    assert np.array_equal(ab.cpu().numpy(), ab_n.cpu().numpy())

"""Right-hand sides of any magnitude: the moments grow with its square and the squared norms of the Hankel
SVD's columns with its fourth power, whose products leave the range of a double from 1e38 on.  Orders on
every side of the factorisation's kernels (64, 80, 136).

Tolerance: the eigenvalues do not depend on the scale; both sides solve to residuals below 1e-11 in the
same order of sums, so they agree to 1e-8, the bar of the batched solves against the dense oracle, and the
largest singular value goes with the square of the scale to 1e-8."""
import numpy as np
import pytest

import workloads as W
from oracle import qep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M", [(8, 8), (10, 8), (17, 8)])
def test_eigenvalues_do_not_depend_on_the_scale(cuda, L, M):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(8, 8, 12, 0.4, 4, 6, 991, 992, with_proj=True, r_c=1.1)
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 993)).to(cuda)
    s, prm = cbs.System.from_workload(sysw), cbs.default_params(n_rhs=L, n_mom=M, tol=1e-11)
    lam, _, _, info, rc = s.solve(1.3, V, prm, want_vectors=False)
    assert rc == 0 and len(lam) > 0
    for e in (-60, -30, 30, 37, 38, 39, 40, 41, 45, 60):
        print(L, M, e, flush=True)
        got, _, _, gi, rc = s.solve(1.3, V * 10.0 ** e, prm, want_vectors=False)
        assert rc == 0 and len(got) == len(lam) and qep.match_sets(got, lam) <= 1e-8
        assert abs(gi.sigma_first * 10.0 ** (-2 * e) - info.sigma_first) <= 1e-8 * info.sigma_first

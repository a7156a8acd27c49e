"""Energies whose Hankel SVDs run side by side, against the same energies one call each: orders on
either side of the kernels' changes (64, 128), more energies than a group holds (32) and groups that
are not full, on the path that carries a run in one workgroup and on the work queue.

Tolerance: the two solve to residuals below 1e-11 in another order of sums, so the largest singular value
and the eigenvalues agree to 1e-8, the bar of the batched solves against the dense oracle.  The rank
itself follows the solves' residuals, which are noise, and may differ where a singular value lies at
that floor."""
import numpy as np
import pytest

import workloads as W
from oracle import qep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M,nE,queue", [(8, 8, 7, False), (4, 8, 35, False), (16, 5, 3, False), (17, 8, 2, False),
                                          (8, 8, 5, True)])
def test_groups_match_single_calls(cuda, monkeypatch, L, M, nE, queue):
    import torch
    import paper_1709_09347_amd as cbs
    if queue:
        monkeypatch.setenv("CBS_RUN_WG", "0")
    sysw = W.make_system(8, 8, 12, 0.4, 4, 6, 971, 972, with_proj=True, r_c=1.1)
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 973)).to(cuda)
    E = np.linspace(0.9, 1.6, nE)
    s, prm = cbs.System.from_workload(sysw), cbs.default_params(n_rhs=L, n_mom=M, tol=1e-11)
    print(L, M, nE, queue, flush=True)
    lam, infos, rc = cbs.solve_batched([s], E, [V], prm)
    assert rc == 0
    for e in range(nE):
        one, _, _, info, _ = s.solve(E[e], V, prm, want_vectors=False)
        assert abs(infos[e].sigma_first - info.sigma_first) <= 1e-8 * info.sigma_first
        assert len(lam[0][e]) == len(one) > 0
        assert qep.match_sets(lam[0][e], one) <= 1e-8

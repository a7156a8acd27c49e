"""A Hankel SVD that runs out of sweeps is reported, not used: its singular values would decide the rank.
Held to one sweep, where these matrices need six or more (the default is 60), at the orders of both forms (one
workgroup up to 64, column blocks beyond), alone and in a batch, and solved again at the default."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M", [(8, 8), (16, 8), (17, 8)])
def test_too_few_sweeps_are_an_error(cuda, monkeypatch, L, M):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(8, 8, 12, 0.4, 4, 6, 971, 972, with_proj=True, r_c=1.1)
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 973)).to(cuda)
    s, prm = cbs.System.from_workload(sysw), cbs.default_params(n_rhs=L, n_mom=M, tol=1e-11)
    print(L, M, flush=True)
    monkeypatch.setenv("CBS_SVD_SWEEPS", "1")
    with pytest.raises(cbs.CbsError, match="did not converge"):
        s.solve(1.3, V, prm, want_vectors=False)
    lam, infos, rc = cbs.solve_batched([s], np.array([1.2, 1.3]), [V], prm)
    assert rc == cbs.CBS_EEIG and [i.status for i in infos] == [cbs.CBS_EEIG] * 2 and all(len(q) == 0 for q in lam[0])
    monkeypatch.delenv("CBS_SVD_SWEEPS")
    lam, _, _, _, rc = s.solve(1.3, V, prm, want_vectors=False)
    assert rc == 0 and len(lam) > 0

"""The tall products of the extraction on either side of their change of kernel (points times columns =
1,250,000), with inner dimensions that are no multiple of the rows requested at a time (8, then 2) and
columns that are no multiple of a thread's (4, then 16): the orthonormal basis of the moments' span, from
the solve's dump of its arrays.  Below the spectrum the annulus is empty and every direction is kept.

Tolerance: the shifted Cholesky QR's last pass leaves m eps times a modest factor (1e-14 at m = 15), and its
projection reproduces the moments to their own rounding times the same: 1e-12 is taken for both."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,L", [(12, 15), (32, 15), (40, 15), (40, 17)])
def test_basis_spans_the_moments(cuda, monkeypatch, tmp_path, nz, L):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(48, 48, nz, 0.4, 2, 6, 731)
    monkeypatch.setenv("CBS_DUMP", str(tmp_path))
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 732)).to(cuda)
    print(sysw.n * L, flush=True)
    info = cbs.System.from_workload(sysw).solve(-3.0, V, cbs.default_params(n_rhs=L, n_mom=1, n_q=4), want_vectors=False)[3]
    assert info.rank == L
    Q = np.fromfile(tmp_path / "Q.bin", dtype=np.complex128).reshape(L, -1)
    S = np.fromfile(tmp_path / "S.bin", dtype=np.complex128).reshape(2, L, -1)[0]
    assert np.abs(Q.conj() @ Q.T - np.eye(L)).max() <= 1e-12
    assert np.linalg.norm(S - (S @ Q.conj().T) @ Q) <= 1e-12 * np.linalg.norm(S)

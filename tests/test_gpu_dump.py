"""The dump of the extraction's intermediate arrays: U where the factorisation has it, T W = U Sigma, and no
file of that name where only the right vectors are computed.

Tolerance: one-sided Jacobi is backward stable, with an error of a modest multiple of n eps |T| (n = 16:
4e-15); 1e-12 |T| is taken, as for the singular values."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extraction", ["CBS_RR", "CBS_HANKEL"])
def test_left_vectors_only_where_they_are_computed(cuda, monkeypatch, tmp_path, extraction):
    import torch
    import paper_1709_09347_amd as cbs
    L, M = 4, 4
    n = L * M
    sysw = W.config(1).systems[0]
    monkeypatch.setenv("CBS_DUMP", str(tmp_path))
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 71)).to(cuda)
    prm = cbs.default_params(n_rhs=L, n_mom=M, extraction=getattr(cbs, extraction))
    cbs.System.from_workload(sysw).solve(0.3, V, prm, want_vectors=False)
    read = lambda name: np.fromfile(tmp_path / f"{name}.bin", dtype=np.complex128).reshape(n, n).T  # noqa: E731
    assert (tmp_path / "U.bin").exists() == (extraction == "CBS_HANKEL")
    if extraction == "CBS_HANKEL":
        T, U, Wv = read("T"), read("U"), read("W")
        sg, perm = np.fromfile(tmp_path / "sigma.bin"), np.fromfile(tmp_path / "perm.bin", dtype=np.int32)
        assert np.abs(T @ Wv[:, perm] - U[:, perm] * sg).max() <= 1e-12 * sg[0]

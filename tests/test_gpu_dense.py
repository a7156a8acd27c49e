"""The small dense kernels of the extraction on what a solve hands them: right singular vectors of the
Hankel matrix at the orders where the kernels change (one column a lane up to 64, two up to 128, the
copy in global memory beyond; one workgroup or column blocks), and the reduced eigenproblem on
either side of the one-wave kernel's order (64), read from the solve's dump of its intermediate arrays.

Tolerances: one-sided Jacobi and Householder QR are backward stable, with an error of a modest
multiple of n eps |A| (n = 256: 6e-14); 1e-12 |A| is taken for the singular values and W's orthogonality,
1e-11 |M| for the distance of M - theta I from singular (QR adds its 60 n sweeps' worth of eps at most)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _dump(cuda, monkeypatch, tmp_path, E, L, M, **prm):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.config(1).systems[0]
    monkeypatch.setenv("CBS_DUMP", str(tmp_path))
    s = cbs.System.from_workload(sysw)
    V = torch.from_numpy(W.make_rhs(sysw.n, L, 71)).to(cuda)
    print(E, L, M, flush=True)
    out = s.solve(E, V, cbs.default_params(n_rhs=L, n_mom=M, **prm), want_vectors=False)

    def read(name, cols=None, dtype=np.complex128):
        a = np.fromfile(tmp_path / f"{name}.bin", dtype=dtype)
        return a if cols is None else a.reshape(cols, -1).T

    return out, read


@pytest.mark.parametrize("L,M", [(1, 1), (3, 1), (4, 4), (8, 8), (13, 5), (16, 8), (43, 3), (16, 16)])
def test_right_singular_vectors(cuda, monkeypatch, tmp_path, L, M):
    n = L * M
    _, read = _dump(cuda, monkeypatch, tmp_path, 0.3, L, M)
    T, Wv, sg, perm = read("T", n), read("W", n), read("sigma", dtype=np.float64), read("perm", dtype=np.int32)
    ref = np.linalg.svd(T, compute_uv=False)
    assert sorted(perm) == list(range(n))
    assert np.abs(sg - ref).max() <= 1e-12 * ref[0]
    Ws = Wv[:, perm]
    kept = sg > 1e-13 * sg[0]
    assert np.abs(Ws[:, kept].conj().T @ Ws[:, kept] - np.eye(kept.sum())).max() <= 1e-12
    assert np.abs(np.linalg.norm(T @ Ws, axis=0) - sg).max() <= 1e-12 * ref[0]


@pytest.mark.parametrize("L,M", [(2, 1), (8, 2), (8, 4), (11, 3)])
def test_reduced_eigenproblem(cuda, monkeypatch, tmp_path, L, M):
    # an empty annulus keeps all L M directions, so the linearised problem has order 2 L M: 4, 32, 64, 66
    out, read = _dump(cuda, monkeypatch, tmp_path, -3.0, L, M)
    n = 2 * out[3].rank
    assert n == 2 * L * M
    A, theta = read("Minv", n), read("theta")
    scale = np.linalg.norm(A, 2)
    for t in theta:
        assert np.linalg.svd(A - t * np.eye(n), compute_uv=False)[-1] <= 1e-11 * scale
    assert abs(theta.sum() - np.trace(A)) <= 1e-11 * scale * n

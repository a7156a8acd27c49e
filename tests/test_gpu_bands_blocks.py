"""Bands in blocks at the orders where the Cholesky factorisation of the block changes kernel: 6 and 32
vectors (256 threads), 34 and 96 (1024 threads), 98 (global memory), against dense eigenvalues of H(k).

Tolerance: the eigenvalues of a Hermitian matrix lie within the residual norm of the Ritz values, here
tol (|theta| + 1) with tol = 1e-10; the dense solution's own error is N eps |H| = 504 x 2.2e-16 x 100
= 1.1e-11.  The vectors are orthonormal after two unshifted passes to m eps times a modest factor: 1e-12."""
import numpy as np
import pytest

import workloads as W
from oracle import ham, qep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 25, 26, 76, 78])
def test_block_orders(cuda, nb):
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(7, 8, 9, 0.45, 4, 5, 901, 902, with_proj=True, r_c=1.3)
    h0, hp, hm = ham.build(sysw).blocks_dense()
    a = sysw.nz * sysw.h
    k = 0.37 * np.pi / a
    print(nb, sysw.n, flush=True)
    eps, res, vecs, _, rc = cbs.System.from_workload(sysw).bands([k], nb, tol=1e-10, want_vectors=True)
    assert rc == 0
    want = qep.bands_dense(h0, hp, hm, k, a, nb)
    assert np.abs(eps[0] - want).max() <= 1.1e-10 * (np.abs(want).max() + 1) + 1.1e-11
    X = vecs[0].cpu().numpy()
    assert np.abs(X.conj() @ X.T - np.eye(nb)).max() <= 1e-12

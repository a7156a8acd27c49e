"""Small cells with more runs than the chip has CUs, where two runs share a CU (two points a thread), with
the projectors' tables in LDS and, where twice that would not fit, without: every run against the same
run solved in a batch of its own, which takes one point a thread, and some against the oracle.

Tolerance: the same recurrences with the sums added in another order, 12 steps from the start, where
the residual has not fallen far: 1e-10 relative, the bar that the large cells' iterates are held to."""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cell", [(8, 8, 9, 4, 5, 1.1), (8, 8, 16, 6, 12, 1.4), (16, 8, 8, 8, 0, 0.0), (8, 8, 8, 4, 4, 1.0)])
def test_two_runs_per_cu(cuda, cell):
    import torch
    import paper_1709_09347_amd as cbs
    nx, ny, nz, fd, na, rc = cell
    sysw = W.make_system(nx, ny, nz, 0.4, fd, na or 3, 951, 952, with_proj=rc > 0, r_c=rc or 1.0)
    z = 1.6 * np.exp(2j * np.pi * (np.arange(33) + 0.5) / 33)
    V = W.make_rhs(sysw.n, 8, 953)
    print(cell, flush=True)
    s, prm = cbs.System.from_workload(sysw), cbs.default_params(max_iter=12, tol=1e-14)
    many = s.bicg(0.3, z, torch.from_numpy(V).to(cuda), prm)
    y, yt = many[0].cpu().numpy(), many[1].cpu().numpy()
    for lo in range(0, 33, 11):
        few = s.bicg(0.3, z[lo:lo + 11], torch.from_numpy(V).to(cuda), prm)
        for a, b in ((y, few[0].cpu().numpy()), (yt, few[1].cpu().numpy())):
            d = np.linalg.norm(a[lo:lo + 11] - b, axis=2) / np.linalg.norm(b, axis=2)
            assert d.max() <= 1e-10
        assert np.array_equal(many[2][lo:lo + 11], few[2])
    H = ham.build(sysw)
    for j in (0, 17):
        want, wantd = _steps(H, z[j], V[3], 12)
        assert np.linalg.norm(y[j, 3] - want) <= 1e-10 * np.linalg.norm(want)
        assert np.linalg.norm(yt[j, 3] - wantd) <= 1e-10 * np.linalg.norm(wantd)


def _steps(H, z, v, n):
    """n steps of BiCG with the dual, as the paper's Sec. 3.2 pairs the systems, on the oracle's operator."""
    zd = 1 / np.conj(z)
    r, rt = v.copy(), v.copy()
    p, pt = r.copy(), rt.copy()
    x, xt = np.zeros_like(v), np.zeros_like(v)
    rho = np.vdot(rt, r)
    for _ in range(n):
        q, qt = H.apply(z, p, 0.3), H.apply(zd, pt, 0.3)
        a = rho / np.vdot(pt, q)
        x, xt = x + a * p, xt + np.conj(a) * pt
        r, rt = r - a * q, rt - np.conj(a) * qt
        new = np.vdot(rt, r)
        b, rho = new / rho, new
        p, pt = r + b * p, rt + np.conj(b) * pt
    return x, xt

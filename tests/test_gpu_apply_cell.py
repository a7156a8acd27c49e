"""GPU: the operator on cells that one workgroup takes, at the edges of that rule.

k_ap_cell takes cells of at most 1024 points with 1 to 12 atoms and at most 2560 ball entries; the
cells here lie on and just past each of those lines, against the oracle's sparse operator.  The
tolerance is the operator's own: a point's value is a sum of a few hundred products, so 1e-13 of
the largest term in complex128 and 2e-6 in complex64.
"""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu

CELLS = {
    # name: (nx, ny, nz, h, points across the stencil, atoms, cut-off radius)
    "1024 points": (8, 8, 16, 0.4, 8, 6, 1.1),
    "1040 points": (8, 10, 13, 0.4, 8, 6, 1.1),
    "fewer points than a wave": (3, 3, 5, 0.5, 2, 2, 0.7),
    "rows shorter than the stencil": (3, 2, 9, 0.5, 8, 3, 0.6),
    "12 atoms": (7, 9, 11, 0.4, 6, 12, 0.9),
    "13 atoms": (7, 9, 11, 0.4, 6, 13, 0.9),
    "many entries": (10, 10, 10, 0.4, 4, 9, 1.6),
    "too many entries": (10, 10, 10, 0.4, 4, 11, 1.7),
}


@pytest.mark.parametrize("name", list(CELLS))
def test_cells_at_the_edges(cuda, name):
    import torch
    import paper_1709_09347_amd as cbs
    nx, ny, nz, h, fd, atoms, rc = CELLS[name]
    sysw = W.make_system(nx, ny, nz, h, fd, atoms, 401, 402, with_proj=True, r_c=rc)
    H, s, E = ham.build(sysw), cbs.System.from_workload(sysw), 0.3
    for nv, dtype, tol in ((1, np.complex128, 1e-13), (66, np.complex128, 1e-13), (3, np.complex64, 2e-6)):
        rng = np.random.default_rng(nv)
        x = (rng.standard_normal((nv, sysw.n)) + 1j * rng.standard_normal((nv, sysw.n))).astype(dtype)
        z = np.exp(rng.uniform(-0.7, 0.7, nv) + 1j * rng.uniform(-np.pi, np.pi, nv))
        xt = torch.from_numpy(x).to(cuda)
        print(name, nv, np.dtype(dtype).name, flush=True)
        y = s.apply(E, z, xt).cpu().numpy().astype(np.complex128)
        s.apply(E, z, xt, y=xt)   # in place: every vector is read before its first point is written
        assert np.array_equal(xt.cpu().numpy().astype(np.complex128), y)
        x = x.astype(np.complex128)
        want = np.stack([H.apply(z[v], x[v], E) for v in range(nv)])
        scale = np.abs(want).max(axis=1, keepdims=True) + 50 * np.abs(x).max(axis=1, keepdims=True)
        assert (np.abs(y - want) / scale).max() <= tol

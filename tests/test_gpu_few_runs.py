"""BiCG on cells past the one-workgroup path with too few runs to fill the chip: the stencil marches
in z segments (down to one plane, shorter than the stencil's half-width), the projections may share its
launch (one or two items to a workgroup) and the update takes short chunks.  Against the oracle's recurrence after a fixed number of steps, primal and dual, for staged
planes that fit the prefetch registers and planes that don't.

Tolerance: the same recurrences with the sums added in another order, 12 steps from the start, where
the residual has not fallen far: 1e-10 relative, the bar that the large cells' iterates are held to."""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu

# nx, ny, nz, order, atoms, ball radius, nodes, right-hand sides
CELLS = {
    "one_run_planes": (16, 17, 9, 8, 0, 0.0, 1, 1),
    "odd_segments": (23, 19, 17, 6, 9, 1.7, 3, 5),
    "ragged_tile_unstaged_ahead": (130, 7, 11, 8, 4, 1.1, 2, 2),
    "order_2": (21, 20, 13, 2, 5, 1.6, 2, 3),
    "order_4_two_segments": (24, 24, 10, 4, 6, 1.6, 3, 30),
    "two_items_a_workgroup": (32, 17, 12, 6, 7, 1.6, 3, 3),
    "wide_ball": (18, 18, 13, 6, 3, 2.5, 1, 3),
}


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


@pytest.mark.parametrize("name", sorted(CELLS))
def test_iterates_match_the_oracle(cuda, monkeypatch, name):
    import torch
    import paper_1709_09347_amd as cbs
    nx, ny, nz, fd, na, rc, nodes, L = CELLS[name]
    monkeypatch.setenv("CBS_RUN_WG", "0")   # the general path, whatever the size
    sysw = W.make_system(nx, ny, nz, 0.4, fd, na or 3, 711, 712, with_proj=rc > 0, r_c=rc or 1.0)
    z = np.array([2.0 * np.exp(0.4j), 1.7 * np.exp(2.3j), 0.6 * np.exp(-1.1j)])[:nodes]
    V = W.make_rhs(sysw.n, L, 713)
    print(name, sysw.n, flush=True)
    s = cbs.System.from_workload(sysw)
    out = s.bicg(0.3, z, torch.from_numpy(V).to(cuda), cbs.default_params(max_iter=12, tol=1e-14))
    torch.cuda.synchronize()
    y, yt, it = out[0].cpu().numpy(), out[1].cpu().numpy(), out[2]
    H = ham.build(sysw)
    for j in range(nodes):
        for l in range(0, L, max(1, L // 3)):
            want, wantd = _steps(H, z[j], V[l], 12)
            assert it[j, l] == 12
            assert np.linalg.norm(y[j, l] - want) <= 1e-10 * np.linalg.norm(want)
            assert np.linalg.norm(yt[j, l] - wantd) <= 1e-10 * np.linalg.norm(wantd)

"""A value of x that is not finite reaches the points whose sums it enters and no others: its stencil
neighbours and the balls that hold it.  On the cells that one workgroup takes, in separate launches and
with two vector groups a workgroup, whose matrix products work on blocks of 16 points and multiply
the zeros of those outside a ball.

Tolerance: away from those points the sums are the same ones, at most in another order, so the
operator's own bar holds against the run with a finite value in the place: 1e-13 of the largest term in
complex128 and 2e-6 in complex64.  The other vectors of the block take the same path in both: equal bits."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# nx, ny, nz, order, atoms, ball radius, vectors
CELLS = {
    "one workgroup": (8, 8, 12, 4, 5, 1.1, 3),
    "separate launches": (19, 17, 13, 6, 7, 1.5, 3),
    "two vector groups": (41, 40, 41, 4, 12, 2.0, 16),
}


def _reach(sysw, p, n0):
    """Points whose sums x[n0] enters."""
    nx, ny, nz = sysw.nx, sysw.ny, sysw.nz
    ix, iy, iz = n0 % nx, n0 // nx % ny, n0 // (nx * ny)
    out = {n0}
    for j in range(-p, p + 1):
        out |= {(ix + j) % nx + nx * (iy + ny * iz), ix + nx * ((iy + j) % ny + ny * iz), ix + nx * (iy + ny * ((iz + j) % nz))}
    pr = sysw.proj
    for a in range(pr.n_atoms):
        ball = pr.ball_idx[pr.ball_off[a]:pr.ball_off[a + 1]]
        if n0 in ball:
            out |= set(ball.tolist())
    return np.array(sorted(out))


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("name", list(CELLS))
def test_a_value_that_is_not_finite_stays_in_its_balls(cuda, name, dtype, value):
    import torch
    import paper_1709_09347_amd as cbs
    nx, ny, nz, fd, atoms, rc, nv = CELLS[name]
    sysw = W.make_system(nx, ny, nz, 0.4, fd, atoms, 821, 822, with_proj=True, r_c=rc)
    s = cbs.System.from_workload(sysw)
    rng = np.random.default_rng(823)
    x = (rng.standard_normal((nv, sysw.n)) + 1j * rng.standard_normal((nv, sysw.n))).astype(dtype)
    z = np.exp(rng.uniform(-0.7, 0.7, nv) + 1j * rng.uniform(-np.pi, np.pi, nv))
    n0, v0 = int(sysw.proj.ball_idx[sysw.proj.ball_off[2] + 3]), 1
    bad = x.copy()
    bad[v0, n0] = value
    reach = _reach(sysw, fd // 2, n0)
    away = np.setdiff1d(np.arange(sysw.n), reach)
    tol = 1e-13 if dtype == np.complex128 else 2e-6
    print(name, np.dtype(dtype).name, value, len(reach), flush=True)
    ways = [lambda q: s.apply(0.3, z, q)]
    if dtype == np.complex128:
        ways.append(lambda q: s.apply_parts(0.3, z, 1 - z, 0.5 * z, q))
    for way in ways:
        want = way(torch.from_numpy(x).to(cuda)).cpu().numpy()
        got = way(torch.from_numpy(bad).to(cuda)).cpu().numpy()
        others = np.arange(nv) != v0
        assert np.array_equal(got[others], want[others])
        assert not np.isfinite(got[v0, reach]).any()
        scale = np.abs(want[v0]).max() + 150 * np.abs(x[v0]).max()
        assert np.abs(got[v0, away] - want[v0, away]).max() <= tol * scale

"""Restarts, precision changes and replacements of the launch-per-step iteration, driven on purpose, with
the solution's pending directions between them: on a small cell with few runs, where x takes each direction
on the next iteration, and in a batch that fills the chip, where it takes two on every second one and
a run may be marked with one pending or with two.

Every run must reach tol with solutions whose residuals, primal and dual, recomputed by the oracle, meet
1e-10, as for the other restart tests.  A pending term that a replacement lost, or added twice, would
show in the residuals right after it, by as much as the residual itself: they are compared between the two
forms of the iteration, run by run.  Tolerance there: the vectors of the complex64 phase are rounded to
6e-8, |P| is about 100 and |x| up to 10 |b|, so the residuals that a replacement computes anew differ by about
1e-4 |b|; the recurrences before it go by scalars of the same accuracy at residuals above 1e-2, a per cent,
and two are taken."""
import numpy as np
import pytest

import workloads as W
from oracle import ham, ss

pytestmark = pytest.mark.gpu

CELLS = {
    "few runs": lambda: (W.config(1).systems[0], [0, 10, 16, 31], 4),
    "full batch": lambda: (W.make_system(32, 32, 6, 0.4, 6, 8, 981, 982, with_proj=True, r_c=1.1), list(range(32)) + [0], 8),
}


def _case(cuda, monkeypatch, name):
    import torch
    import paper_1709_09347_amd as cbs
    monkeypatch.setenv("CBS_RUN_WG", "0")   # the general path, whatever the size
    sysw, sel, L = CELLS[name]()
    z1, _, z2, _ = ss.quadrature(0.5, 32)
    V = W.make_rhs(sysw.n, L, 3)
    return cbs.System.from_workload(sysw), ham.build(sysw), z1[sel], z2[sel], V, torch.from_numpy(V).to(cuda)


def _check(H, z, zd, V, out):
    Y, Yt, iters, relres, info, rc = out[:6]
    assert rc == 0 and relres.max() <= 1e-10
    order = np.argsort(iters, axis=None)
    some = np.unravel_index(np.unique(np.concatenate([order[:2], order[-6:], order[::max(1, len(order) // 16)]])), iters.shape)
    for j, l in zip(*some):
        y, yt, nv = Y[j, l].cpu().numpy(), Yt[j, l].cpu().numpy(), np.linalg.norm(V[l])
        assert np.linalg.norm(V[l] - H.apply(z[j], y, 0.3)) <= 1e-10 * nv, (j, l)
        assert np.linalg.norm(V[l] - H.apply(zd[j], yt, 0.3)) <= 1e-10 * nv, (j, l)


@pytest.mark.parametrize("name", list(CELLS))
@pytest.mark.parametrize("precision", [0, 1])
def test_restart_of_diverging_runs(cuda, monkeypatch, name, precision):
    import paper_1709_09347_amd as cbs
    s, H, z, zd, V, Vt = _case(cuda, monkeypatch, name)
    print(name, precision, flush=True)
    prm = cbs.default_params(precision=precision, max_iter=20000)
    out = s.bicg(0.3, z, Vt, prm, history=(1, 2000))
    assert out[5] == 0 and out[4].restarts == 0
    # half the largest rise of a residual above its running minimum sends at least that run to a restart
    r = np.asarray(out[6]).reshape(2000, -1, 2).max(axis=2)
    rise = 1.0
    for run in range(r.shape[1]):
        x = r[:, run][r[:, run] > 0]
        rise = max(rise, float(np.max(x[20:] / np.minimum.accumulate(x)[20:])))
    monkeypatch.setenv("CBS_DIVERGE_FACTOR", f"{rise / 2:.6g}")
    out = s.bicg(0.3, z, Vt, prm)
    print(f"largest rise {rise:.3g}; restarts {out[4].restarts}, iterations {out[2].min()}-{out[2].max()}", flush=True)
    assert out[4].restarts > 0
    _check(H, z, zd, V, out)


@pytest.mark.parametrize("name", list(CELLS))
@pytest.mark.parametrize("window", [1, 2, 5])
def test_replacements_in_complex64(cuda, monkeypatch, name, window):
    # with a short window every complex64 run is replaced again and again, on even and on odd iterations,
    # until it restarts in complex128
    import paper_1709_09347_amd as cbs
    s, H, z, zd, V, Vt = _case(cuda, monkeypatch, name)
    print(name, window, flush=True)
    out = s.bicg(0.3, z, Vt, cbs.default_params(precision=cbs.CBS_MIXED, inner_tol=1e-3, lo_window=window, max_iter=20000))
    print(f"restarts {out[4].restarts}, iterations {out[2].min()}-{out[2].max()}", flush=True)
    assert out[4].restarts > 0
    _check(H, z, zd, V, out)


@pytest.mark.parametrize("window", [1, 2, 5, 6, 15, 16, 29, 30])
def test_residuals_after_replacements_agree_between_the_forms(cuda, monkeypatch, window):
    import paper_1709_09347_amd as cbs
    s, H, z, zd, V, Vt = _case(cuda, monkeypatch, "full batch")
    K = window + 24
    prm = cbs.default_params(precision=cbs.CBS_MIXED, inner_tol=0.5, lo_window=window, max_iter=20000)
    print(window, flush=True)
    many = np.asarray(s.bicg(0.3, z, Vt, prm, history=(1, K))[6]).reshape(K, len(z), -1)
    for j in (0, 13, 31):
        few = np.asarray(s.bicg(0.3, z[j:j + 1], Vt, prm, history=(1, K))[6]).reshape(K, -1)
        d = np.abs(many[:, j] - few)
        print(j, "smallest residual", few.min(), "of the tolerance", (d / (2e-2 * few + 1e-4)).max(), flush=True)
        assert np.isfinite(few).all() and np.all(d <= 2e-2 * few + 1e-4)

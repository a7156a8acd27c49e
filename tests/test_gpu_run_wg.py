"""Small cells, where one workgroup carries a run through its iterations: against the oracle's BiCG
after a fixed number of steps, primal and dual, at the edges of what a thread owns (one, two and
eight points) and of the cells the path takes; unfinished runs carried from launch to launch must
not change a bit, nor their histories; and the launch-per-step path gives the same counts.

Tolerance: the same recurrences with the sums added in another order, 12 steps from the start, where
the residual has not fallen far: 1e-10 relative, the bar that the large cells' iterates are held to."""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu

CELLS = {
    "one_wave": (3, 2, 5, 2, 0, 0.0),
    "edge_1024": (8, 8, 16, 4, 5, 0.0),
    "past_1024": (5, 5, 41, 8, 4, 1.4),
    "proj_768": (8, 8, 12, 6, 6, 1.5),
    "edge_2048": (16, 8, 16, 8, 7, 1.6),
    "past_2048": (13, 9, 18, 6, 9, 1.7),
    "edge_4096": (16, 16, 16, 8, 12, 2.0),
}


def _case(name):
    nx, ny, nz, fd, na, rc = CELLS[name]
    s = W.make_system(nx, ny, nz, 0.4, fd, na or 3, 611, 612, with_proj=rc > 0, r_c=rc or 1.0)
    z = np.array([2.0 * np.exp(0.4j), 1.7 * np.exp(2.3j), 0.6 * np.exp(-1.1j)])
    return s, z, W.make_rhs(s.n, 2, 613)


def _bicg(cuda, sysw, z, V, **prm):
    import torch
    import paper_1709_09347_amd as cbs
    s = cbs.System.from_workload(sysw)
    out = s.bicg(0.3, z, torch.from_numpy(V).to(cuda), cbs.default_params(**prm), history=(1, 64))
    torch.cuda.synchronize()
    return out[0].cpu().numpy(), out[1].cpu().numpy(), out[2], out[3], out[6]


@pytest.mark.parametrize("name", sorted(CELLS))
def test_iterates_match_the_oracle(cuda, name):
    sysw, z, V = _case(name)
    H = ham.build(sysw)
    print(name, sysw.n, flush=True)
    y, yt, it, _, _ = _bicg(cuda, sysw, z, V, max_iter=12, tol=1e-14)
    for j in range(len(z)):
        for l in range(V.shape[0]):
            want, wantd = _steps(H, z[j], V[l], 12)
            assert it[j, l] == 12
            assert np.linalg.norm(y[j, l] - want) <= 1e-10 * np.linalg.norm(want)
            assert np.linalg.norm(yt[j, l] - wantd) <= 1e-10 * np.linalg.norm(wantd)


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


@pytest.mark.parametrize("name", ["one_wave", "proj_768", "past_1024", "past_2048"])
def test_launch_boundaries_change_nothing(cuda, monkeypatch, name):
    sysw, z, V = _case(name)
    ref = _bicg(cuda, sysw, z, V, max_iter=60, tol=1e-9)
    monkeypatch.setenv("CBS_RUN_WG", "7")
    got = _bicg(cuda, sysw, z, V, max_iter=60, tol=1e-9)
    for a, b in zip(ref, got):
        assert np.array_equal(a, b, equal_nan=True)
    monkeypatch.setenv("CBS_RUN_WG", "0")
    gen = _bicg(cuda, sysw, z, V, max_iter=12, tol=1e-14)
    monkeypatch.delenv("CBS_RUN_WG")
    here = _bicg(cuda, sysw, z, V, max_iter=12, tol=1e-14)
    assert np.array_equal(gen[2], here[2])
    assert np.linalg.norm(gen[0] - here[0]) <= 1e-10 * np.linalg.norm(gen[0])


def test_zero_and_nonfinite_right_hand_sides(cuda, monkeypatch):
    import torch
    import paper_1709_09347_amd as cbs
    sysw, z, V = _case("proj_768")
    V[0] = 0
    s = cbs.System.from_workload(sysw)
    out = {}
    for mode in ("1024", "0"):
        monkeypatch.setenv("CBS_RUN_WG", mode)
        y, yt, it, rel, info, rc = s.bicg(0.3, z, torch.from_numpy(V).to(cuda), cbs.default_params(tol=1e-9))
        assert torch.all(y[:, 0] == 0) and torch.all(yt[:, 0] == 0) and np.all(it[:, 0] == 0)
        W1 = V.copy()
        W1[1, 5] = np.inf
        _, _, it2, _, info2, rc2 = s.bicg(0.3, z, torch.from_numpy(W1).to(cuda), cbs.default_params(tol=1e-9))
        out[mode] = (rc, rc2, it2.tolist(), info2.restarts)
    assert out["1024"] == out["0"]

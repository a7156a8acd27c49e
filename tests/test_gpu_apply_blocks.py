"""The vector-major operator kernels where their splits can go wrong: block sizes around the
vector groups (4 in the bra, 8 in the ket, 64 per launch), rows that do not divide into tiles,
planes that do not divide into z segments, a cell too wide for the pipelined staging and for two
LDS planes, one plane per half-width, point groups with more keys than one wave lists (256), an
output that is its own input.  Against the oracle's sparse operator.

Tolerance: a term of P x passes through at most 2p + 10 + n_keys roundings (the z queue, the in-plane
sum, the phases, the ket), each at most eps of the sum of the terms' moduli, which is below 50 max|x|
+ max|Px| here: 100 eps = 2.3e-14 in complex128 (1e-13 taken), 100 eps = 1.2e-5 in complex64 at worst
and sqrt(100) eps = 1.2e-6 for independent roundings (2e-6 taken, as for the other operator tests)."""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu

CELLS = {
    "ragged": lambda: W.make_system(7, 11, 13, 0.45, 8, 4, 301, 302, with_proj=True, r_c=1.6),
    "ragged, several workgroups": lambda: W.make_system(9, 11, 13, 0.45, 8, 4, 301, 302, with_proj=True, r_c=1.6),
    "wide": lambda: W.make_system(200, 9, 6, 0.5, 8, 3, 303, 304, with_proj=True, r_c=1.2),
    "thin": lambda: W.make_system(1, 1, 4, 0.5, 8, 2, 305),
    "crowded": lambda: W.make_system(8, 8, 12, 0.4, 4, 300, 306, 307, with_proj=True, r_c=2.0),
    "local": lambda: W.make_system(61, 23, 10, 0.4, 2, 9, 308),
}


def _run(cuda, name, nv, dtype, how):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = CELLS[name]()
    H = ham.build(sysw)
    rng = np.random.default_rng(nv)
    x = (rng.standard_normal((nv, sysw.n)) + 1j * rng.standard_normal((nv, sysw.n))).astype(dtype)
    z = np.exp(rng.uniform(-0.7, 0.7, nv) + 1j * rng.uniform(-np.pi, np.pi, nv))
    E, s = 0.3, cbs.System.from_workload(sysw)
    xt = torch.from_numpy(x).to(cuda)
    x = x.astype(np.complex128)
    print(name, nv, np.dtype(dtype).name, how, flush=True)
    if how == "parts":
        c = rng.standard_normal((3, nv)) + 1j * rng.standard_normal((3, nv))
        y = s.apply_parts(E, c[0], c[1], c[2], xt)
        one = [H.apply(w, x[v], E) for v in range(nv) for w in (1, -1, 1j)]
        # H0 - E, H+ and H- from P at three points of the unit circle
        p1, pm, pi = (np.stack(one[k::3]) for k in range(3))
        a0 = 0.5 * (p1 + pm)
        s1, s2 = 0.5 * (p1 - pm), (pi - a0) / 1j
        want = c[0][:, None] * a0 + c[1][:, None] * 0.5 * (s1 + s2) + c[2][:, None] * 0.5 * (s1 - s2)
        scale_c = np.abs(c).max() * 3
    else:
        y = s.apply(E, z, xt, y=xt) if how == "inplace" else s.apply(E, z, xt)
        want = np.stack([H.apply(z[v], x[v], E) for v in range(nv)])
        scale_c = 1.0
    y = y.cpu().numpy().astype(np.complex128)
    scale = np.abs(want).max(axis=1, keepdims=True) + 50 * scale_c * np.abs(x).max(axis=1, keepdims=True)
    err = (np.abs(y - want) / scale).max()
    assert err <= (1e-13 if dtype == np.complex128 else 2e-6), err


@pytest.mark.parametrize("nv", [1, 3, 4, 9, 17, 65])
def test_block_sizes(cuda, nv):
    _run(cuda, "ragged", nv, np.complex128, "apply")
    _run(cuda, "ragged", nv, np.complex64, "apply")
    _run(cuda, "ragged", nv, np.complex128, "parts")


@pytest.mark.parametrize("nv", [1, 4, 9, 17, 65])
def test_block_sizes_in_separate_launches(cuda, nv):
    # past 1024 points the three parts are launches of their own
    _run(cuda, "ragged, several workgroups", nv, np.complex128, "apply")
    _run(cuda, "ragged, several workgroups", nv, np.complex64, "apply")
    _run(cuda, "ragged, several workgroups", nv, np.complex128, "parts")


@pytest.mark.parametrize("name", ["wide", "thin", "crowded", "local"])
@pytest.mark.parametrize("how", ["apply", "parts", "inplace"])
def test_cells(cuda, name, how):
    _run(cuda, name, 5, np.complex128, how)
    if how != "parts":
        _run(cuda, name, 2, np.complex64, how)

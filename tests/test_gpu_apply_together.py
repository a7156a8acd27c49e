"""The operator's projection in one launch with its local part: several items (an atom and its
vectors) per workgroup, a last workgroup with one item too few, and the atom counts on either side of
where the launches part.  Against the oracle's sparse operator.

Tolerance: a term of P x passes through at most 2p + 10 + n_keys roundings (the z queue, the in-plane
sum, the phases, the ket), each at most eps of the sum of the terms' moduli, which is below 50 max|x|
+ max|Px| here: 100 eps = 2.3e-14 in complex128 (1e-13 taken), 100 eps = 1.2e-5 in complex64 at worst
and sqrt(100) eps = 1.2e-6 for independent roundings (2e-6 taken, as for the other operator tests)."""
import numpy as np
import pytest

import workloads as W
from oracle import ham

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("atoms,nv", [(513, 2), (576, 1), (577, 2), (260, 3), (289, 4), (577, 5)])
def test_items_shared_by_a_workgroup(cuda, atoms, nv, dtype):
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(33, 30, 7, 0.4, 4, atoms, 801, 802, with_proj=True, r_c=0.7)
    H = ham.build(sysw)
    rng = np.random.default_rng(803)
    x = (rng.standard_normal((nv, sysw.n)) + 1j * rng.standard_normal((nv, sysw.n))).astype(dtype)
    z = np.exp(rng.uniform(-0.7, 0.7, nv) + 1j * rng.uniform(-np.pi, np.pi, nv))
    print(atoms, nv, np.dtype(dtype).name, flush=True)
    y = cbs.System.from_workload(sysw).apply(0.3, z, torch.from_numpy(x).to(cuda)).cpu().numpy().astype(np.complex128)
    want = np.stack([H.apply(z[v], x[v].astype(np.complex128), 0.3) for v in range(nv)])
    scale = np.abs(want).max(axis=1, keepdims=True) + 50 * np.abs(x).max(axis=1, keepdims=True)
    err = (np.abs(y - want) / scale).max()
    assert err <= (1e-13 if dtype == np.complex128 else 2e-6), err


@pytest.mark.parametrize("dtype", [np.complex128, np.complex64])
@pytest.mark.parametrize("nv", [9, 16, 31])
def test_two_vector_groups_a_workgroup(cuda, nv, dtype):
    # the product with the projectors takes two groups of eight vectors a workgroup from 2048
    # (point group, vector group) pairs on: 65536 points make 1024 point groups
    import torch
    import paper_1709_09347_amd as cbs
    sysw = W.make_system(41, 40, 41, 0.4, 4, 12, 811, 812, with_proj=True, r_c=2.0)
    H = ham.build(sysw)
    rng = np.random.default_rng(813)
    x = (rng.standard_normal((nv, sysw.n)) + 1j * rng.standard_normal((nv, sysw.n))).astype(dtype)
    z = np.exp(rng.uniform(-0.7, 0.7, nv) + 1j * rng.uniform(-np.pi, np.pi, nv))
    print(nv, np.dtype(dtype).name, flush=True)
    y = cbs.System.from_workload(sysw).apply(0.3, z, torch.from_numpy(x).to(cuda)).cpu().numpy().astype(np.complex128)
    for v in (0, 7, 8, nv - 1):
        want = H.apply(z[v], x[v].astype(np.complex128), 0.3)
        err = np.abs(y[v] - want).max() / (np.abs(want).max() + 50 * np.abs(x[v]).max())
        assert err <= (1e-13 if dtype == np.complex128 else 2e-6), err

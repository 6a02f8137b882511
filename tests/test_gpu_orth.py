"""Cholesky QR's basis against numpy's QR of the same block, at the edges of
the Gram kernel's 16-column real blocks (k = 8, 16, 24) and of its row groups.

Tolerance: CholQR2 is orthonormal to O(u); Q's difference from a Householder Q
is bounded by about u cond(Y), cond(Y) <= 1e2 here: 1e-12."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_util import to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(23, 12), (17, 16), (61, 40)])
@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 16, 17, 24, 25, 31, 32])
def test_basis_matches_householder_qr(nx, ny, k):
    import paper_1902_01458_amd as rr
    w = W.small("o", nx, ny, nu=5e-2)
    prob = rr.BurgersProblem.from_workload(w)
    f = rr.factor(prob, [0.7, 2.0], "fp64", k_max=32)
    Q = to_np(f.sketch_solve(k, 3, 0))
    Y = to_np(f.solve(rr.sketch(prob, k, 3).expand(2, -1, -1).contiguous()))
    f.check()
    for i in range(2):
        assert np.linalg.cond(Y[i]) < 1e2
        q, r = np.linalg.qr(Y[i].T)
        q = q * (np.diag(r) / np.abs(np.diag(r)))
        assert np.linalg.norm(Q[i].T - q, 2) <= 1e-12
        assert np.linalg.norm(Q[i].conj() @ Q[i].T - np.eye(k), 2) <= 1e-14 * k
    f.free()

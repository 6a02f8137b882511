"""The stencil apply at the edges of its launch: workgroups a shift on both
sides of one, of eight and of the number from which strips are dealt to the
XCDs; ragged strips; more columns than a group.

Tolerance: the six products of a row, 1e-13 of the largest entry (n u for the
few terms a row has would be 1e-15)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operator as op
from tests.gpu_util import oracle_problem, to_np

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("nx,ny,shifts,k", [
    (1, 1, 3, 2), (16, 8, 40, 5), (4, 128, 2, 3), (5, 128, 2, 3), (28, 128, 2, 3), (32, 128, 2, 3),
    (33, 128, 2, 3), (250, 128, 1, 2), (253, 128, 1, 2), (260, 128, 1, 2), (70, 37, 9, 17)])
def test_apply_matches_oracle(nx, ny, shifts, k, adjoint):
    w = W.small("ap", nx, ny, nu=2e-2)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr().BurgersProblem.from_workload(w)
    oms = [0.7 + 0.3 * i - 0.1j * (i % 3) for i in range(shifts)]
    rng = np.random.Generator(np.random.PCG64(nx * ny))
    X = rng.standard_normal((shifts, k, w.n)) + 1j * rng.standard_normal((shifts, k, w.n))
    Y = to_np(prob.apply(oms, torch.tensor(X, device="cuda"), adjoint=adjoint))
    for i, om in enumerate(oms):
        M = op.shifted(L, om)
        ref = ((M.conj().T if adjoint else M) @ X[i].T).T
        np.testing.assert_allclose(Y[i], ref, rtol=0, atol=1e-13 * np.abs(ref).max())

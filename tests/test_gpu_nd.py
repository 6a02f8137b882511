"""The nested-dissection LU against LAPACK's banded solve: single leaves,
fronts at and past the one-launch inverse (P = 64, 80 .. 208), ragged halves,
thin grids, and column counts at the edges of the 16-column blocks and of the
32-column groups.

Tolerances, as for the band LU on the same kind of operator: 1e-11 in FP64 and
1e-4 for unrefined FP32 (kappa ~ 1e2 here, times eps_32 and the n-fold sums)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operator as op
from oracle.solver import ShiftedSolver
from tests.gpu_util import oracle_problem, to_np

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


CASES = [  # (nx, ny, k)
    (1, 1, 1),       # one node
    (8, 4, 16),      # one leaf, 64 unknowns
    (11, 3, 1),      # two leaves under one separator
    (33, 17, 17),    # ragged halves
    (32, 65, 15),    # separators of 64 unknowns, the widest one-launch inverse
    (40, 41, 33),    # 80: two pivot tiles, the second of 16; two column groups
    (150, 104, 20),  # 208 = 3 x 64 + 16: four pivot tiles
    (90, 129, 32),   # 180 -> 192
    (3, 300, 5),     # thin, split along y
    (400, 1, 31),
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,k", CASES)
def test_solves_match_oracle(prec, nx, ny, k):
    w = W.small("nd", nx, ny, nu=2e-2)
    k = min(k, w.n, 32 if prec == "mixed" else k)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr().BurgersProblem.from_workload(w)
    oms = [0.4, 2.5 - 0.1j, 1.1]
    f = rr().factor(prob, oms, prec, k_max=k, refine_tol=1.0)
    rng = np.random.Generator(np.random.PCG64(12))
    Bm = rng.standard_normal((3, k, w.n)) + 1j * rng.standard_normal((3, k, w.n))
    Bt = torch.tensor(Bm, device="cuda")
    X = to_np(f.solve(Bt))
    Z = to_np(f.adjoint_solve(Bt))
    one = to_np(f.solve(Bt[:, :1].contiguous()))
    f.check()
    tol = 1e-11 if prec == "fp64" else 1e-4
    for i, om in enumerate(oms):
        S = ShiftedSolver(op.shifted(L, om), "gb")
        for got, ref in ((X[i], S.solve(Bm[i].T).T), (Z[i], S.solve_adjoint(Bm[i].T).T),
                         (one[i], S.solve(Bm[i, :1].T).T)):
            err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
            assert err <= tol, (i, err)
    f.free()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_refactor_and_solve_repeat_bitwise(prec):
    w = W.small("nd", 90, 70, nu=1e-2)
    prob = rr().BurgersProblem.from_workload(w)
    f = rr().factor(prob, [0.4, 2.5], prec, k_max=9)
    g = torch.Generator(device="cuda").manual_seed(3)
    B = torch.randn((2, 9, w.n), dtype=torch.complex128, device="cuda", generator=g)
    X = to_np(f.solve(B))
    for _ in range(5):
        f.refactor()
        np.testing.assert_array_equal(to_np(f.solve(B)), X)
    f.check()
    f.free()


def test_zero_pivot_is_reported():
    """L = 0 at omega = 0: every pivot is zero."""
    prob = rr().BurgersProblem.from_coefficients(np.zeros((12, 9, 12)))
    f = rr().factor(prob, [0.0], "fp64", k_max=2)
    with pytest.raises(rr().RRError) as e:
        f.check()
    assert e.value.status == 2
    f.free()


@pytest.mark.parametrize("scale", [1e42, 1e-42])
def test_factors_that_fp32_does_not_hold_are_reported(scale):
    """A mixed handle without refinement: the inverses are formed in FP64, and
    an element beyond FP32's range counts as a bad pivot, not as an infinity
    in the results.  (L scaled by 1e42 has inverses that FP32 rounds to zero
    or, with the couplings, overflows on.)"""
    rng = np.random.Generator(np.random.PCG64(8))
    coef = rng.standard_normal((33, 17, 12))
    coef[..., 0] -= 8.0
    coef[..., 6] -= 8.0
    prob = rr().BurgersProblem.from_coefficients(coef * scale)
    f = rr().factor(prob, [0.7 * scale], "mixed", k_max=2, refine_tol=1.0)
    with pytest.raises(rr().RRError) as e:
        f.check()
    assert e.value.status == 2
    f.free()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_many_shifts_take_the_leaves_by_width(prec):
    """160 shifts of 20 narrow and 12 wide leaves run them in two launches: the same
    bits as the same shifts a few at a time, which do not."""
    w = W.small("nd", 37, 29, nu=1e-2)
    prob = rr().BurgersProblem.from_workload(w)
    oms = [0.3 + 0.05 * i for i in range(160)]
    g = torch.Generator(device="cuda").manual_seed(4)
    B = torch.randn((len(oms), 3, w.n), dtype=torch.complex128, device="cuda", generator=g)
    f = rr().factor(prob, oms, prec, k_max=3, refine_tol=1.0)
    X, Z = to_np(f.solve(B)), to_np(f.adjoint_solve(B))
    f.check()
    f.free()
    for i0 in (0, 77, 155):
        f = rr().factor(prob, oms[i0:i0 + 5], prec, k_max=3, refine_tol=1.0)
        part = B[i0:i0 + 5].contiguous()
        np.testing.assert_array_equal(to_np(f.solve(part)), X[i0:i0 + 5])
        np.testing.assert_array_equal(to_np(f.adjoint_solve(part)), Z[i0:i0 + 5])
        f.check()
        f.free()

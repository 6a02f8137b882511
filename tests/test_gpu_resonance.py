"""Default mixed handles next to an eigenvalue of L, where the FP32 factors
contract least: solves and adjoint solves still converge within the default
six corrections, to the accuracy of an FP64 direct solve.

Shifts lie delta |lambda| from the eigenvalue lambda of L with the largest real
part, at an angle to the direction away from the spectrum.

Tolerance: refinement leaves 1e-10, and it and LAPACK's solve each carry the
forward error of a backward stable method, a modest multiple of u kappa(M)
(10 here), with kappa(M) = ||M|| ||M^-1|| from power iterations."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operator as op
from oracle.probe import spectral_norm
from oracle.solver import ShiftedSolver
from tests.gpu_util import oracle_problem, to_np

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


def near(nx, ny, nu, delta, angle):
    w = W.small("i", nx, ny, nu=nu)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    lam = np.linalg.eigvals(L.toarray())
    lam0 = lam[np.argmax(lam.real)]
    omega = -1j * (lam0 + delta * abs(lam0) * np.exp(1j * angle))
    M = op.shifted(L, omega)
    S = ShiftedSolver(M, "gb")
    x = np.random.default_rng(1).standard_normal(w.n) + 0j
    for _ in range(10):  # ||M^-1|| by power iterations on M^-H M^-1
        x = S.solve_adjoint(S.solve(x / np.linalg.norm(x)))
    kappa = spectral_norm(M, iters=50) * np.sqrt(np.linalg.norm(x))
    return w, omega, S, 1e-10 + 10 * 1.1e-16 * kappa


GRIDS = [(32, 16, 1e-2, 0.0), (24, 48, 1e-2, 0.0), (40, 40, 2e-3, 0.0),
         # blocks whose unpivoted inverses grow
         (19, 8, 0.012718553384797597, 0.0), (13, 13, 0.016769632772920734, 0.0),
         (24, 17, 0.002242694104895137, -1.02248152557075),
         (25, 23, 0.00659996176983551, -1.1685227269381682),
         (20, 11, 0.0069041977183398945, -0.7284989908738247),
         (19, 24, 0.004842359566141959, 0.5188977931291681),
         (17, 13, 0.01639794398556262, 1.1029487298118226),
         (23, 8, 0.005107938793322731, 0.35869567957332027)]


@pytest.mark.parametrize("delta", [1e-4, 1e-5])
@pytest.mark.parametrize("nx,ny,nu,angle", GRIDS)
def test_mixed_solves_converge_next_to_an_eigenvalue(nx, ny, nu, angle, delta):
    w, omega, S, tol = near(nx, ny, nu, delta, angle)
    rng = np.random.default_rng(0)
    B = rng.standard_normal((1, 4, w.n)) + 1j * rng.standard_normal((1, 4, w.n))
    Bt = torch.as_tensor(B, device="cuda")
    f = rr().factor(rr().BurgersProblem.from_workload(w), [omega], "mixed", k_max=4)
    for solve, ref in ((f.solve, S.solve), (f.adjoint_solve, S.solve_adjoint)):
        X = to_np(solve(Bt))[0]
        f.check()
        Y = ref(B[0].T).T
        err = np.linalg.norm(X - Y) / np.linalg.norm(Y)
        print(f"\n{f.refine_count()} corrections, error {err:.1e} of {tol:.1e}")
        assert err <= tol
    f.free()

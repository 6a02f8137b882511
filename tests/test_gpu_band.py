"""The band LU, which an explicit superblock asks for: the shapes that the band
makes (tiles per half-band against waves, early and final updates, superblocks
of 256 rows), its repeatability, more shifts than one factor launch takes, and
the autotuner's band picks.

Tolerances: 1e-11 for FP64 solves against LAPACK's on these operators (kappa
about 1e2), 1e-9 for refined mixed ones (refinement to 1e-10), 1e-10 / 1e-8 for
gains."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import operator as op
from oracle import resolvent as ores
from oracle import sketch as osk
from oracle.solver import ShiftedSolver
from tests.gpu_util import gain_errors, oracle_problem, to_np

pytestmark = pytest.mark.gpu


def rr():
    import paper_1902_01458_amd as m
    return m


def rows256(ny, tile):
    """The superblock of 256 rows, at most the half-band's tiles."""
    return max(1, min(-(-2 * ny // tile), 256 // tile))


SOLVE_CASES = [  # (nx, ny, tile, k)
    (10, 6, 32, 3),     # ragged n and b
    (13, 20, 64, 17),
    (24, 40, 32, 5),
    (9, 48, 64, 20),
    (16, 96, 32, 12),   # B = 6 tiles per half-band: early and final updates
    (12, 100, 64, 32),  # B = 4 at the 64 tile, ragged n, k = 32
    (8, 160, 32, 20),   # B = 10 at the 32 tile: superblock steps with more tiles than waves
    (6, 288, 64, 20),   # B = 9 at the 64 tile: the same
    (30, 40, 32, 40),   # two column groups (FP64)
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nx,ny,tile,k", SOLVE_CASES)
def test_solves_match_oracle(prec, nx, ny, tile, k):
    w = W.small("s", nx, ny, nu=2e-2)
    k = min(k, 32) if prec == "mixed" else k
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr().BurgersProblem.from_workload(w)
    oms = [0.4, 2.5]
    f = rr().factor(prob, oms, prec, k_max=k, tile=tile, superblock=rows256(ny, tile))
    rng = np.random.Generator(np.random.PCG64(11))
    Bm = rng.standard_normal((2, k, w.n)) + 1j * rng.standard_normal((2, k, w.n))
    Bt = torch.tensor(Bm, device="cuda")
    X = to_np(f.solve(Bt))
    Z = to_np(f.adjoint_solve(Bt))
    f.check()
    tol = 1e-11 if prec == "fp64" else 1e-9
    for i, om in enumerate(oms):
        S = ShiftedSolver(op.shifted(L, om), "gb")
        for got, ref in ((X[i], S.solve(Bm[i].T).T), (Z[i], S.solve_adjoint(Bm[i].T).T)):
            assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
    f.free()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("superblock", [4, -1])
def test_refactor_is_bitwise_repeatable(prec, superblock):
    """Each band tile is written twice per launch and read from other
    workgroups, usually on other XCDs: a stale read gives another factor."""
    w = W.small("r", 96, 64, nu=5e-3, omegas=tuple(0.3 * 1.5 ** i for i in range(8)), k=8)
    prob = rr().BurgersProblem.from_workload(w)
    f = rr().factor(prob, list(w.omegas), prec, k_max=w.k, tile=64, superblock=superblock)
    Bm = rr().sketch(prob, w.k, seed=0).unsqueeze(0).expand(8, w.k, prob.n).contiguous()
    X0 = f.solve(Bm).clone()
    f.check()
    for _ in range(4):
        f.refactor()
        X = f.solve(Bm)
        f.check()
        assert torch.equal(X, X0)
    R = Bm - prob.apply(list(w.omegas), X0)
    rel = (torch.linalg.vector_norm(R, dim=2) / torch.linalg.vector_norm(Bm, dim=2)).max()
    assert float(rel) < (1e-12 if prec == "fp64" else 1e-8)
    f.free()


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-8)])
@pytest.mark.parametrize("k", [1, 4])
def test_more_shifts_than_one_factor_launch(prec, tol, k):
    omegas = tuple(np.linspace(0.1, 7.0, 70))  # 64 + 6
    w = W.small("g", 12, 10, nu=2e-2, omegas=omegas, k=k)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr().BurgersProblem.from_workload(w)
    out = rr().resolvent(prob, list(omegas), k=k, q=1, seed=w.seed, precision=prec, tile=32,
                         superblock=1)
    Om = osk.test_matrix(w.n, k, phi, w.seed)
    for i in (0, 1, 63, 64, 65, 69):
        ref = ores.randomized_resolvent(L, omegas[i], Om, q=1)
        assert gain_errors(to_np(out["sigma_B"])[i], ref.sigma_B).max() <= tol, i
        assert gain_errors(to_np(out["sigma_AV"])[i], ref.sigma_AV).max() <= tol, i
    out["factors"].free()


@pytest.mark.parametrize("tile,superblock", [(64, 2), (64, -1), (32, 8)])
def test_picks_with_a_superblock_match_oracle(tile, superblock):
    """What the autotuner may pick, used the way its result is meant to be."""
    w = W.small("at", 48, 40, nu=1e-2, omegas=(0.6, 2.2), k=10, q=1)
    prob = rr().BurgersProblem.from_workload(w)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    refs = [ores.randomized_resolvent(L, om, osk.test_matrix(w.n, w.k, phi, w.seed), q=w.q)
            for om in w.omegas]
    tune = {"tile": tile, "grid": 256, "superblock": superblock}
    out = rr().sweep(prob, list(w.omegas), w.k, q=w.q, seed=w.seed, tune=tune)
    res = rr().resolvent(prob, list(w.omegas), k=w.k, q=w.q, seed=w.seed, **tune)
    for i, r in enumerate(refs):
        for got in (out, res):
            assert gain_errors(to_np(got["sigma_AV"][i]), r.sigma_AV).max() <= 1e-10
    res["factors"].free()


def test_the_autotuners_own_pick_matches_oracle():
    w = W.small("at", 48, 40, nu=1e-2, omegas=(0.6, 2.2), k=10, q=1)
    prob = rr().BurgersProblem.from_workload(w)
    t = rr().autotune(prob, list(w.omegas), w.k, "fp64")
    out = rr().resolvent(prob, list(w.omegas), k=w.k, q=w.q, seed=w.seed, tile=t["tile"],
                         grid=t["grid"], superblock=t["superblock"])
    U, coef, L, phi, hx, hy = oracle_problem(w)
    Om = osk.test_matrix(w.n, w.k, phi, w.seed)
    for i, om in enumerate(w.omegas):
        r = ores.randomized_resolvent(L, om, Om, q=w.q)
        assert gain_errors(to_np(out["sigma_AV"][i]), r.sigma_AV).max() <= 1e-10
    out["factors"].free()

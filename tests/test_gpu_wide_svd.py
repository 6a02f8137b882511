"""The wide SVD at the edges of its forms: odd widths, whose Jacobi is padded by
a column of zeros, the 32-wide blocks of the Cholesky, and both sides of k = 100,
where A leaves LDS.  All gains against the oracle; V orthonormal to 1e-12: a
column passes some 8 sweeps x 100 rotations, each within a few units in the last
place (4e-13)."""
import numpy as np
import pytest

import workloads as W
from oracle import resolvent as ores
from oracle import sketch as osk
from tests.gpu_util import gain_errors, oracle_problem, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [33, 64, 65, 99, 100, 101])
def test_wide_gains_match_oracle(k):
    import paper_1902_01458_amd as rr
    w = W.small("ws", 17, 16, nu=5e-2)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr.BurgersProblem.from_workload(w)
    out = rr.resolvent(prob, [0.7, 2.0], k=k, q=0, seed=3, precision="fp64")
    Om = osk.test_matrix(w.n, k, phi, seed=3)
    for i, om in enumerate([0.7, 2.0]):
        ref = ores.randomized_resolvent(L, om, Om, q=0)
        assert gain_errors(to_np(out["sigma_B"])[i], ref.sigma_B).max() <= 1e-10
        assert gain_errors(to_np(out["sigma_AV"])[i], ref.sigma_AV).max() <= 1e-10
        V = to_np(out["V"])[i]
        assert np.linalg.norm(V.conj() @ V.T - np.eye(k), 2) <= 1e-12


@pytest.mark.parametrize("k", [359, 360, 361, 384])
def test_gains_on_both_sides_of_a_waves_pairs(k):
    """Past k = 360 a wave takes a pair of columns, up to it 16 lanes.  V
    orthonormal: 10 sweeps x 360 rotations, two units in the last place each
    (8e-13 a column), sqrt(k) = 19 times that in the 2-norm: 2e-11."""
    import paper_1902_01458_amd as rr
    w = W.small("ws", 17, 16, nu=5e-2)
    U, coef, L, phi, hx, hy = oracle_problem(w)
    prob = rr.BurgersProblem.from_workload(w)
    out = rr.resolvent(prob, [2.0], k=k, q=0, seed=3, precision="fp64")
    ref = ores.randomized_resolvent(L, 2.0, osk.test_matrix(w.n, k, phi, seed=3), q=0)
    assert gain_errors(to_np(out["sigma_B"])[0], ref.sigma_B).max() <= 1e-10
    assert gain_errors(to_np(out["sigma_AV"])[0], ref.sigma_AV).max() <= 1e-10
    V = to_np(out["V"])[0]
    assert np.linalg.norm(V.conj() @ V.T - np.eye(k), 2) <= 2e-11

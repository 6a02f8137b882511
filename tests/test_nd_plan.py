"""The plan of the nested-dissection LU (rr_nd_plan, host only): its fronts and
index tables carry a numpy multifrontal elimination, written from the block
formulas alone, to the solution of the same system; its arenas do not overlap
and its launches cover every tile once.

Tolerance of the solves: n u kappa for these well-conditioned systems is far
below 1e-11 relative (FP64 products of at most 200 x 200 blocks)."""
import ctypes
import subprocess
import sys

import numpy as np
import pytest

from oracle import operator as op
from paper_1902_01458_amd import _lib

FIELDS = ("p q P Q row bor childA childB baseA baseB urow a b12 f21 s t depth").split()
TILE = 64


def values(nx, ny, what):
    L = _lib.lib()
    n = L.rr_nd_plan(nx, ny, what, None, 0)
    out = np.zeros(n, dtype=np.int64)
    assert L.rr_nd_plan(nx, ny, what, out.ctypes.data_as(ctypes.c_void_p), n) == n
    return out


def plan(nx, ny):
    fronts = [dict(zip(FIELDS, map(int, f))) for f in values(nx, ny, 0).reshape(-1, len(FIELDS))]
    return (fronts, values(nx, ny, 1), values(nx, ny, 2), values(nx, ny, 3),
            values(nx, ny, 4).reshape(-1, 4), values(nx, ny, 5))


GRIDS = [(4, 4), (1, 1), (7, 5), (1, 70), (70, 1), (2, 40), (33, 17), (24, 48), (65, 9), (40, 40),
         (19, 64), (80, 71)]


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_plan_carries_a_multifrontal_elimination(nx, ny):
    fronts, pdof, bmap, grow, _, totals = plan(nx, ny)
    rng = np.random.default_rng(nx * 1000 + ny)
    coef = rng.standard_normal((nx, ny, 12))
    coef[..., 0] -= 8.0
    coef[..., 6] -= 8.0
    M = op.shifted(op.assemble(coef), 0.7 - 0.1j).tocsr()
    n, rows, allrows = 2 * nx * ny, int(totals[0]), int(totals[1])
    assert sorted(pdof[pdof >= 0]) == list(range(n)) and len(pdof) == allrows
    assert grow.max(initial=rows) == rows
    F = {}
    for f in range(len(fronts) - 1, -1, -1):
        x = fronts[f]
        p, q = x["p"], x["q"]
        piv = pdof[x["row"]:x["row"] + p]
        assert (pdof[x["row"] + p:x["row"] + x["P"]] == -1).all()
        bor = pdof[grow[x["bor"]:x["bor"] + q]]
        assert (grow[x["bor"] + q:x["bor"] + x["Q"]] == rows).all()
        D = np.zeros((p + q, p + q), dtype=complex)
        both = np.concatenate([piv, bor])
        D[:] = M[both][:, both].toarray()
        D[p:, p:] = 0.0
        if x["childA"] < 0:  # a border unknown has one neighbour in a leaf
            at = bmap[x["bor"]:x["bor"] + q]
            only = np.zeros((p, q), dtype=bool)
            only[at, np.arange(q)] = True
            assert (D[:p, p:][~only] == 0).all() and (D[p:, :p][~only.T] == 0).all()
        else:
            assert x["row"] + x["P"] <= rows
        for half, name in enumerate("AB"):
            c = x["child" + name]
            if c < 0:
                continue
            assert fronts[c]["depth"] == x["depth"] + 1
            bm = bmap[x["bor"]:x["bor"] + q]
            mine = np.flatnonzero((bm >= 0) & (bm % 2 == half))
            at = np.concatenate([np.arange(p), p + mine])
            src = np.concatenate([x["base" + name] + np.arange(p), bm[mine] // 2])
            assert len(set(src)) == len(src) == fronts[c]["q"]
            # the half's border is these unknowns, in this order
            cb = pdof[grow[fronts[c]["bor"] + src]]
            np.testing.assert_array_equal(cb, both[at])
            D[np.ix_(at, at)] += F[c]["S"][np.ix_(src, src)]
        A = np.linalg.inv(D[:p, :p])
        B12 = A @ D[:p, p:]
        F[f] = {"A": A, "B12": B12, "F21": D[p:, :p], "S": D[p:, p:] - D[p:, :p] @ B12}
    b = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    for adjoint in (False, True):
        rhs = np.zeros(allrows, dtype=complex)
        rhs[pdof >= 0] = b[pdof[pdof >= 0]]
        u, z, sol, X = {}, {}, np.zeros(rows + 1, dtype=complex), np.zeros(n, dtype=complex)
        for f in range(len(fronts) - 1, -1, -1):
            x, g = fronts[f], F[f]
            b1 = rhs[x["row"]:x["row"] + x["p"]].copy()
            up = np.zeros(x["q"], dtype=complex)
            for half, name in enumerate("AB"):
                c = x["child" + name]
                if c >= 0:
                    b1 += u[c][x["base" + name]:x["base" + name] + x["p"]]
                    bm = bmap[x["bor"]:x["bor"] + x["q"]]
                    mine = (bm >= 0) & (bm % 2 == half)
                    up[mine] += u[c][bm[mine] // 2]
            z[f] = b1 if adjoint else g["A"] @ b1
            u[f] = up - (g["B12"].conj().T @ b1 if adjoint else g["F21"] @ z[f])
        for f, x in enumerate(fronts):
            x2 = sol[grow[x["bor"]:x["bor"] + x["q"]]]
            g = F[f]
            x1 = (g["A"].conj().T @ (z[f] - g["F21"].conj().T @ x2) if adjoint
                  else z[f] - g["B12"] @ x2)
            if x["childA"] >= 0:
                sol[x["row"]:x["row"] + x["p"]] = x1
            X[pdof[x["row"]:x["row"] + x["p"]]] = x1
        K = (M.conj().T if adjoint else M)
        assert np.linalg.norm(K @ X - b) <= 1e-11 * np.linalg.norm(b)


@pytest.mark.parametrize("nx,ny", GRIDS + [(300, 200), (20, 400)])
def test_plan_arenas_and_tasks(nx, ny):
    fronts, pdof, bmap, grow, tasks, totals = plan(nx, ny)
    rows, allrows, border, factor, s0, s1, temp, u0, u1, ntasks = map(int, totals)
    assert len(tasks) == ntasks and len(bmap) == len(grow) == border

    def disjoint(spans, size):
        end = 0
        for lo, n in sorted(spans):
            assert lo >= end and n >= 0
            end = lo + n
        assert end <= size

    disjoint([(x["row"], x["P"]) for x in fronts], allrows)
    disjoint([(x["bor"], x["Q"]) for x in fronts], border)
    disjoint([(x[o], n) for x in fronts for o, n in (("a", x["P"] ** 2), ("b12", x["P"] * x["Q"]),
                                                      ("f21", x["P"] * x["Q"]))
              if o == "a" or x["childA"] >= 0], factor)
    want = {}

    def expect(f, key, n=1):
        want[(f,) + key] = want.get((f,) + key, 0) + n

    for d in range(max(x["depth"] for x in fronts) + 1):
        level = [(f, x) for f, x in enumerate(fronts) if x["depth"] == d]
        disjoint([(x["s"], x["Q"] ** 2) for _, x in level], (s0, s1)[d % 2])
        disjoint([(x["urow"], x["Q"]) for _, x in level], (u0, u1)[d % 2])
        disjoint([(x["t"], x["P"] * x["Q"] + 2 * TILE * x["P"] + 4 * TILE * TILE)
                  for _, x in level if x["P"] > TILE], temp)
        assert all(x["P"] <= TILE for _, x in level if x["childA"] < 0)
    for f, x in enumerate(fronts):
        np_, nq = -(-x["P"] // TILE), -(-x["Q"] // TILE)
        T = [(i, j) for i in range(np_) for j in range(np_)]
        if x["childA"] < 0:
            expect(f, (0, 0, 0))
            continue
        for i in range(nq):
            for j in range(nq):
                expect(f, (i, j, 0))  # S
        for i in range(1 if x["P"] <= 32 else x["P"] // 16):
            expect(f, (i, 0, 0))  # down
        if x["P"] <= TILE:
            expect(f, (0, 0, 0))
            continue
        for i, j in T:
            expect(f, (i, j, 0))  # F11
            for k in range(np_):
                expect(f, (i, j, k))  # update
        for i in range(np_):
            expect(f, (i, 0, 0))  # gather
            for j in range(nq):
                expect(f, (i, j, 1))
                expect(f, (j, i, 2))
                expect(f, (i, j, 0))  # B12
            for k in range(np_):
                if i != k:
                    expect(f, (i, k, 0))
                    expect(f, (i, k, 1))
        for i in range(x["P"] // 16):
            expect(f, (i, 0, 0))
        for i in range(x["Q"] // 16):
            expect(f, (i, 0, 0))
    got = {}
    for t in map(tuple, tasks.tolist()):
        got[t] = got.get(t, 0) + 1
    assert got == want


def test_plan_rejects_bad_arguments():
    L = _lib.lib()
    assert L.rr_nd_plan(0, 4, 0, None, 0) == -1
    assert L.rr_nd_plan(4, 4, 6, None, 0) == -1
    assert L.rr_nd_plan(1 << 15, 1 << 15, 5, None, 0) == -1


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nx,ny", [(64, 32), (101, 45), (20, 400), (256, 128), (1024, 512),
                                   (4000, 12), (50000, 16), (1, 20000), (20000, 1)])
def test_nested_dissection_needs_no_more_memory_than_the_band(nx, ny, prec):
    """What fitted before fits: a default handle against the band LU's at its default tile."""
    L = _lib.lib()
    for nw in (1, 7):
        assert 0 < L.rr_factor_bytes(nx, ny, nw, 8, prec, 0) <= L.rr_factor_bytes(nx, ny, nw, 8,
                                                                                   prec, 64)


@pytest.mark.parametrize("nx,ny", GRIDS + [(300, 200), (20, 400), (5, 1200), (129, 127)])
def test_sizes_counted_by_blocks_are_the_plans(nx, ny):
    fronts, pdof, bmap, grow, tasks, totals = plan(nx, ny)
    tree = [x for x in fronts if x["childA"] >= 0]
    depth = max(x["depth"] for x in fronts) + 1

    def per_level(size, parity):
        return max([sum(size(x) for x in fronts if x["depth"] == d)
                    for d in range(depth) if d % 2 == parity], default=0)

    def temp(x):
        return x["P"] * x["Q"] + 2 * TILE * x["P"] + 4 * TILE * TILE if x["P"] > TILE else 0

    want = [sum(x["P"] for x in tree), sum(x["P"] for x in fronts), sum(x["Q"] for x in fronts),
            sum(x["P"] ** 2 for x in fronts) + sum(2 * x["P"] * x["Q"] for x in tree),
            per_level(lambda x: x["Q"] ** 2, 0), per_level(lambda x: x["Q"] ** 2, 1),
            max(per_level(temp, 0), per_level(temp, 1)),
            per_level(lambda x: x["Q"], 0), per_level(lambda x: x["Q"], 1), len(tasks)]
    assert totals.tolist() == want


@pytest.mark.parametrize("nx,ny", [(16384, 8192), (40000, 40000), (2 ** 31 - 1, 1),
                                   (2 ** 20, 2 ** 20), (2 ** 31 - 1, 2 ** 31 - 1)])
def test_the_size_of_a_grid_of_any_size_is_answered_at_once(nx, ny):
    """In a process of its own: an exception through the C entry ends it."""
    code = ("import time\n"
            "from paper_1902_01458_amd import _lib\n"
            "L = _lib.lib()\n"
            f"t = time.perf_counter(); b = L.rr_factor_bytes({nx}, {ny}, 1, 8, 0, 0)\n"
            "print(b, time.perf_counter() - t)\n")
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=110)
    assert out.returncode == 0, out.stderr[-500:]
    size, seconds = out.stdout.split()
    assert int(size) >= min(2 * nx * ny * 16 * 16, 2 ** 64 - 1)  # 16 entries a row at least
    assert float(seconds) < 0.1

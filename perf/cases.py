"""The measured workloads: what a user of this package has it do, through its public entry points.

Every operator is the linearised Burgers operator about the shear layer of
`workloads`, with smoothed noise of the 1024 x 512 configuration's amplitude
drawn from the seed (it also separates the layer's nearly degenerate gains, so
that modes are well defined).  Grids run from 24 x 12 to 1024 x 512 nodes,
sketch widths from 2 to 128, batches from 1 to 64 shifts.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1902_01458_amd as rr
import workloads

# --- cases -------------------------------------------------------------------
# kind   what a pass is
#   resolvent  rr.resolvent: a handle made, Algorithm 1, the handle dropped
#   sweep      rr.sweep: gains over a list of shifts (handle and graph inside)
#   sigma_one  the differentiable leading gain, forward and backward
#   pass       refactor, sketch, subspace iteration, adjoint solve, gains on a kept handle
#   project    the same up to the adjoint solve (steps 1-4)
#   solve / adjoint   one solve on a kept handle
#   krylov     one solve of a handle without an LU
#   apply      the shifted operator applied to a block


def _case(name, kind, nx, ny, shifts, k, precision="fp64", q=0, nu=1e-2, wide=False, **more):
    c = {"name": name, "kind": kind, "nx": nx, "ny": ny, "shifts": shifts, "k": k,
         "precision": precision, "q": q, "nu": nu, "wide": wide, **more}
    return c


def listed():
    return [
        # the smallest configuration, as a script calls it: one frequency, everything in one call
        _case("resolvent_64x32", "resolvent", 64, 32, 1, 10),
        # a coarse survey over a ragged grid in mixed precision
        _case("sweep_mixed_101x45", "sweep", 101, 45, 12, 7, "mixed"),
        # the frequency sweep of 64 shifts
        _case("sweep_256x128", "sweep", 256, 128, 64, 10),
        # one step of base-flow sensitivity: gain and its gradient at 4 shifts
        _case("sigma_one_256x128", "sigma_one", 256, 128, 4, 12, nu=5e-3),
        # one frequency at the benchmark's grid: latency of a whole FP64 pass
        _case("pass_512x256", "pass", 512, 256, 1, 20, q=1, nu=2e-3, wide=True),
        # the benchmark's batch, mixed precision, up to the projected operator
        _case("project_mixed_512x256x16", "project", 512, 256, 16, 20, "mixed", q=1, nu=2e-3,
              wide=True),
        # a block of right-hand sides on kept factors, FP64, forward
        _case("solve_512x256x8", "solve", 512, 256, 8, 20, nu=2e-3, wide=True),
        # the same adjoint, in mixed precision with its refinement
        _case("adjoint_mixed_512x256x8", "adjoint", 512, 256, 8, 20, "mixed", nu=2e-3, wide=True),
        # the largest grid, one frequency, the widest narrow sketch
        _case("solve_1024x512", "solve", 1024, 512, 1, 32, nu=1e-3),
        # a sketch wider than 32 columns (the k study)
        _case("pass_wide_64x32", "pass", 64, 32, 1, 100),
        # a solve without any LU
        _case("krylov_128x64", "krylov", 128, 64, 1, 10, solver="bicgstab", precond="ilu0"),
        # residual checks: the operator applied to the benchmark's block
        _case("apply_512x256x16", "apply", 512, 256, 16, 20, nu=2e-3, wide=True),
    ]


def _between(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    kind = rng.choice(("resolvent", "sweep", "sigma_one", "pass", "project", "solve", "adjoint",
                       "solve", "pass", "wide", "krylov", "apply"))
    precision = rng.choice(("fp64", "mixed"))
    small = kind in ("resolvent", "wide", "krylov")
    lo = 40 if kind == "wide" else 24
    nx = _between(rng, lo, 96 if kind == "wide" else 128 if small else 512)
    ny = _between(rng, lo // 2, min(nx, 48 if kind == "wide" else 64 if small else 256))
    c = _case(None, kind, nx, ny, _between(rng, 1, 8), _between(rng, 2, 32), precision,
              q=rng.choice((0, 1)))
    del c["name"]
    if kind in ("resolvent", "sigma_one", "pass", "krylov", "apply"):
        c["precision"] = "fp64"
    if kind == "sweep":
        c["shifts"] = _between(rng, 2, 24)
        c["q"] = rng.choice((0, 1))
    if kind == "wide":
        c.update(kind="pass", precision="fp64", k=_between(rng, 33, 128), shifts=_between(rng, 1, 2))
    if kind == "krylov":
        c.update(solver="bicgstab", precond="ilu0", shifts=1,
                 k=_between(rng, 2, 16))
    if kind in ("solve", "adjoint"):
        c["q"] = 0
    return c


# --- inputs ------------------------------------------------------------------


def _blur(m, width=8.0):
    """The m x m matrix of a Gaussian filter of `width` nodes, cut off at 4 widths."""
    i = torch.arange(m, dtype=torch.float64)
    d = i[:, None] - i[None, :]
    g = torch.exp(-0.5 * (d / width) ** 2) * (d.abs() <= 4 * width)
    return g.cuda()


def _setup(case, seed):
    """(base flow on the GPU, domain, frequencies) of a case."""
    nx, ny = case["nx"], case["ny"]
    domain = (0.0, 16.0, -4.0, 4.0) if case["wide"] else (0.0, 8.0, -2.0, 2.0)
    w = workloads.Workload("case", nx, ny, domain, case["nu"], (1.0,), case["k"], case["q"],
                           stretch=2.0 if case["wide"] else 1.0)
    g = torch.Generator().manual_seed(int(seed))
    noise = torch.randn((nx + 2, ny + 2), dtype=torch.float64, generator=g).cuda()
    noise = _blur(nx + 2) @ noise @ _blur(ny + 2)
    U = torch.from_numpy(workloads.base_flow(w)).cuda() + 0.05 * noise / noise.abs().max()
    m = case["shifts"]
    # log-spaced over [0.25, 8], each moved by up to 5 %; one shift sits near 2
    at = [0.25 * 32.0 ** (i / (m - 1)) for i in range(m)] if m > 1 else [2.0]
    move = torch.rand(m, dtype=torch.float64, generator=g).tolist()
    return U, domain, [a * (0.95 + 0.1 * t) for a, t in zip(at, move)]


def _block(case, seed):
    """A block of complex normal right-hand sides."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    return torch.randn((case["shifts"], case["k"], 2 * case["nx"] * case["ny"]),
                       dtype=torch.complex128, device="cuda", generator=g)


def prepare(case, seed):
    U, domain, omegas = _setup(case, seed)
    kind, nx, ny = case["kind"], case["nx"], case["ny"]
    s = {"case": case, "seed": int(seed), "omegas": omegas}
    if kind == "sigma_one":
        s["args"] = (nx, ny, domain)
        s["U"] = U.requires_grad_(True)
        s["nu"] = torch.tensor(case["nu"], dtype=torch.float64, device="cuda", requires_grad=True)
        s["omega"] = torch.tensor(omegas, dtype=torch.float64, device="cuda",
                                  requires_grad=True)
        s["weight"] = torch.linspace(0.5, 1.5, len(omegas), dtype=torch.float64, device="cuda")
        return s
    s["prob"] = rr.BurgersProblem.from_base_flow(U, nx, ny, domain, case["nu"])
    if kind in ("solve", "adjoint", "krylov", "apply"):
        s["B"] = _block(case, seed)
    if kind in ("pass", "project", "solve", "adjoint"):
        s["f"] = rr.factor(s["prob"], omegas, case["precision"], k_max=case["k"])
    if kind == "krylov":
        s["f"] = rr.factor(s["prob"], omegas, "fp64", k_max=case["k"], solver=case["solver"],
                           precond=case["precond"], krylov_maxit=400, krylov_tol=1e-12)
    if kind in ("pass", "project"):
        s["Q"], s["Z"] = s["f"].empty_block(case["k"]), s["f"].empty_block(case["k"])
    elif kind in ("solve", "adjoint", "krylov"):
        s["X"] = s["f"].empty_block(case["k"])
    return s


# --- one pass ----------------------------------------------------------------


def _phased(V, U, Q):
    """Modes with their phase fixed, as a program does that compares or plots them: the
    component of each response mode along the first basis vector is real and positive."""
    a = torch.linalg.vecdot(Q[:, :1], U)
    a = (a.conj() / a.abs())[:, :, None]
    return {"V": V * a, "U": U * a}


def run(s):
    c = s["case"]
    kind, k, q, seed = c["kind"], c["k"], c["q"], s["seed"]
    if kind == "resolvent":
        out = rr.resolvent(s["prob"], s["omegas"], k, q, seed, c["precision"])
        out.pop("factors").free()
        return {**{m: out[m] for m in ("sigma_B", "sigma_AV", "Q")},
                **_phased(out["V"], out["U"], out["Q"])}
    if kind == "sweep":
        out = rr.sweep(s["prob"], s["omegas"], k, q, seed, c["precision"])
        return {m: out[m] for m in ("sigma_B", "sigma_AV")}
    if kind == "sigma_one":
        s1 = rr.sigma_one(s["U"], s["nu"], s["omega"], *s["args"], k=k, q=q, seed=seed,
                          precision=c["precision"])
        g = torch.autograd.grad((s1 * s["weight"]).sum(), (s["U"], s["nu"], s["omega"]))
        return {"sigma": s1.detach(), "dU": g[0], "dnu": g[1], "domega": g[2]}
    if kind == "apply":
        return s["prob"].apply(s["omegas"], s["B"])
    f = s["f"]
    if kind in ("solve", "krylov"):
        return f.solve(s["B"], out=s["X"])
    if kind == "adjoint":
        return f.adjoint_solve(s["B"], out=s["X"])
    f.refactor()
    f.sketch_solve(k, seed, q, out=s["Q"])
    f.adjoint_solve(s["Q"], out=s["Z"])
    if kind == "project":
        return {"Q": s["Q"], "Z": s["Z"]}
    s["out"] = f.gains(s["Q"], s["Z"], "av", out=s.get("out"))
    return {"Q": s["Q"], "Z": s["Z"], **s["out"],
            **_phased(s["out"]["V"], s["out"]["U"], s["Q"])}


# --- what a pass cannot do without ----------------------------------------------


@functools.lru_cache(maxsize=None)
def _elimination(nx, ny, left, right, low, high):
    """(multiply-adds, factor entries) of eliminating an nx x ny block of nodes, two
    unknowns each, in nested-dissection order; the flags say which sides border on
    separators eliminated later."""
    if nx < ny:
        nx, ny, left, right, low, high = ny, nx, low, high, left, right
    border = 2 * (ny * (left + right) + nx * (low + high))  # unknowns of those separators
    if nx * ny <= 4 or nx < 3:
        p, parts = 2 * nx * ny, ()
    else:
        a = (nx - 1) // 2
        p = 2 * ny
        parts = (_elimination(a, ny, left, True, low, high),
                 _elimination(nx - 1 - a, ny, True, right, low, high))
    return (p ** 3 / 3 + p * p * border + p * border * border + sum(x[0] for x in parts),
            p * p + 2 * p * border + sum(x[1] for x in parts))


def work(case):
    """Each input read and each output written once, the factors of a sparse direct
    solver written once and read once a solve, and that solver's arithmetic."""
    nx, ny, m, k, kind = case["nx"], case["ny"], case["shifts"], case["k"], case["kind"]
    n, e = 2 * nx * ny, 8 if case["precision"] == "mixed" else 16
    block = 16 * k * n * m
    if kind in ("apply", "krylov"):  # one application of the stencil at the least
        return {"bytes": 2 * block + 96 * nx * ny, "flops": 8 * 6 * k * n * m}
    mac, entries = _elimination(nx, ny, False, False, False, False)
    one = {"bytes": 2 * block + entries * e * m, "flops": 8 * entries * k * m}
    if kind in ("solve", "adjoint"):
        return one
    solves = (2 if kind == "project" else 3) + 2 * case["q"]
    orth = 8 * k * k * n * m
    return {"bytes": solves * one["bytes"] + entries * e * m,
            "flops": 8 * mac * m + solves * (one["flops"] + 2 * orth)}


# --- the same in plain torch ---------------------------------------------------


def _operator(case, U, domain):
    """Stencil of L by nodes: dicts of (nx, ny) arrays for the u- and the v-row."""
    nx, ny, nu = case["nx"], case["ny"], case["nu"]
    hx, hy = (domain[1] - domain[0]) / (nx + 1), (domain[3] - domain[2]) / (ny + 1)
    Uc = U[1:-1, 1:-1]
    Ux = (U[2:, 1:-1] - U[:-2, 1:-1]) / (2 * hx)
    Uy = (U[1:-1, 2:] - U[1:-1, :-2]) / (2 * hy)
    lap = -2 * nu * (1 / hx ** 2 + 1 / hy ** 2)
    east, west = nu / hx ** 2 - Uc / (2 * hx), nu / hx ** 2 + Uc / (2 * hx)
    north = torch.full_like(Uc, nu / hy ** 2)
    return {"uu": lap - Ux, "uv": -Uy, "vv": torch.full_like(Uc, lap), "E": east, "W": west,
            "N": north, "phi": torch.sqrt(Ux ** 2 + Uy ** 2) + 0.1}


def _lines(op, omegas):
    """M = i omega - L by grid lines (all nodes of one x): the diagonal blocks without the
    shift, (nx, b, b), and the diagonals that couple a line to the next and the previous one."""
    nx, ny = op["E"].shape
    b = 2 * ny
    D = torch.zeros((nx, b, b), dtype=torch.complex128, device=op["E"].device)
    u = torch.arange(0, b, 2, device=D.device)
    D[:, u, u], D[:, u + 1, u + 1], D[:, u, u + 1] = -op["uu"] + 0j, -op["vv"] + 0j, -op["uv"] + 0j
    for s in (0, 1):
        D[:, u[:-1] + s, u[1:] + s] = -op["N"][:, :-1] + 0j
        D[:, u[1:] + s, u[:-1] + s] = -op["N"][:, 1:] + 0j
    return D, -op["E"].repeat_interleave(2, 1), -op["W"].repeat_interleave(2, 1)


class _Direct:
    """Block elimination line by line, with every pivot block inverted."""

    def __init__(self, op, omegas):
        self.D, self.E, self.W = _lines(op, omegas)
        nx, b, _ = self.D.shape
        om = torch.tensor(omegas, dtype=torch.float64, device=self.D.device)
        shift = 1j * om[:, None, None] * torch.eye(b, dtype=torch.complex128, device=om.device)
        self.inv = []
        S = self.D[0] + shift
        for i in range(nx):
            self.inv.append(torch.linalg.inv(S))
            if i + 1 < nx:
                S = self.D[i + 1] + shift - (self.W[i + 1][:, None] * self.inv[i]
                                             * self.E[i][None, :])

    def solve(self, B, adjoint=False):
        m, k, _ = B.shape
        nx, b, _ = self.D.shape
        R = B.reshape(m, k, nx, b)
        out = torch.empty_like(R)
        T = [v.conj() if adjoint else v.transpose(1, 2) for v in self.inv]
        low, up = (self.E, self.W) if adjoint else (self.W, self.E)
        for i in range(nx):
            r = R[:, :, i]
            if i:
                r = r - (low[i - 1] if adjoint else low[i]) * out[:, :, i - 1]
            out[:, :, i] = r @ T[i].contiguous()
        for i in range(nx - 2, -1, -1):
            r = (up[i + 1] if adjoint else up[i]) * out[:, :, i + 1]
            out[:, :, i] -= r @ T[i].contiguous()
        return out.reshape(m, k, nx * b)


def _philox(rows, cols, seed):
    """Philox4x32-10 at counters (row, column, 0, 0) under the key made of the seed: words 0..3."""
    M = np.uint64(0xFFFFFFFF)
    r, c = np.meshgrid(np.arange(rows, dtype=np.uint64), np.arange(cols, dtype=np.uint64),
                       indexing="ij")
    x = [r, c, np.zeros_like(r), np.zeros_like(r)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p, t = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(t >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), t & M,
             (p >> np.uint64(32)) ^ x[3] ^ np.uint64(k1), p & M]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x


def _theta(case, phi, seed):
    """The weighted complex normal test matrix, (k, n)."""
    n, k = 2 * case["nx"] * case["ny"], case["k"]
    x = _philox(n, k, seed)
    cut = [((x[i] << np.uint64(32)) | x[i + 1]) >> np.uint64(11) for i in (0, 2)]
    u1, u2 = (cut[0] + 1.0) * 2.0 ** -53, cut[1] * 2.0 ** -53  # in (0, 1] and [0, 1)
    w = np.sqrt(-np.log(u1)) * np.exp(2j * np.pi * u2)
    w = torch.from_numpy(np.ascontiguousarray(w.T)).to(phi.device)
    return w * phi.reshape(-1).repeat_interleave(2)


def _orth(Y):
    """Q of the QR with a positive real diagonal, for columns stored along the last axis."""
    Q, R = torch.linalg.qr(Y.transpose(1, 2))
    d = torch.diagonal(R, dim1=1, dim2=2)
    return (Q * (d / d.abs())[:, None, :]).transpose(1, 2)


def exact(case, seed):
    kind, k, q = case["kind"], case["k"], case["q"]
    if case["nx"] * case["ny"] * case["ny"] * case["shifts"] > 3e8 or kind == "sigma_one":
        return None
    U, domain, omegas = _setup(case, seed)
    op = _operator(case, U, domain)
    if kind == "apply":
        X = _block(case, seed).reshape(case["shifts"], k, case["nx"], 2 * case["ny"])
        D, E, W = _lines(op, omegas)
        om = torch.tensor(omegas, dtype=torch.float64, device=U.device)
        Y = 1j * om[:, None, None, None] * X
        for i in range(case["nx"]):
            Y[:, :, i] += X[:, :, i] @ D[i].T.contiguous()
        Y[:, :, :-1] += E[:-1] * X[:, :, 1:]
        Y[:, :, 1:] += W[1:] * X[:, :, :-1]
        return Y.reshape(case["shifts"], k, -1)
    A = _Direct(op, omegas)
    if kind in ("solve", "krylov"):
        return A.solve(_block(case, seed))
    if kind == "adjoint":
        return A.solve(_block(case, seed), adjoint=True)
    Q = _orth(A.solve(_theta(case, op["phi"], int(seed)).expand(len(omegas), -1, -1)))
    for _ in range(q):
        Q = _orth(A.solve(_orth(A.solve(Q, adjoint=True))))
    Z = A.solve(Q, adjoint=True)
    if kind == "project":
        return {"Q": Q, "Z": Z}
    _, sigma, Wh = torch.linalg.svd(Z.conj(), full_matrices=False)
    V = Wh.conj().contiguous()  # rows: the forcing modes, up to a phase each
    R = A.solve(V)
    gains = torch.linalg.norm(R, dim=2)
    out = {"sigma_B": sigma, "sigma_AV": gains}
    if kind == "sweep":
        return out
    out.update(_phased(V, R / gains[:, :, None], Q), Q=Q)
    return {**out, "Z": Z} if kind == "pass" else out

"""Timed workloads of the solver: what a program that uses the library has it do.

``listed()`` names the workloads, ``draw(rng)`` makes one more of the same ranges,
``prepare(case, seed)`` makes what the program holds before the call (matrix, right-hand
side, and for repeated solves the hierarchy), ``run(state)`` is one pass through the public
entry points, ``work(case)`` the bytes and operations a pass cannot do without and
``exact(case, seed)`` the solution from a plain 64-bit Krylov iteration in torch.

Kinds of use (``kind``):

* ``setup_solve``  a new matrix: hierarchy setup and one preconditioned CG solve.
* ``resetup``      new values on a kept pattern (a time step, a Newton step), then a solve.
* ``solve``        another right-hand side on a kept hierarchy.
* ``gmres``        the same for a nonsymmetric operator, by restarted GMRES.
* ``many``         several kept hierarchies solved together in lockstep.
* ``serve``        independent setup + solve requests from host arrays through the server.

Problem families (``family``), all on the GPU from torch (``serve``: on the host):

* ``fd5`` / ``fd7``  5- and 7-point finite volumes with geometrically graded last axis.
* ``cd7``            fd7 plus an upwinded constant velocity (nonsymmetric).
* ``kappa``          27-point trilinear elements, coefficients over six decades.
* ``mesh``           27-point trilinear elements on a randomly perturbed, 100:1 stretched
                     mesh, with node coordinates (distance-Laplacian strength).
* ``beam``           elastic cantilever, 3 unknowns per node, rigid-body modes.

Whole-number outputs (iterations, level sizes) and every eigenvalue estimate of the
hierarchy come back with the solution.  The final relative residual does not: it is the
rounding of a 1e-8 remainder, with few significant digits.
"""
from __future__ import annotations

import functools
import itertools
import math

import numpy as np
import torch

from paper_2103_10476_amd import problems, solver

DEV = "cuda"
F64 = torch.float64


def _case(name, kind, family, nx, ny, nz, variants="", precision="fp64", rtol=1e-8, count=1,
          aspect=1000.0):
    return {"name": name, "kind": kind, "family": family, "nx": nx, "ny": ny, "nz": nz,
            "variants": variants, "precision": precision, "rtol": rtol, "count": count,
            "aspect": aspect}


def listed():
    return [
        # the smallest call: a 2-D grid of 4,096 unknowns, bound by launches and readbacks
        _case("grid64_setup_solve", "setup_solve", "fd5", 64, 64, 1, aspect=100.0),
        # an ordinary small 3-D system with odd sides, all four prolongator adaptations
        _case("cube47_all_variants", "setup_solve", "fd7", 47, 45, 49,
              "sprsfy,offlmp,1norm,cnstrnt"),
        # the benchmark's cube: 2.1M unknowns, plain smoothed aggregation
        _case("cube128_setup_solve", "setup_solve", "fd7", 128, 128, 128),
        # the largest: 4.1M unknowns, FP32 V-cycle inside FP64 CG to 1e-10
        _case("cube160_fp32", "setup_solve", "fd7", 160, 160, 160, precision="fp32",
              rtol=1e-10),
        # heterogeneous coefficients, 970K unknowns, 27-point rows
        _case("kappa100_setup_solve", "setup_solve", "kappa", 100, 100, 100, "offlmp,1norm"),
        # unstructured-looking mesh with coordinates: distance-Laplacian strength
        _case("mesh60_coords", "setup_solve", "mesh", 60, 60, 60, "offlmp", rtol=1e-10),
        # elasticity: systems hierarchy with six rigid-body modes, 180K unknowns
        _case("beam96_systems", "setup_solve", "beam", 96, 24, 24),
        # a time step: new values on the kept pattern, odd sides, 872K unknowns
        _case("cube101_resetup", "resetup", "fd7", 101, 97, 89, "offlmp,1norm"),
        # another right-hand side on a kept hierarchy
        _case("cube96_solve", "solve", "fd7", 96, 96, 96),
        # a nonsymmetric operator, kept hierarchy, GMRES(30)
        _case("convection90_gmres", "gmres", "cd7", 90, 93, 87, "offlmp,1norm"),
        # eight kept hierarchies of different sizes solved together, FP32 V-cycle
        _case("many8_fp32", "many", "fd7", 40, 40, 40, "offlmp,1norm", "fp32", 1e-10, count=8),
        # a dozen serving requests from host arrays
        _case("serve12", "serve", "fd7", 40, 40, 40, "offlmp,1norm", "fp32", 1e-10, count=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds, families and ranges."""
    kind, family = rng.choice([("setup_solve", "fd5"), ("setup_solve", "fd7"),
                               ("setup_solve", "fd7"), ("setup_solve", "kappa"),
                               ("setup_solve", "mesh"), ("setup_solve", "beam"),
                               ("resetup", "fd7"), ("solve", "fd7"), ("gmres", "cd7"),
                               ("many", "fd7"), ("serve", "fd7")])
    variants = rng.choice(["offlmp,1norm", "1norm", "offlmp,1norm,cnstrnt",
                           "sprsfy,offlmp,1norm"])
    precision = rng.choice(["fp64", "fp32"])
    count, aspect = 1, 10.0 ** rng.uniform(1.0, 3.0)
    if family == "fd5":
        side = _log_int(rng, 48, 700)
        n = (side, max(32, side + rng.randint(-15, 15)), 1)
    elif family == "beam":
        side = rng.randint(8, 24)
        n, variants = (side * rng.randint(2, 4), side, side), ""
    elif kind in ("many", "serve"):
        side, count = rng.randint(20, 44), rng.randint(3, 12)
        n, variants = (side, side, side), "offlmp,1norm"
    else:
        hi = {"kappa": 96, "mesh": 60}.get(family, 124)
        side = _log_int(rng, 20, hi)
        n = tuple(min(hi, max(18, side + rng.randint(-4, 4))) for _ in range(3))
        if family == "kappa":
            variants = rng.choice(["offlmp,1norm", "offlmp,1norm,cnstrnt"])
        if family == "mesh":
            variants = rng.choice(["offlmp", "offlmp,1norm"])
    if family == "cd7":
        variants = "offlmp,1norm"
    c = _case("", kind, family, *n, variants, precision, rng.choice([1e-8, 1e-10]), count,
              round(aspect, 2))
    del c["name"]
    return c


# --------------------------------------------------------------------------------------
# Problems, assembled on the GPU
# --------------------------------------------------------------------------------------

def _rng(seed, salt=0):
    return np.random.Generator(np.random.PCG64([int(seed) & 0xFFFFFFFF, salt]))


def _stencil_csr(shape, offsets, coeff):
    """CSR of a structured stencil: unknowns of a (x, y, z) grid, x fastest; ``coeff[t]`` (of
    shape (z, y, x)) couples each unknown to its neighbour at ``offsets[t]``; couplings that
    leave the grid are not stored."""
    nx, ny, nz = shape
    order = sorted(range(len(offsets)),
                   key=lambda t: offsets[t][0] + nx * (offsets[t][1] + ny * offsets[t][2]))
    ax = [torch.arange(m, device=DEV) for m in (nx, ny, nz)]
    ok = torch.empty(nz, ny, nx, len(order), dtype=torch.bool, device=DEV)
    val = torch.empty(nz, ny, nx, len(order), dtype=F64, device=DEV)
    col = torch.empty(nz, ny, nx, len(order), dtype=torch.int32, device=DEV)
    idx = torch.arange(nx * ny * nz, device=DEV).reshape(nz, ny, nx)
    for k, t in enumerate(order):
        d = offsets[t]
        inside = [((a + s) >= 0) & ((a + s) < m) for a, s, m in zip(ax, d, (nx, ny, nz))]
        ok[..., k] = (inside[2][:, None, None] & inside[1][None, :, None]
                      & inside[0][None, None, :])
        val[..., k] = coeff[t]
        col[..., k] = idx + (d[0] + nx * (d[1] + ny * d[2]))
    n = nx * ny * nz
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(ok.reshape(n, -1).sum(1), 0)
    return n, rp, col[ok], val[ok]


def _fd(case, velocity=None):
    """5- or 7-point finite volumes of problems.fd5_stretched / fd7_stretched, with the
    upwinded velocity of problems.cd7_upwind when one is given."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    flat = case["family"] == "fd5"
    if flat:
        ny, nz = 1, ny
    h = 1.0 / (nx + 1)
    hz = torch.from_numpy(problems.graded_spacing(nz, case["aspect"])).to(DEV)
    dz = (0.5 * (hz[:-1] + hz[1:]))[:, None, None]
    lo, up = hz[:-1][:, None, None], hz[1:][:, None, None]
    if flat:
        side, down, up = dz / h, h / lo, h / up
        diag = 2.0 * side + down + up
        offs = [(0, 0, -1), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 0, 1)]
        return _stencil_csr((nx, ny, nz), offs, [-down, -side, diag, -side, -up])
    side, down, up = dz, h * h / lo, h * h / up
    diag = 4.0 * side + down + up
    offs = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    if velocity is None:
        return _stencil_csr((nx, ny, nz), offs, [-down, -side, -side, diag, -side, -side, -up])
    qx, qy, qz = velocity[0] * h * dz, velocity[1] * h * dz, velocity[2] * h * h
    return _stencil_csr((nx, ny, nz), offs, [-down - qz, -side - qy, -side - qx,
                                             diag + qx + qy + qz, -side, -side, -up])


def _hex_csr(K):
    """27-point stiffness of the interior nodes of a grid of hexahedra; ``K`` holds the
    element matrices, (z, y, x, 8, 8)."""
    ez, ey, ex = K.shape[:3]
    offs = list(itertools.product((-1, 0, 1), repeat=3))
    coeff = []
    for d in offs:
        c = torch.zeros(ez - 1, ey - 1, ex - 1, dtype=F64, device=DEV)
        for e in itertools.product((0, 1), repeat=3):
            a = [1 - v for v in e]
            b = [s + t for s, t in zip(a, d)]
            if min(b) < 0 or max(b) > 1:
                continue
            c += K[e[2]:ez - 1 + e[2], e[1]:ey - 1 + e[1], e[0]:ex - 1 + e[0],
                   a[0] + 2 * a[1] + 4 * a[2], b[0] + 2 * b[1] + 4 * b[2]]
        coeff.append(c)
    return _stencil_csr((ex - 1, ey - 1, ez - 1), offs, coeff)


def _kappa(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    K = torch.tensor([[float(v) for v in r] for r in problems.q1_element_matrix(
        1.0 / case["nx"], 1.0 / case["nx"], 1.0 / case["nx"])], dtype=F64, device=DEV)
    kappa = 10.0 ** _rng(seed, 1).uniform(-3.0, 3.0, size=shape)
    return _hex_csr(torch.from_numpy(kappa).to(DEV)[..., None, None] * K)


def _mesh(case, seed):
    """Perturbed cube of problems.perturbed_cube_nodes' recipe: (csr, interior coordinates)."""
    m = (case["nz"], case["ny"], case["nx"])
    base = np.stack(np.meshgrid(*[np.arange(k + 1) / k for k in m], indexing="ij")[::-1], -1)
    move = 0.2 * _rng(seed, 2).uniform(size=base.shape) / np.asarray(m[::-1])
    X = torch.from_numpy((base + move) * np.array([1.0, 1.0, 100.0])).to(DEV)
    corner = [(a & 1, (a >> 1) & 1, (a >> 2) & 1) for a in range(8)]
    P = [X[c[2]:m[0] + c[2], c[1]:m[1] + c[1], c[0]:m[2] + c[0]] for c in corner]
    K = torch.zeros(*m, 8, 8, dtype=F64, device=DEV)
    g = 1.0 / math.sqrt(3.0)
    for q in itertools.product((-g, g), repeat=3):
        dN = []
        for c in corner:
            s = [2 * v - 1 for v in c]
            f = [1.0 + s[k] * q[k] for k in range(3)]
            dN.append([s[0] * f[1] * f[2] / 8, f[0] * s[1] * f[2] / 8, f[0] * f[1] * s[2] / 8])
        J = [sum(P[a] * dN[a][k] for a in range(8)) for k in range(3)]  # dx / dxi_k
        C = [torch.linalg.cross(J[1], J[2]), torch.linalg.cross(J[2], J[0]),
             torch.linalg.cross(J[0], J[1])]
        det = (J[0] * C[0]).sum(-1)
        G = [sum(C[k] * dN[a][k] for k in range(3)) / det[..., None] for a in range(8)]
        for a in range(8):
            for b in range(8):
                K[..., a, b] += det * (G[a] * G[b]).sum(-1)
    return _hex_csr(K), X[1:-1, 1:-1, 1:-1].reshape(-1, 3).contiguous()


@functools.lru_cache(maxsize=1)
def _beam(nx, ny, nz):
    p, _, modes = problems.elastic_beam(nx, ny, nz, 5.0)
    return p, modes


def _problem(case, seed):
    """(n, rp, col, val) on the GPU and what else the setup takes.  The seed scales the
    operator's values (a material constant) where it does not decide the coefficients."""
    scale = float(_rng(seed, 3).uniform(0.5, 2.0))
    family, extra = case["family"], {}
    if family == "kappa":
        A = _kappa(case, seed)
    elif family == "mesh":
        A, extra["coords"] = _mesh(case, seed)
    elif family == "beam":
        p, modes = _beam(case["nx"], case["ny"], case["nz"])
        A = (p.n, *(torch.from_numpy(v).to(DEV) for v in (p.rp, p.col, p.val)))
        extra.update(nullspace=torch.from_numpy(modes).to(DEV), block_size=3)
    else:
        A = _fd(case, (1.0, 0.5, 0.25) if family == "cd7" else None)
    return (A[0], A[1], A[2], A[3] * scale), extra


def _rhs(n, seed, salt=4):
    return torch.from_numpy(_rng(seed, salt).uniform(-1.0, 1.0, size=n)).to(DEV)


def _rows(A):
    return torch.repeat_interleave(torch.arange(A[0], device=DEV), (A[1][1:] - A[1][:-1]).long())


def _stepped(A, seed):
    """The next time step's values on A's pattern: another step length and a reaction term
    that adds up to 5% to each diagonal entry."""
    n, rp, col, val = A
    rows = _rows(A)
    more = 1.0 + 0.05 * (_rhs(n, seed, 5) + 1.0) / 2.0
    return torch.where(rows == col, val * more[rows], val) * float(_rng(seed, 6).uniform(0.5, 2))


def _options(case):
    family = case["family"]
    return solver.Options(
        theta=0.025 if family == "mesh" else 0.02,
        variants=[v for v in case["variants"].split(",") if v], precision=case["precision"],
        rtol=case["rtol"], cheb_boost=1.1 if case["variants"] or family == "beam" else 1.0,
        dist_power=2 if family == "mesh" else 1,
        coarse_solver="lu" if family == "cd7" else "cholesky")


def _members(case):
    """The systems of a ``many`` or ``serve`` case: sides from 16 up to the case's, and
    gradings, in a fixed order."""
    for k in range(case["count"]):
        side = 16 + (case["nx"] - 16) * ((5 * k) % case["count"]) // max(1, case["count"] - 1)
        yield k, dict(case, nx=side, ny=side, nz=side, aspect=10.0 ** (1.0 + (k % 5) / 2.0))


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind, "options": _options(case)}
    if kind in ("many", "serve"):
        state["systems"] = []
        for k, c in _members(case):
            A, _ = _problem(c, seed + 1000 * k)
            state["systems"].append((A, _rhs(A[0], seed + 1000 * k)))
        if kind == "many":
            state["handles"] = [solver.setup(A, options=state["options"])
                                for A, _ in state["systems"]]
        else:
            state["systems"] = [((A[0], *(v.cpu().numpy() for v in A[1:])), b.cpu().numpy())
                                for A, b in state["systems"]]
            state["server"] = solver.Server(hbm_budget=8 << 30, max_slots=4)
        return state
    state["A"], state["extra"] = _problem(case, seed)
    state["b"] = _rhs(state["A"][0], seed)
    if kind != "setup_solve":
        state["handle"] = solver.Hierarchy(*state["A"], options=state["options"],
                                           **state["extra"])
    if kind == "resetup":  # a program that steps in time has made a step before
        n, rp, col, val = state["A"]
        state["handle"].resetup(val)
        state["values"] = _stepped(state["A"], seed)
    return state


def _hierarchy_outputs(h):
    info = h.info()
    return {k: info[k] for k in ("n", "nnz", "nnz_p", "lambda", "omega", "smoother_lambda")}


def run(state):
    kind = state["kind"]
    if kind == "setup_solve":
        h = solver.Hierarchy(*state["A"], options=state["options"], **state["extra"])
        x, iterations, _, _ = h.solve(state["b"])
        return {"x": x, "iterations": iterations, **_hierarchy_outputs(h)}
    if kind == "resetup":
        h = state["handle"]
        h.resetup(state["values"])
        x, iterations, _, _ = h.solve(state["b"])
        return {"x": x, "iterations": iterations, **_hierarchy_outputs(h)}
    if kind == "solve":
        x, iterations, _, _ = state["handle"].solve(state["b"])
        return {"x": x, "iterations": iterations}
    if kind == "gmres":
        x, iterations, _, _ = state["handle"].solve_gmres(state["b"])
        return {"x": x, "iterations": iterations}
    if kind == "many":
        got = solver.solve_many(state["handles"], [b for _, b in state["systems"]])
        return {"x": [g[0] for g in got], "iterations": [g[1] for g in got]}
    server = state["server"]
    tickets = [server.submit(A, b, state["options"], borrow=True) for A, b in state["systems"]]
    got = [server.wait(t, A[0]) for t, (A, _) in zip(tickets, state["systems"])]
    return {"x": [x for x, _ in got], "iterations": [r["iterations"] for _, r in got]}


# --------------------------------------------------------------------------------------
# What a pass cannot do without, and the solution in 64 bits
# --------------------------------------------------------------------------------------

def _size(case):
    """(unknowns, stored entries) of a case's matrix."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if case["family"] == "fd5":
        return nx * ny, 5 * nx * ny - 2 * nx - 2 * ny
    if case["family"] in ("kappa", "mesh"):
        return ((nx - 1) * (ny - 1) * (nz - 1),
                (3 * nx - 5) * (3 * ny - 5) * (3 * nz - 5))
    if case["family"] == "beam":
        return (3 * nx * (ny + 1) * (nz + 1),
                9 * (3 * nx - 2) * (3 * ny + 1) * (3 * nz + 1))
    return nx * ny * nz, 7 * nx * ny * nz - 2 * (nx * ny + ny * nz + nx * nz)


def work(case):
    """The matrix and right-hand side read once, the solution written once; one product with
    the matrix is the least that tells a solution from another vector."""
    systems = ([c for _, c in _members(case)] if case["kind"] in ("many", "serve") else [case])
    sizes = [_size(c) for c in systems]
    return {"bytes": float(sum(12 * nnz + 4 * (n + 1) + 16 * n for n, nnz in sizes)),
            "flops": float(sum(2 * nnz for _, nnz in sizes))}


def _krylov(A, b, symmetric):
    """The solution of A x = b by Jacobi-preconditioned CG (BiCGStab for a nonsymmetric A),
    restarted on the true residual until that stops falling."""
    n, rp, col, val = A
    M = torch.sparse_csr_tensor(rp, col, val, size=(n, n))
    rows = _rows(A)
    inv = torch.empty(n, dtype=F64, device=DEV)
    on_diagonal = rows == col
    inv[rows[on_diagonal]] = 1.0 / val[on_diagonal]
    x, best, goal = torch.zeros_like(b), math.inf, float(b.norm())
    for _ in range(6):
        r = b - M @ x
        left = float(r.norm())
        if left > 0.5 * best or left < 1e-15 * goal:
            break
        best = left
        r0, dx = r.clone(), torch.zeros_like(b)
        z = inv * r
        p, rho = (z.clone(), r @ z) if symmetric else (r.clone(), r0 @ r)
        for step in range(20000):
            if symmetric:
                q = M @ p
                alpha = rho / (p @ q)
                dx += alpha * p
                r -= alpha * q
                z = inv * r
                last, rho = rho, r @ z
                p = z + (rho / last) * p
            else:
                y = inv * p
                v = M @ y
                alpha = rho / (r0 @ v)
                s = r - alpha * v
                w = inv * s
                t = M @ w
                omega = (t @ s) / (t @ t)
                dx += alpha * y + omega * w
                r = s - omega * t
                last, rho = rho, r0 @ r
                p = r + (rho / last) * (alpha / omega) * (p - omega * v)
            if step % 25 == 24 and not float(r.norm()) > 1e-9 * left:
                break
        x = x + dx
    return x


def exact(case, seed):
    if case["kind"] in ("many", "serve"):
        xs = []
        for k, c in _members(case):
            A, _ = _problem(c, seed + 1000 * k)
            xs.append(_krylov(A, _rhs(A[0], seed + 1000 * k), True))
        return {"x": xs}
    A, _ = _problem(case, seed)
    b = _rhs(A[0], seed)
    if case["kind"] == "resetup":
        A = (*A[:3], _stepped(A, seed))
    return {"x": _krylov(A, b, case["family"] != "cd7")}

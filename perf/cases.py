"""The timed workloads of the solver library: seeded finite-volume systems on
boxes of hexahedra, each taken through the package's public entry points.

`listed()` names the cases, `draw(rng)` gives others of the same ranges,
`prepare(case, seed)` builds the device inputs and the handles a program keeps
(mesh, matrix, hierarchy, batch), `run(state)` is one pass, `work(case)` what a
pass cannot do without, and `exact(case, seed)` the outputs by a plain torch
FP64 implementation on the structured grid.

Inputs follow the recipes of `fvcases` (unit and lognormal conductivities, the
graded cavity, the upwind momentum system, the transient heat equation, the
lid-driven PISO box, batches of uneven cubes), drawn on the GPU.  Cells are
numbered naturally, or by levels i + j + k with each level in natural order:
the Cuthill-McKee order of a box, whose bandwidth is that of the permuted and
RCM-renumbered meshes the benchmark uses (27.7k rows at 192^3).

Solves go to tight tolerances (1e-10 and below), so that the solution is fixed
well beyond the rounding of any one summation order.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1505_07630_amd as fv

DEV = "cuda"
F64 = torch.float64


# ----------------------------------------------------------------- the cases

def listed():
    return [
        # smallest call: a coarse mesh solved once, bound by launches and host round trips
        {"name": "pipecg_12x12x12", "kind": "solve", "nx": 12, "ny": 12, "nz": 12, "coef": "unit", "order": "natural",
         "method": "pipecg", "precond": "jacobi", "tol": 1e-10},
        # the 32^3 Laplace cube: the usual small serving-size solve
        {"name": "pipecg_laplace32", "kind": "solve", "nx": 32, "ny": 32, "nz": 32, "coef": "unit", "order": "natural",
         "method": "pipecg", "precond": "jacobi", "tol": 1e-10},
        # standard CG on a ragged mid-size mesh in Cuthill-McKee order
        {"name": "cg_61x67x64", "kind": "solve", "nx": 61, "ny": 67, "nz": 64, "coef": "lognormal", "order": "levels",
         "method": "cg", "precond": "jacobi", "tol": 1e-11},
        # the headline workload: 7.08M cells, lognormal conductivities, folded pipelined Jacobi-PCG
        {"name": "pipecg_varcoef192", "kind": "solve", "nx": 192, "ny": 192, "nz": 192, "coef": "lognormal",
         "order": "levels", "method": "pipecg", "precond": "jacobi", "tol": 1e-10},
        # FP32 iterations re-anchored to the FP64 residual
        {"name": "mixed_128x120x136", "kind": "mixed", "nx": 128, "ny": 120, "nz": 136, "coef": "lognormal",
         "order": "levels", "update_every": 16, "tol": 1e-11},
        # icoFoam's momentum predictor: three velocity components by BiCGSTAB
        {"name": "momentum3_128", "kind": "momentum", "nx": 128, "ny": 128, "nz": 128, "order": "levels", "ncomp": 3,
         "precond": "jacobi", "tol": 1e-11},
        # laplacianFoam's time loop: assemble, refresh, solve from the previous field
        {"name": "transient_96x100x104", "kind": "transient", "nx": 96, "ny": 100, "nz": 104, "order": "levels",
         "steps": 4, "method": "pipecg", "tol": 1e-10},
        # AMG-PCG with the hierarchy already built (the same system solved again and again)
        {"name": "amg_varcoef192", "kind": "amg", "nx": 192, "ny": 192, "nz": 192, "coef": "lognormal",
         "order": "levels", "method": "cg", "tol": 1e-11},
        # one-off AMG solve of the graded cavity's pressure equation: matrix, hierarchy and solve
        {"name": "amg_setup_cavity128", "kind": "amg_setup", "nx": 128, "ny": 128, "nz": 32, "coef": "cavity",
         "order": "natural", "method": "cg", "tol": 1e-11},
        # an icoFoam PISO step: momentum, hierarchy refresh, two pressure correctors
        {"name": "piso_amg_96", "kind": "piso", "nx": 96, "ny": 96, "nz": 96, "order": "levels", "pressure": "amg",
         "steps": 1, "tol": 1e-11},
        # many uneven systems in one persistent launch
        {"name": "batch_48", "kind": "batch", "nsys": 48, "edge_lo": 16, "edge_hi": 64, "sizes": 5,
         "method": "pipecg", "tol": 1e-10},
        # a differentiable solve: forward and adjoint with all gradients
        {"name": "autograd_40x36x44", "kind": "autograd", "nx": 40, "ny": 36, "nz": 44, "coef": "lognormal",
         "order": "natural", "method": "pipecg", "tol": 1e-11},
    ]


def _box(rng, lo, hi):
    """A ragged box of about n cells, log(n) uniform over [lo, hi]."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    a, b = math.exp(rng.uniform(-0.3, 0.3)), math.exp(rng.uniform(-0.3, 0.3))
    e = n ** (1.0 / 3.0)
    nx, ny = max(4, round(e * a)), max(4, round(e * b))
    nz = max(4, round(n / (nx * ny)))
    while nx * ny * nz > hi:
        nz -= 1
    return {"nx": nx, "ny": ny, "nz": nz}


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "mixed", "momentum", "transient", "amg", "amg_setup", "piso",
                       "batch", "autograd"])
    order = rng.choice(["natural", "levels"])
    if kind == "solve":
        method = rng.choice(["pipecg", "pipecg", "cg", "cg", "pipecg_literal"])
        precond = "jacobi" if method == "pipecg_literal" else rng.choice(["jacobi", "jacobi", "jacobi", "none"])
        coef = "unit" if precond == "none" else rng.choice(["unit", "lognormal", "lognormal"])
        return {"kind": kind, **_box(rng, 1500, 1200000 if precond == "none" else 4500000), "coef": coef,
                "order": order, "method": method, "precond": precond, "tol": 1e-10}
    if kind == "mixed":
        return {"kind": kind, **_box(rng, 30000, 4000000), "coef": "lognormal", "order": order,
                "update_every": rng.choice([10, 16]), "tol": 1e-11}
    if kind == "momentum":
        return {"kind": kind, **_box(rng, 8000, 6000000), "order": order, "ncomp": rng.randint(1, 3),
                "precond": "jacobi", "tol": 1e-11}
    if kind == "transient":
        return {"kind": kind, **_box(rng, 8000, 4000000), "order": order, "steps": rng.randint(2, 5),
                "method": rng.choice(["pipecg", "cg"]), "tol": 1e-10}
    if kind == "amg":
        return {"kind": kind, **_box(rng, 30000, 6000000), "coef": rng.choice(["lognormal", "unit"]), "order": order,
                "method": rng.choice(["cg", "cg", "pipecg"]), "tol": 1e-11}
    if kind == "amg_setup":
        coef = rng.choice(["lognormal", "cavity"])
        return {"kind": kind, **_box(rng, 30000, 900000 if coef == "cavity" else 4000000), "coef": coef,
                "order": "natural" if coef == "cavity" else order, "method": "cg", "tol": 1e-11}
    if kind == "piso":
        pressure = rng.choice(["amg", "amg", "jacobi"])
        return {"kind": kind, **_box(rng, 8000, 1500000 if pressure == "amg" else 300000), "order": order,
                "pressure": pressure, "steps": rng.randint(1, 2), "tol": 1e-11}
    if kind == "batch":
        lo = rng.randint(6, 24)
        return {"kind": kind, "nsys": rng.randint(8, 96), "edge_lo": lo, "edge_hi": rng.randint(lo + 4, 64),
                "sizes": rng.randint(0, 10 ** 6), "method": rng.choice(["pipecg", "cg"]), "tol": 1e-10}
    return {"kind": kind, **_box(rng, 2000, 1000000), "coef": "lognormal", "order": order,
            "method": rng.choice(["pipecg", "cg"]), "tol": 1e-11}


# ----------------------------------------------------------------- structured inputs

class _Gen:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed))

    def uniform(self, *shape, lo=-1.0, hi=1.0):
        return torch.rand(*shape, generator=self.g, device=DEV, dtype=F64) * (hi - lo) + lo

    def lognormal(self, *shape):
        return torch.exp(torch.randn(*shape, generator=self.g, device=DEV, dtype=F64))


AXES = (2, 1, 0)  # the grid dimension of x, y, z in a (nz, ny, nx) array


def _lo(a, d):
    """The owner side of the faces normal to axis d (0 = x): all but the last."""
    return a.narrow(AXES[d], 0, a.shape[AXES[d]] - 1)


def _hi(a, d):
    return a.narrow(AXES[d], 1, a.shape[AXES[d]] - 1)


def _side(a, d, high):
    return a.select(AXES[d], a.shape[AXES[d]] - 1 if high else 0)


class Grid:
    """Addressing of an nx x ny x nz box: LDU faces in (owner, neighbour)
    order, the numbering, and the maps from structured arrays to both."""

    def __init__(self, case):
        nx, ny, nz = self.shape = case["nx"], case["ny"], case["nz"]
        n = self.n = nx * ny * nz
        c = torch.arange(n, device=DEV).view(nz, ny, nx)
        if case["order"] == "levels":
            k, j, i = torch.meshgrid(torch.arange(nz, device=DEV), torch.arange(ny, device=DEV),
                                     torch.arange(nx, device=DEV), indexing="ij")
            by = torch.argsort(((i + j + k).view(-1) * n + c.view(-1)))
            self.new = torch.empty_like(by)
            self.new[by] = torch.arange(n, device=DEV)
        else:
            self.new = c.reshape(-1)
        num = self.new.view(nz, ny, nx)
        o = torch.cat([_lo(num, d).reshape(-1) for d in range(3)])
        m = torch.cat([_hi(num, d).reshape(-1) for d in range(3)])  # every numbering here keeps owner < neighbour
        self.fcount = [_lo(num, d).numel() for d in range(3)]
        self.forder = torch.argsort(o * n + m)
        self.owner = o[self.forder].to(torch.int32)
        self.nb = m[self.forder].to(torch.int32)
        self.F = int(o.numel())

    def cells(self, a):
        """A (..., nz, ny, nx) array in the numbering, flat per leading index."""
        flat = a.reshape(*a.shape[:-3], self.n)
        out = torch.empty_like(flat)
        out[..., self.new] = flat
        return out.contiguous()

    def faces(self, three):
        """Three structured face arrays (x, y, z) in LDU order."""
        return torch.cat([t.reshape(-1) for t in three])[self.forder].contiguous()

    def box(self, v):
        """The inverse of cells()."""
        nx, ny, nz = self.shape
        return v[..., self.new].reshape(*v.shape[:-1], nz, ny, nx)


def _row_sums(upper, lower, extra):
    """diag = -sum of the row's off-diagonal entries + extra."""
    diag = extra.clone()
    for d in range(3):
        _lo(diag, d).sub_(upper[d])
        _hi(diag, d).sub_(lower[d])
    return diag


def _face_shapes(shape):
    nx, ny, nz = shape
    return [(nz, ny, nx - 1), (nz, ny - 1, nx), (nz - 1, ny, nx)]


def _laplacian(case, seed):
    """Structured (diag, upper[3], b) of a diffusion system."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    shape, g = (nz, ny, nx), _Gen(seed)
    zero = torch.zeros(shape, device=DEV, dtype=F64)
    if case["coef"] == "unit":
        up = [torch.full(s, -1.0, device=DEV, dtype=F64) for s in _face_shapes((nx, ny, nz))]
        _side(zero, 2, False).add_(2.0)
        return _row_sums(up, up, zero), up, g.uniform(*shape)
    if case["coef"] == "lognormal":
        up = [-g.lognormal(*s) for s in _face_shapes((nx, ny, nz))]
        _side(zero, 0, False).add_(2.0 * g.lognormal(nz, ny))
        _side(zero, 0, True).add_(2.0 * g.lognormal(nz, ny))
        return _row_sums(up, up, zero), up, g.uniform(*shape)
    # the graded cavity: heights shrink by 1.02 per cell toward y-max, Neumann walls, cell 0 pinned
    h = 1.0 / nx
    dy = 1.02 ** (-torch.arange(ny, device=DEV, dtype=F64))
    dy = dy / dy.sum()
    dyc = dy.view(1, ny, 1)
    mid = (0.5 * (dy[1:] + dy[:-1])).view(1, ny - 1, 1)
    fs = _face_shapes((nx, ny, nz))
    w = [(dyc * h / h).expand(fs[0]), (h * h / mid).expand(fs[1]), (dyc * h / h).expand(fs[2])]
    area = [(dyc * h).expand(fs[0]), torch.full(fs[1], h * h, device=DEV, dtype=F64), (dyc * h).expand(fs[2])]
    up = [-t.contiguous() for t in w]
    diag = _row_sums(up, up, zero)
    for d in range(3):
        up[d].view(-1)[0] = 0.0  # the faces of cell 0
    U = g.uniform(3, *shape)
    b = torch.zeros(shape, device=DEV, dtype=F64)
    for d in range(3):
        phi = 0.5 * (_lo(U[d], d) + _hi(U[d], d)) * area[d]
        _lo(b, d).sub_(phi)
        _hi(b, d).add_(phi)
    b -= b.mean()
    b.view(-1)[0] = 0.0
    return diag, up, b


def _vortex_flux(shape, h, theta):
    """Face fluxes of curl(psi e_z), exact psi differences: no net outflow."""
    nx, ny, nz = shape
    Ly, Lz = ny * h, nz * h
    a = 1.0 / (1.5 * math.pi * max(1.0, 1.0 / Ly))
    ar = lambda m: torch.arange(m, device=DEV, dtype=F64)  # noqa: E731
    zc = 1.0 + 0.5 * torch.sin(2.0 * math.pi * ((ar(nz) + 0.5) * h) / Lz + theta)
    node = a * torch.sin(math.pi * ar(ny + 1) * h / Ly).view(-1, 1) * torch.sin(math.pi * ar(nx + 1) * h).view(1, -1)
    fx = (node[1:, 1:nx] - node[:-1, 1:nx]) * h
    fy = -(node[1:ny, 1:] - node[1:ny, :-1]) * h
    return [(zc.view(-1, 1, 1) * fx).contiguous(), (zc.view(-1, 1, 1) * fy).contiguous(),
            torch.zeros(nz - 1, ny, nx, device=DEV, dtype=F64)]


def _convection(phi, D, extra):
    """Upwind (diag, upper[3], lower[3]) of fluxes phi and diffusion D."""
    up = [-D - torch.clamp(-p, min=0.0) for p in phi]
    lo = [-D - torch.clamp(p, min=0.0) for p in phi]
    diag = extra.clone()
    for d in range(3):
        _lo(diag, d).add_(D + torch.clamp(phi[d], min=0.0))
        _hi(diag, d).add_(D + torch.clamp(-phi[d], min=0.0))
    return diag, up, lo


def _walls(shape, value):
    """value per wall face of each cell."""
    nx, ny, nz = shape
    w = torch.zeros(nz, ny, nx, device=DEV, dtype=F64)
    for d in range(3):
        _side(w, d, False).add_(value)
        _side(w, d, True).add_(value)
    return w


def _momentum(case, seed):
    nx, ny, nz = shape = case["nx"], case["ny"], case["nz"]
    g, h, nu = _Gen(seed), 1.0 / case["nx"], 0.01
    theta = 2.0 * math.pi * float(np.random.default_rng(seed).random())
    D, dt, vol = nu * h, 2.0 * h, h ** 3
    phi = _vortex_flux(shape, h, theta)
    diag, up, lo = _convection(phi, D, _walls(shape, 2.0 * D) + vol / dt)
    b = vol / dt * g.uniform(case["ncomp"], nz, ny, nx) + vol * g.uniform(case["ncomp"], nz, ny, nx)
    _side(b[0], 1, True).add_(2.0 * D)
    return diag, up, lo, b


def _transient(case, seed):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    g = _Gen(seed)
    k = [g.lognormal(*s) for s in _face_shapes((nx, ny, nz))]
    kl, kh = 2.0 * g.lognormal(nz, ny), 2.0 * g.lognormal(nz, ny)
    bdiag = torch.zeros(nz, ny, nx, device=DEV, dtype=F64)
    bsrc = g.uniform(nz, ny, nx, lo=0.5, hi=1.0)
    _side(bdiag, 0, False).add_(kl)
    _side(bdiag, 0, True).add_(kh)
    _side(bsrc, 0, False).add_(kl)
    return k, bdiag, bsrc, 0.25


def _piso(case, seed):
    nx, ny, nz = shape = case["nx"], case["ny"], case["nz"]
    h, nu = 1.0 / nx, 0.01
    theta = 2.0 * math.pi * float(np.random.default_rng(seed).random())
    phi = _vortex_flux(shape, h, theta)
    U = torch.zeros(3, nz, ny, nx, device=DEV, dtype=F64)
    bgrad = torch.zeros(3, nz, ny, nx, device=DEV, dtype=F64)
    blid = torch.zeros(nz, ny, nx, device=DEV, dtype=F64)
    for d in range(3):
        _lo(U[d], d).add_(0.5 * phi[d] / h ** 2)
        _hi(U[d], d).add_(0.5 * phi[d] / h ** 2)
        _side(bgrad[d], d, False).add_(-1.0)
        _side(bgrad[d], d, True).add_(1.0)
    _side(blid, 1, True).add_(2.0 * nu * h)
    return phi, U, _walls(shape, 2.0 * nu * h), blid, bgrad, h, nu


def _batch_edges(case):
    return np.random.default_rng(case["sizes"]).integers(case["edge_lo"], case["edge_hi"] + 1,
                                                         size=case["nsys"]).tolist()


def _batch_systems(case, seed):
    for s, e in enumerate(_batch_edges(case)):
        one = {"nx": e, "ny": e, "nz": e, "coef": "lognormal", "order": "natural"}
        yield (one, *_laplacian(one, seed * 1000 + s))


# ----------------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "batch":
        parts, addr = {"d": [], "u": [], "b": [], "o": [], "m": []}, {}
        coff, foff = [0], [0]
        for one, diag, up, b in _batch_systems(case, seed):
            e = one["nx"]
            if e not in addr:
                addr[e] = Grid(one)
            g = addr[e]
            parts["d"].append(g.cells(diag))
            parts["u"].append(g.faces(up))
            parts["b"].append(g.cells(b))
            parts["o"].append(g.owner)
            parts["m"].append(g.nb)
            coff.append(coff[-1] + g.n)
            foff.append(foff[-1] + g.F)
        c = {k: torch.cat(v) for k, v in parts.items()}
        s["B"] = fv.Batch(coff, foff, c["o"], c["m"], c["d"], c["u"])
        s["b"] = c["b"]
        return s
    g = Grid(case)
    mesh = s["mesh"] = fv.Mesh(g.n, g.owner, g.nb)
    if kind == "momentum":
        diag, up, lo, b = _momentum(case, seed)
        s["A"] = fv.Matrix(mesh, g.cells(diag), g.faces(up), g.faces(lo))
        s["b"] = g.cells(b)
        return s
    if kind == "transient":
        k, bdiag, bsrc, dt = _transient(case, seed)
        s["k"], s["bdiag"], s["bsrc"], s["dt"] = g.faces(k), g.cells(bdiag), g.cells(bsrc), dt
        s["w"] = torch.ones(g.F, device=DEV, dtype=F64)
        s["vol"] = torch.ones(g.n, device=DEV, dtype=F64)
        s["T0"] = torch.zeros(g.n, device=DEV, dtype=F64)
        diag, upper, _ = fv.assemble_transient(mesh, s["k"], s["w"], s["vol"], s["bdiag"], s["bsrc"], dt, s["T0"])
        s["A"] = fv.Matrix(mesh, diag, upper)
        return s
    if kind == "piso":
        phi, U, bwall, blid, bgrad, h, nu = _piso(case, seed)
        axis = [torch.full(t.shape, d, device=DEV, dtype=torch.int8) for d, t in enumerate(phi)]
        s["ps"] = fv.Piso(mesh, g.faces(axis), torch.ones(g.F, device=DEV, dtype=torch.int8), g.cells(bwall),
                          g.cells(blid), g.cells(bgrad), h, nu, pressure_solver=case["pressure"])
        s["U0"], s["phi0"], s["dt"] = g.cells(U), g.faces(phi), h
        s["p0"] = torch.zeros(g.n, device=DEV, dtype=F64)
        return s
    diag, up, b = _laplacian(case, seed)
    diag, upper, b = g.cells(diag), g.faces(up), g.cells(b)
    s["b"] = b
    if kind == "autograd":
        s["target"] = g.cells(_Gen(seed + 7919).uniform(case["nz"], case["ny"], case["nx"]))
        s["leaves"] = [t.requires_grad_(True) for t in (diag, upper, b)]
    elif kind == "amg_setup":
        s["diag"], s["upper"] = diag, upper
    else:
        s["A"] = fv.Matrix(mesh, diag, upper, fp32_copy=kind == "mixed")
        if kind == "amg":
            s["M"] = fv.AMG(s["A"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "solve":
        return fv.solve(s["A"], s["b"], tol=case["tol"], maxit=20000, method=case["method"],
                        precond=case["precond"])[0]
    if kind == "mixed":
        return fv.solve_mixed_reliable(s["A"], s["b"], tol=case["tol"], update_every=case["update_every"])[0]
    if kind == "momentum":
        return fv.solve_bicgstab_multi(s["A"], s["b"], tol=case["tol"], precond=case["precond"])[0]
    if kind == "transient":
        T = s["T0"].clone()
        fv.transient_run(s["A"], s["k"], s["w"], s["vol"], s["bdiag"], s["bsrc"], s["dt"], case["steps"], T,
                         tol=case["tol"], method=case["method"])
        return T
    if kind == "amg":
        return fv.solve_amg(s["M"], s["b"], tol=case["tol"], method=case["method"])[0]
    if kind == "amg_setup":
        A = fv.Matrix(s["mesh"], s["diag"], s["upper"])
        M = fv.AMG(A)
        x = fv.solve_amg(M, s["b"], tol=case["tol"], method=case["method"])[0]
        M.close()
        A.close()
        return x
    if kind == "piso":
        U, p, phi = s["U0"].clone(), s["p0"].clone(), s["phi0"].clone()
        fv.piso_run(s["ps"], s["dt"], case["steps"], U, p, phi, tol_u=case["tol"], tol_p=case["tol"])
        return {"U": U, "p": p, "phi": phi}
    if kind == "batch":
        return fv.solve_batched(s["B"], s["b"], tol=case["tol"], maxit=20000, method=case["method"])[0]
    diag, upper, b = s["leaves"]
    x = fv.fv_solve(diag, upper, None, b, s["mesh"], tol=case["tol"], method=case["method"])
    loss = 0.5 * (x - s["target"]).square().sum()
    gd, gu, gb = torch.autograd.grad(loss, [diag, upper, b])
    return {"x": x.detach(), "diag": gd, "upper": gu, "b": gb}


# ----------------------------------------------------------------- work

def _counts(nx, ny, nz):
    n = nx * ny * nz
    return n, 3 * n - nx * ny - ny * nz - nx * nz


def work(case):
    """Bytes: the LDU arrays (8 B diagonal; 8 B value and 8 B addressing per
    face), right-hand sides in and results out, once.  Flops: the iterations'
    product (2 per entry) and vector work (about 20 per row), with iteration
    counts of the usual growth: edge^1 for Krylov on a Laplacian (about 8 per
    cell of the longest edge to 1e-10), constant for the others."""
    kind = case["kind"]
    if kind == "batch":
        by = fl = 0.0
        for e in _batch_edges(case):
            n, F = _counts(e, e, e)
            by += 24 * n + 16 * F
            fl += 8 * e * (22 * n + 4 * F)
        return {"bytes": by, "flops": fl}
    n, F = _counts(case["nx"], case["ny"], case["nz"])
    edge = max(case["nx"], case["ny"], case["nz"])
    it = 22 * n + 4 * F
    if kind in ("solve", "mixed"):
        return {"bytes": 24 * n + 16 * F, "flops": 8 * edge * it}
    if kind == "momentum":
        return {"bytes": 8 * n + 24 * F + 16 * n * case["ncomp"], "flops": 60 * case["ncomp"] * 2 * it}
    if kind == "transient":
        return {"bytes": 40 * n + 24 * F, "flops": case["steps"] * 70 * it}
    if kind in ("amg", "amg_setup"):
        return {"bytes": 24 * n + 16 * F, "flops": 45 * 5 * it}
    if kind == "piso":
        return {"bytes": 104 * n + 26 * F, "flops": case["steps"] * (3 * 40 * 2 * it + 2 * (
            45 * 5 if case["pressure"] == "amg" else 10 * edge) * it)}
    return {"bytes": 40 * n + 24 * F, "flops": 2 * 8 * edge * it}


# ----------------------------------------------------------------- FP64 results on the structured grid

def _product(diag, up, lo, x):
    y = diag * x
    for d in range(3):
        _lo(y, d).addcmul_(up[d], _hi(x, d))
        _hi(y, d).addcmul_(lo[d], _lo(x, d))
    return y


def _cg(diag, up, b, x0=None, tol=1e-15, maxit=12000):
    """Jacobi-PCG in FP64 until the recursive residual is at rounding level,
    restarted once from the true residual."""
    x = torch.zeros_like(b) if x0 is None else x0.clone()
    bn = float(b.norm())
    if bn == 0.0:
        return torch.zeros_like(b)
    for tol_now in (tol * 100, tol):
        r = b - _product(diag, up, up, x)
        z = r / diag
        p, gamma = z.clone(), torch.dot(r.view(-1), z.view(-1))
        for it in range(maxit):
            q = _product(diag, up, up, p)
            alpha = gamma / torch.dot(p.view(-1), q.view(-1))
            x.add_(alpha * p)
            r.sub_(alpha * q)
            torch.div(r, diag, out=z)
            new = torch.dot(r.view(-1), z.view(-1))
            if it % 20 == 19 and not float(r.norm()) > tol_now * bn:
                break
            p.mul_(new / gamma).add_(z)
            gamma = new
    return x


def _bicgstab(diag, up, lo, b, x0=None, tol=1e-15, maxit=400):
    """Jacobi-preconditioned BiCGSTAB in FP64, restarted from the true
    residual until it no longer falls."""
    x = torch.zeros_like(b) if x0 is None else x0.clone()
    bn, dot = float(b.norm()), lambda u, v: torch.dot(u.reshape(-1), v.reshape(-1))  # noqa: E731
    for _ in range(3):
        r = b - _product(diag, up, lo, x)
        if float(r.norm()) <= 4 * tol * bn:
            break
        goal = max(tol * bn, 1e-12 * float(r.norm()))
        hat, p, rho = r.clone(), r.clone(), dot(r, r)
        for _ in range(maxit):
            ph = p / diag
            v = _product(diag, up, lo, ph)
            alpha = rho / dot(hat, v)
            r.sub_(alpha * v)
            x.add_(alpha * ph)
            if not float(r.norm()) > goal:
                break
            sh = r / diag
            t = _product(diag, up, lo, sh)
            w = dot(t, r) / dot(t, t)
            x.add_(w * sh)
            r.sub_(w * t)
            if not float(r.norm()) > goal:
                break
            new = dot(hat, r)
            p = r + (new / rho) * (alpha / w) * (p - w * v)
            rho = new
    return x


def _exact_piso(case, seed):
    phi, U, bwall, blid, bgrad, h, nu = _piso(case, seed)
    p, dt, V, D = torch.zeros_like(blid), h, h ** 3, nu * h

    def grad(q):
        g = bgrad * q
        for d in range(3):
            pf = 0.5 * (_lo(q, d) + _hi(q, d))
            _lo(g[d], d).add_(pf)
            _hi(g[d], d).sub_(pf)
        return g / h

    for _ in range(case["steps"]):
        diag, up, lo = _convection(phi, D, bwall + V / dt)
        bH = V / dt * U
        bH[0] += blid
        rhs = bH - V * grad(p)
        U = torch.stack([_bicgstab(diag, up, lo, rhs[k], U[k]) for k in range(3)])
        for _ in range(2):
            H = torch.stack([(bH[k] - (_product(diag, up, lo, U[k]) - diag * U[k])) / diag for k in range(3)])
            rAU = V / diag
            phiH = [h * h * 0.5 * (_lo(H[d], d) + _hi(H[d], d)) for d in range(3)]
            cf = [h * 0.5 * (_lo(rAU, d) + _hi(rAU, d)) for d in range(3)]
            up_p = [-c for c in cf]
            pdiag = _row_sums(up_p, up_p, torch.zeros_like(p))
            for d in range(3):
                up_p[d].view(-1)[0] = 0.0
            prhs = torch.zeros_like(p)
            for d in range(3):
                _lo(prhs, d).sub_(phiH[d])
                _hi(prhs, d).add_(phiH[d])
            prhs.view(-1)[0] = 0.0
            p = _cg(pdiag, up_p, prhs, p)
            phi = [phiH[d] - cf[d] * (_hi(p, d) - _lo(p, d)) for d in range(3)]
            U = H - rAU * grad(p)
    return U, p, phi


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return torch.cat([_cg(d, u, b).reshape(-1) for _, d, u, b in _batch_systems(case, seed)])
    g = Grid(case)
    if kind == "momentum":
        diag, up, lo, b = _momentum(case, seed)
        return torch.stack([g.cells(_bicgstab(diag, up, lo, b[k])) for k in range(case["ncomp"])])
    if kind == "transient":
        k, bdiag, bsrc, dt = _transient(case, seed)
        up = [-t for t in k]
        diag = _row_sums(up, up, bdiag + 1.0 / dt)
        T = torch.zeros_like(bsrc)
        for _ in range(case["steps"]):
            T = _cg(diag, up, T / dt + bsrc, T)
        return g.cells(T)
    if kind == "piso":
        U, p, phi = _exact_piso(case, seed)
        return {"U": g.cells(U), "p": g.cells(p), "phi": g.faces(phi)}
    diag, up, b = _laplacian(case, seed)
    x = _cg(diag, up, b)
    if kind != "autograd":
        return g.cells(x)
    lam = _cg(diag, up, x - _Gen(seed + 7919).uniform(case["nz"], case["ny"], case["nx"]))
    gu = [-(_lo(lam, d) * _hi(x, d) + _hi(lam, d) * _lo(x, d)) for d in range(3)]
    return {"x": g.cells(x), "diag": g.cells(-lam * x), "upper": g.faces(gu), "b": g.cells(lam)}

"""The work that programs have this framework do, as cases that can be timed.

Whole solves (vemg.Solver.solve) of the pressure Poisson equation on thin
tetrahedral boxes with broken columns, from a few thousand unknowns to the
2.2 million of the benchmark, one right-hand side and batches of two to nine,
in FP64 and both mixed precisions, with every top boundary; a product with A
(Solver.matvec), one application of the preconditioner (Solver.apply), and a
serving stream over several resident meshes (vemg.Server).

A program sets a mesh up once and solves many right-hand sides on it, so the
handles are kept by mesh and options; the right-hand sides come from the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_0912_1976_amd as vemg

_AXIS_ORDERS = ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))
_EXACT_NODES = 11000  # meshes whose exact() is a dense factorisation of seconds


def _case(name, kind, nx, ny, nz, eps, nrhs=1, precision="fp64", top_bc="pinned", pc="vl_as", rtol=1e-10,
          shuffled=False):
    return dict(name=name, kind=kind, nx=nx, ny=ny, nz=nz, eps=eps, nrhs=nrhs, precision=precision, top_bc=top_bc,
                pc=pc, rtol=rtol, shuffled=shuffled)


def listed():
    return [
        # the smallest configuration: a test basin, where the latency of every launch counts
        _case("solve 17x17x9", "solve", 17, 17, 9, 1e-2),
        # the smallest serving mesh, three right-hand sides (run as a batch of four), whole top fixed
        _case("solve 25x25x17 mixed dirichlet x3", "solve", 25, 25, 17, 1e-2, 3, "mixed_pc", "dirichlet"),
        # a regional mesh of odd sizes numbered as a mesh generator leaves it, five fields (run as a batch of eight)
        _case("solve 53x41x21 mixed x5 shuffled", "solve", 53, 41, 21, 4e-3, 5, "mixed_pc", shuffled=True),
        # FP32 Krylov space with reliable updates, at the aspect ratio where that form is used
        _case("solve 65x65x17 mixed_ir", "solve", 65, 65, 17, 1e-2, 1, "mixed_ir", rtol=1e-8),
        # free surface (Robin top), a pair of right-hand sides
        _case("solve 113x105x21 robin x2", "solve", 113, 105, 21, 1.6e-3, 2, top_bc="robin"),
        # the multigrid cycle without the additive smoother
        _case("solve 121x113x25 vl_sor", "solve", 121, 113, 25, 1.6e-3, 1, pc="vl_sor", rtol=1e-8),
        # the ordinary configuration: one right-hand side on half a million unknowns
        _case("solve 129x129x33", "solve", 129, 129, 33, 1e-3, 1, rtol=1e-8),
        # a mixed-precision batch on a million unknowns
        _case("solve 177x177x33 mixed x8", "solve", 177, 177, 33, 2.5e-4, 8, "mixed_pc", rtol=1e-8),
        # the benchmark's batch of eight, and a single right-hand side on the same handle
        _case("solve 257x257x33 x8", "solve", 257, 257, 33, 1e-4, 8, rtol=1e-8),
        _case("solve 257x257x33", "solve", 257, 257, 33, 1e-4, 1, rtol=1e-8),
        # a residual check in a time-stepping program: the bare product with A
        _case("matvec 129x129x33", "matvec", 129, 129, 33, 1e-3),
        # requests of 1 to 8 right-hand sides over three resident meshes
        _case("serve 25^2 49^2 129^2", "serve", 129, 129, 33, 6.3e-4, 27, "mixed_pc", rtol=1e-8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        nx, nz = _log_int(rng, 11, 181), _log_int(rng, 6, 41)
        ny = max(9, int(nx * rng.uniform(0.6, 1.0)))
        # a coarsest level near its limit of 8192 unknowns takes a minute of host time to invert at setup: the
        # two largest listed meshes stand for it
        dense = max(_coarsest(nx * ny, (10.6, 10.6)), _coarsest(nx * ny * (nz - 1), (23.5, 18.3)))
        if 1500 <= nx * ny * nz <= 1050000 and dense <= 4500:
            break
    kind = rng.choice(("solve",) * 8 + ("matvec", "precond"))
    eps = float("%.2g" % 10 ** rng.uniform(-3.6, -2))
    precision = rng.choice(("fp64", "fp64", "mixed_pc"))
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, eps=eps, nrhs=rng.choice((1, 1, 2, 3, 4, 5, 8, 9)) if kind == "solve" else 1,
                precision=precision if kind == "solve" else "fp64",
                top_bc=rng.choice(("pinned", "pinned", "dirichlet", "robin")),
                pc=rng.choice(("vl_as", "vl_as", "vl_as", "vl_sor")), rtol=1e-10, shuffled=rng.random() < 0.5)


# ------------------------------------------------------------------ meshes
class _Grid:
    """Thin box [0,1]^2 x [-eps (1 + 0.3 sin sin), 0] on an nx x ny x nz vertex
    grid, six tetrahedra a cell, every interior vertex of every layer moved by
    up to 0.3 grid spacings, so that the columns are broken."""

    def __init__(self, nx, ny, nz, eps, shuffled):
        self.shape = (nz, ny, nx)
        self.tet_corners = []
        for order in _AXIS_ORDERS:
            at, path = [0, 0, 0], [(0, 0, 0)]
            for axis in order:
                at[axis] = 1
                path.append(tuple(at))
            if sum(order[p] > order[q] for p in range(3) for q in range(p + 1, 3)) % 2:
                path[2], path[3] = path[3], path[2]
            self.tet_corners.append(path)
        k, j, i = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
        rng = np.random.default_rng(nx * 1000003 + ny * 1009 + nz)
        free = (i > 0) & (i < nx - 1) & (j > 0) & (j < ny - 1)
        move = [np.where(free, rng.uniform(-0.3, 0.3, self.shape) / (m - 1), 0.0) for m in (nx, ny)]

        def place(scale):
            x, y = i / (nx - 1) + scale * move[0], j / (ny - 1) + scale * move[1]
            floor = eps * (1.0 + 0.3 * np.sin(2 * np.pi * x) * np.sin(2 * np.pi * y))
            return x, y, -floor * (nz - 1 - k) / (nz - 1)

        scale = np.ones(self.shape)
        whole = [self._volume(place(np.zeros(self.shape)), c) for c in self.tet_corners]
        while True:  # the displacement of a flattened tetrahedron's vertices is halved
            self.xyz = place(scale)
            flat = np.zeros(self.shape, bool)
            for c, v in zip(self.tet_corners, whole):
                bad = self._volume(self.xyz, c) <= 0.05 * v
                for a in c:
                    flat[self._at(a)] |= bad
            if not flat.any():
                break
            scale[flat] *= 0.5
        n = nx * ny * nz
        # number[v]: the caller's number of grid vertex v
        self.number = np.random.default_rng(n).permutation(n) if shuffled else np.arange(n)
        ids = self.number.reshape(self.shape)
        self.tets = np.stack([np.stack([ids[self._at(a)] for a in c], -1).reshape(-1, 4) for c in self.tet_corners],
                             1).reshape(-1, 4)
        self.points, self.top = np.empty((n, 3)), np.zeros(n, bool)
        self.points[self.number] = np.stack(self.xyz, -1).reshape(-1, 3)
        self.top[ids[-1].ravel()] = True
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")

    def _at(self, a):
        return tuple(slice(a[d], a[d] + self.shape[2 - d] - 1) for d in (2, 1, 0))

    def _volume(self, xyz, corners):
        p = [np.stack([c[self._at(a)] for c in xyz]) for a in corners]
        a, b, c = (p[t] - p[0] for t in (1, 2, 3))
        return (a[0] * (b[1] * c[2] - b[2] * c[1]) - a[1] * (b[0] * c[2] - b[2] * c[0])
                + a[2] * (b[0] * c[1] - b[1] * c[0])) / 6.0

    @functools.cached_property
    def coords(self):
        return torch.as_tensor(np.stack(self.xyz), device=self.dev)

    @functools.cached_property
    def natural(self):
        return torch.as_tensor(self.number, device=self.dev)

    def volumes(self):
        return [torch.as_tensor(self._volume(self.xyz, c), device=self.dev) for c in self.tet_corners]

    def gradients(self):
        """Per tetrahedron of a cell: its corners, volumes and the gradients of its four hat functions."""
        for c, v in zip(self.tet_corners, self.volumes()):
            p = [self.coords[(slice(None),) + self._at(a)] for a in c]
            a, b, d = (p[t] - p[0] for t in (1, 2, 3))
            g = [torch.linalg.cross(s, t, dim=0) / (6.0 * v) for s, t in ((b, d), (d, a), (a, b))]
            yield c, v, [-(g[0] + g[1] + g[2]), *g]

    def mass(self, f):
        """M f of a nodal field on the grid, consistent P1 mass matrix."""
        out = torch.zeros_like(f)
        for c, v in zip(self.tet_corners, self.volumes()):
            total = sum(f[self._at(a)] for a in c)
            for a in c:
                out[self._at(a)] += v / 20.0 * (total + f[self._at(a)])
        return out

    def stiffness(self, x):
        """A x on the grid, element by element from the differences of a tetrahedron's values."""
        out = torch.zeros_like(x)
        for c, v, g in self.gradients():
            slope = sum(g[t] * (x[self._at(c[t])] - x[self._at(c[0])]) for t in (1, 2, 3))
            for t in range(4):
                out[self._at(c[t])] += v * (g[t] * slope).sum(0)
        return out

    def field(self, rng, eps):
        """A smooth random field: sixteen cosine modes."""
        x, y, z = self.coords
        f = float(rng.standard_normal()) * torch.cos(math.pi / eps * z)
        for k in range(4):
            for m in range(4):
                if k + m:
                    f = f + float(rng.standard_normal()) * torch.cos(k * math.pi * x) * torch.cos(m * math.pi * y)
        return f

    def to_natural(self, f):
        out = torch.empty(f.numel(), dtype=f.dtype, device=f.device)
        out[self.natural] = f.reshape(-1)
        return out


@functools.lru_cache(maxsize=12)
def _grid(nx, ny, nz, eps, shuffled):
    return _Grid(nx, ny, nz, eps, shuffled)


def _alpha(case):
    return 0.03 / case["eps"] if case["top_bc"] == "robin" else 0.0


@functools.lru_cache(maxsize=12)
def _solver(nx, ny, nz, eps, shuffled, precision, top_bc, pc, alpha):
    g = _grid(nx, ny, nz, eps, shuffled)
    return vemg.Solver(g.points, g.tets, g.top, top_bc=top_bc, pc=pc, precision=precision, robin_alpha=alpha, device=0)


@functools.lru_cache(maxsize=2)
def _server(precision, pc, top_bc):
    server, grids = vemg.Server(device=0, precision=precision, pc=pc, top_bc=top_bc), []
    for nx, nz, eps in ((25, 17, 1e-2), (49, 21, 4e-3), (129, 33, 6.3e-4)):
        g = _grid(nx, nx, nz, eps, False)
        grids.append((server.add_mesh(g.points, g.tets, g.top), g, eps))
    return server, grids


def _right_hand_sides(g, eps, top_bc, rng, count):
    out = []
    one = g.mass(torch.ones(g.shape, dtype=torch.float64, device=g.dev))
    for _ in range(count):
        b = g.mass(g.field(rng, eps))
        if top_bc == "pinned":  # the Neumann problem's right-hand side has no constant part
            b = b - one * (b.sum() / one.sum())
        out.append(g.to_natural(b))
    return torch.stack(out)


def _mesh(case):
    return _grid(case["nx"], case["ny"], case["nz"], case["eps"], case["shuffled"])


def _input(case, seed):
    rng, g = np.random.default_rng(seed), _mesh(case)
    if case["kind"] == "solve":
        return _right_hand_sides(g, case["eps"], case["top_bc"], rng, case["nrhs"])
    # a product's input: a smooth field and a tenth of noise, as an iterate has; zero at fixed nodes
    f = g.field(rng, case["eps"]) + 0.1 * torch.as_tensor(rng.standard_normal(g.shape), device=g.dev)
    if case["top_bc"] == "dirichlet":
        f[-1] = 0.0
    if case["top_bc"] == "pinned":
        f[-1, 0, 0] = 0.0
    return g.to_natural(f)


def prepare(case, seed):
    if case["kind"] == "serve":
        server, grids = _server(case["precision"], case["pc"], case["top_bc"])
        rng, requests = np.random.default_rng(seed), []
        for count in (1, 4, 8, 2, 5, 7):  # right-hand sides of the requests, 27 in all, mesh after mesh
            mesh, g, eps = grids[len(requests) % len(grids)]
            requests.append((mesh, _right_hand_sides(g, eps, case["top_bc"], rng, count)))
        return case, server, requests
    s = _solver(case["nx"], case["ny"], case["nz"], case["eps"], case["shuffled"], case["precision"], case["top_bc"],
                case["pc"], _alpha(case))
    x = _input(case, seed)
    if case["kind"] == "precond":  # the preconditioner takes a residual, in the library's order
        x = _right_hand_sides(_mesh(case), case["eps"], case["top_bc"], np.random.default_rng(seed), 1)[0]
        x = x[torch.as_tensor(s.export("perm", np.int64), device=x.device)]
    return case, s, x


def run(state):
    case, handle, data = state
    if case["kind"] == "serve":
        ids = [handle.submit(mesh, b, rtol=case["rtol"]) for mesh, b in data]
        for rid in ids:
            handle.wait(rid)
        return [handle.result(rid)[0] for rid in ids]
    if case["kind"] == "matvec":
        return handle.matvec(data)
    if case["kind"] == "precond":
        return handle.apply(vemg.OP_PRECOND, data, data.numel())
    return handle.solve(data, rtol=case["rtol"], max_iter=5000)[0]


def exact(case, seed):
    if case["kind"] in ("serve", "precond"):
        return None
    g = _mesh(case)
    n = g.points.shape[0]
    fixed = torch.zeros(g.shape, dtype=torch.bool, device=g.dev)
    if case["top_bc"] == "dirichlet":
        fixed[-1] = True
    elif case["top_bc"] == "pinned":
        fixed[-1, 0, 0] = True
    if case["kind"] == "matvec":
        x = _input(case, seed)[g.natural].reshape(g.shape)
        y = g.stiffness(x) + _alpha(case) * _top_mass(g, x)
        return g.to_natural(torch.where(fixed, torch.zeros_like(y), y))
    if n > _EXACT_NODES:
        return None
    ids = np.arange(n).reshape(g.shape)
    a = torch.zeros(n * n, dtype=torch.float64)
    for c, v, grad in g.gradients():  # on the CPU, where the sums have one order
        at = [torch.as_tensor(ids[g._at(t)].ravel()) for t in c]
        for s in range(4):
            for t in range(4):
                a.index_add_(0, at[s] * n + at[t], (v * (grad[s] * grad[t]).sum(0)).reshape(-1).cpu())
    a = a.reshape(n, n).to(g.dev)
    if case["top_bc"] == "robin":
        unit = torch.zeros(g.shape, dtype=torch.float64, device=g.dev)
        for v in ids[-1].ravel():
            unit.reshape(-1)[v] = 1.0
            a[v] += _alpha(case) * _top_mass(g, unit).reshape(-1)
            unit.reshape(-1)[v] = 0.0
    free = torch.nonzero(~fixed.reshape(-1)).reshape(-1)
    a = a[free][:, free]
    b = _input(case, seed)[:, g.natural][:, free].T
    factor = torch.linalg.cholesky(a)
    y = torch.cholesky_solve(b, factor)
    y = y + torch.cholesky_solve(b - a @ y, factor)
    out = torch.zeros((case["nrhs"], n), dtype=torch.float64, device=g.dev)
    out[:, g.natural[free]] = y.T
    return out


def _top_mass(g, x):
    """The Robin term's P1 mass matrix of the top triangles, projected onto (x, y), times x."""
    out = torch.zeros_like(x)
    for c in g.tet_corners:
        on = [a for a in c if a[2] == 1]
        if len(on) != 3:
            continue
        # the top face of the cells of the last layer
        sl = [tuple([slice(-1, None), *g._at(a)[1:]]) for a in on]
        p = [g.coords[(slice(None),) + s] for s in sl]
        area = 0.5 * ((p[1][0] - p[0][0]) * (p[2][1] - p[0][1]) - (p[1][1] - p[0][1]) * (p[2][0] - p[0][0])).abs()
        total = sum(x[s] for s in sl)
        for s in sl:
            out[s] += area / 12.0 * (total + x[s])
    return out


# ------------------------------------------------------------------ work
def _rows(case):
    top = case["nx"] * case["ny"]
    return top, top * (case["nz"] - 1)


def _coarsest(rows, ratios):
    for q in ratios:
        if rows <= 8192:
            break
        rows = rows / q
    return rows


def work(case):
    """A product reads A (13.7 off-diagonals a row: value and column) and its
    input and writes its output once.  An iteration of the solver is a product,
    a forward and a backward sweep and a residual (in all three times A), a
    dozen vectors, and the dense inverses of the two coarsest levels."""
    if case["kind"] == "serve":
        parts = [work(dict(case, kind="solve", nx=nx, ny=nx, nz=nz, nrhs=k))
                 for nx, nz, k in ((25, 17, 3), (49, 21, 9), (129, 33, 15))]
        return {q: sum(p[q] for p in parts) for q in ("bytes", "flops")}
    top, bar = _rows(case)
    n, k = top + bar, case["nrhs"]
    entries = 13.7 * n
    if case["kind"] == "matvec":
        return {"bytes": 12 * entries + 24 * n, "flops": 3 * entries}
    word = 8 if case["precision"] == "fp64" else 4
    dense = 0 if case["top_bc"] == "dirichlet" else _coarsest(top, (10.6, 10.6)) ** 2
    if case["pc"] == "vl_as":
        dense += _coarsest(bar, (23.5, 18.3)) ** 2
    precond = {"bytes": 2 * entries * (4 + word) + 8 * dense + 6 * n * k * word, "flops": (6 * entries + 2 * dense) * k}
    if case["kind"] == "precond":
        return precond
    # iterations to the tolerance, as measured on the listed meshes
    its = max(12.0, 8.2 * (math.log2(n) - 11.3) + 31.0) * math.log10(case["rtol"]) / -8.0
    its *= 1.4 if case["pc"] == "vl_sor" else 1.0
    batches = -(-k // 8)
    return {"bytes": its * (batches * (12 * entries + precond["bytes"]) + 6 * 8 * n * k),
            "flops": its * (3 * entries * k + precond["flops"])}

"""Small meshes of many sweep colours: every pair of the nodes below the top is
joined by an edge, so each has a colour of its own and a sweep takes as many
launches as there are unknowns."""
from collections import defaultdict

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0912_1976_amd as lib  # noqa: E402  (a missing package fails, never skips)

from oracle import precond, solver as osolver  # noqa: E402


class _Mesh:
    pass


def neighbourly_mesh(q):
    """q points of the moment curve (t, t^2, t^3), whose tetrahedra (i, i+1, j,
    j+1) join every pair, under one large triangle, the top, placed corner by
    corner: each is joined to the boundary faces it sees."""
    t = np.linspace(-1, 1, q)
    p = np.stack([t, t**2, t**3], 1)
    tets = [(i, i + 1, j, j + 1) for i in range(q - 1) for j in range(i + 2, q - 1)]
    for a in ((-60.0, -50.0, 40.0), (60.0, -50.0, 40.0), (0.0, 80.0, 40.0)):
        faces = defaultdict(list)  # its opposite corners
        for T in tets:
            for o in range(4):
                faces[tuple(sorted(T[:o] + T[o + 1:]))].append(T[o])
        for F, opposite in faces.items():
            A, B, C = p[list(F)]
            normal = np.cross(B - A, C - A)
            if len(opposite) == 1 and (normal @ (p[opposite[0]] - A)) * (normal @ (np.array(a) - A)) < 0:
                tets.append(F + (len(p),))
        p = np.vstack([p, a])
    tets = np.array(tets)
    e = p[tets]
    neg = np.einsum("ij,ij->i", np.cross(e[:, 1] - e[:, 0], e[:, 2] - e[:, 0]), e[:, 3] - e[:, 0]) < 0
    tets[neg] = tets[neg][:, [1, 0, 2, 3]]
    m = _Mesh()
    m.xyz, m.tets, m.n = p, tets, len(p)
    m.top = np.arange(m.n) >= q
    return m


@pytest.mark.parametrize("q", [20, 80])
def test_many_colours(q):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case colours", q, flush=True)
    m = neighbourly_mesh(q)
    s = lib.Solver(m.xyz, m.tets, m.top, top_bc="R", robin_alpha=1.0, device=0, coarse_max=16)
    o = osolver.setup(m, "R", coarse_max=16, alpha=1.0)
    colour = s.export("colour", np.int32)
    assert len(np.unique(colour[o.n_top:])) == q and len(o.Abar_levels) > 1
    if q == 80:  # a backward sweep's launches, a slice of each colour, against the rows of a dot of 256 rows a block
        assert q + len(np.unique(colour[:o.n_top])) > (-(-o.n // 256) + 8) * 8
    r = np.random.default_rng(3).standard_normal(o.n)
    # the matrices are the oracle's bit for bit; its rounding moves the result by less than the coarsest solve's
    tol = max(1e-12, 50 * np.finfo(float).eps * np.linalg.cond(o.Abar_levels[-1].A.toarray()))
    for pc in ("vl_as", "vl_sor", "vl_add"):
        s.set_preconditioner(pc)
        ref = precond.make(o, pc)(r)
        err = np.linalg.norm(s.apply(lib.OP_PRECOND, r, o.n).cpu().numpy() - ref) / np.linalg.norm(ref)
        print(pc, "rel", err, "tol", tol, flush=True)
        assert err < tol
    s.set_preconditioner("vl_as")
    B = np.random.default_rng(4).standard_normal((8, m.n))
    xb, its, rel, st = s.solve(B, rtol=1e-8)
    assert st == 0 and max(rel) <= 1e-8
    for k in (0, 7):
        x, i1, _, _ = s.solve(B[k], rtol=1e-8)
        assert i1[0] == its[k] and torch.equal(x, xb[k])

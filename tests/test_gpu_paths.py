"""The size-dependent paths of the solve at the sizes where they change: dense
coarsest solves around one chunk, coarse sweeps whose halo exceeds what is
staged, the scalar steps around the sizes that fold, compact or move them, the
lengths of a chunk of iterations, and batches padded to a wider one."""
import ctypes as C

import numpy as np
import pytest
import scipy.sparse as sp

from inputs import box_mesh, fourier_field

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0912_1976_amd as lib  # noqa: E402  (a missing package fails, never skips)

from oracle import amg, precond, solver as osolver  # noqa: E402


class _Mesh:
    def __init__(self, xyz, tets, top):
        self.xyz, self.tets, self.top, self.n = xyz, tets, top, len(xyz)


def _hub(nx, ny, nz):
    """A thin box with one more node below it, joined to every node of its
    bottom: the hub's aggregate is coupled to nearly all the others, so coarse
    rows and patch halos have thousands of entries and the patches of a sweep
    form one long chain."""
    H = 0.05
    m = box_mesh(nx, ny, nz, H, jitter=0.2, seed=5)
    f = np.sort(np.concatenate([m.tets[:, c] for c in ([0, 1, 2], [0, 1, 3], [0, 2, 3], [1, 2, 3])]), axis=1)
    f = np.unique(f[(m.xyz[f, 2] < -H * (1 - 1e-9)).all(axis=1)], axis=0)
    assert len(f) == 2 * (nx - 1) * (ny - 1)
    a = m.xyz[f]
    flip = np.cross(a[:, 1] - a[:, 0], a[:, 2] - a[:, 0])[:, 2] < 0
    f[flip] = f[flip][:, [0, 2, 1]]
    tets = np.concatenate([m.tets, np.column_stack([np.full(len(f), m.n), f])])
    return _Mesh(np.concatenate([m.xyz, [[0.5, 0.5, -H - 1.0]]]), tets,
                 np.concatenate([m.top, [0]]).astype(m.top.dtype))


def _solver(m, mode="R", **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case paths", m.n, mode, kw, flush=True)
    return lib.Solver(m.xyz, m.tets, m.top, top_bc=mode, device=0, robin_alpha=20.0 if mode == "R" else 0.0, **kw)


def _check_cycles(s, o):
    rng = np.random.default_rng(11)
    for op, ref, n, levels in (
            (lib.OP_VCYCLE_S, lambda g: amg.vcycle(o.S_levels, g), o.n_top, (o.S_levels,)),
            (lib.OP_VCYCLE_ABAR, lambda g: amg.vcycle(o.Abar_levels, g), o.n - o.n_top, (o.Abar_levels,)),
            (lib.OP_PRECOND, precond.make(o, "vl_as"), o.n, (o.S_levels, o.Abar_levels))):
        g = rng.standard_normal(n)
        x, want = s.apply(op, g, n).cpu().numpy(), ref(g)
        # coarse operators summed in another order, amplified by the coarsest solve
        tol = max(1e-12, 50 * np.finfo(float).eps * max(np.linalg.cond(L[-1].A.toarray()) for L in levels))
        err = np.linalg.norm(x - want) / np.linalg.norm(want)
        print("op", op, "rel", err, "tol", tol, flush=True)
        assert err < tol


# surface operators of 512 (one chunk exactly), 513 and 1025 unknowns
@pytest.mark.parametrize("nx,ny,mode", [(27, 19, "N"), (27, 19, "R"), (41, 25, "R")])
def test_dense_coarsest_solves_around_a_chunk(nx, ny, mode):
    m = box_mesh(nx, ny, 3, 0.02, jitter=0.2, seed=8)
    s = _solver(m, mode)
    assert s.info()["s_rows"] == [nx * ny - (mode == "N")]
    _check_cycles(s, osolver.setup(m, mode, alpha=20.0 if mode == "R" else 0.0))


@pytest.mark.parametrize("nx,ny,nz", [(41, 41, 2), (61, 59, 3)])
def test_sweeps_with_halos_beyond_the_staged_rows(nx, ny, nz):
    m = _hub(nx, ny, nz)
    s = _solver(m, "N", coarse_max=16)
    ptr, idx = s.export("S.0.A.ptr", np.int64), s.export("S.0.A.idx", np.int32)
    pr = s.export("S.0.patch_row", np.int64)
    halo = 0
    for a, b in zip(pr[:-1], pr[1:]):
        c = np.unique(idx[ptr[a]:ptr[b]])
        halo = max(halo, int(((c < a) | (c >= b)).sum()))
    assert halo > 1024
    _check_cycles(s, osolver.setup(m, "N", coarse_max=16))


@pytest.mark.parametrize("precision", ["fp64", "mixed_pc"])
def test_batches_with_halos_beyond_the_staged_rows(precision):
    m = _hub(41, 41, 2)
    s = _solver(m, "N", coarse_max=16, precision=precision)
    B = np.stack([s.rhs(fourier_field(m.xyz, 0.05, 700 + k)) for k in range(8)])
    x, its, rel, st = s.solve(B, rtol=1e-9)
    assert st == 0 and max(rel) <= 1e-9
    for k in (0, 7):
        xk, ik, _, _ = s.solve(B[k], rtol=1e-9)
        assert ik[0] == its[k] and torch.equal(xk, x[k])


# 65536 | 65559 unknowns: where r.z is summed; 250000 | 250047: where the
# convergence test is; 262144 | 266240: whether eight columns fold their scalars
@pytest.mark.parametrize("nx,ny,nz", [(64, 32, 32), (41, 41, 39), (100, 50, 50), (63, 63, 63), (64, 64, 64),
                                      (65, 64, 64)])
def test_scalar_steps_do_not_depend_on_the_batch_width(nx, ny, nz):
    m = box_mesh(nx, ny, nz, 0.05, jitter=0.2, seed=4)
    s = _solver(m)
    B = np.stack([s.rhs(fourier_field(m.xyz, 0.05, 800 + k)) for k in range(8)])
    perm = s.export("perm", np.int64)
    absA = sp.csr_matrix((np.abs(s.export("Aoff.val", np.float64)), s.export("Aoff.idx", np.int32),
                          s.export("Aoff.ptr", np.int64))) + sp.diags(s.export("diag", np.float64))
    for precision in ("fp64", "mixed_pc"):
        s.set_precision(precision)
        x, its, rel, st = s.solve(B, rtol=1e-8)
        assert st == 0 and max(rel) <= 1e-8
        # A x against b (Robin: every node is an unknown); a row of some 15 products rounds within 32 ulps of |A| |x|
        bk, xa = B[5], x[5].abs().cpu().numpy()
        r = np.linalg.norm(bk - s.matvec(x[5]).cpu().numpy())
        assert r <= 1e-8 * np.linalg.norm(bk) + 32 * np.finfo(float).eps * np.linalg.norm(absA @ xa[perm]), precision
        for k in (0, 5):
            xk, ik, _, _ = s.solve(B[k], rtol=1e-8)
            assert ik[0] == its[k] and torch.equal(xk, x[k]), (precision, k)
        x4, i4, _, _ = s.solve(B[4:], rtol=1e-8)
        assert i4 == its[4:] and torch.equal(x4, x[4:]), precision


@pytest.mark.parametrize("precision", ["fp64", "mixed_pc"])
def test_solves_do_not_depend_on_the_chunk_length(precision):
    m = box_mesh(21, 13, 6, 1e-2, jitter=0.3, seed=2, bathymetry=True)
    ref = None
    for poll in (8, 1, 2, 5, 12, 16, 17, 40):
        s = _solver(m, "N", poll_every=poll, precision=precision, coarse_max=64)
        if ref is None:
            B = np.stack([s.rhs(fourier_field(m.xyz, 1e-2, 900 + k)) * 10.0 ** (3 * k) for k in range(3)])
            # a zero column and an iteration cap inside a chunk
            B[1] = 0.0
        out = [s.solve(B, rtol=1e-9), s.solve(B, rtol=1e-9, max_iter=7)]
        if ref is None:
            ref = out
        for (x, its, _, st), (xr, ir, _, sr) in zip(out, ref):
            assert st == sr and its == ir and torch.equal(x, xr), poll


@pytest.mark.parametrize("nrhs", [1, 3, 5, 9])
def test_batches_are_moved_whole_and_fixed_nodes_stay_out(nrhs):
    m = box_mesh(13, 11, 5, 1e-2, jitter=0.2, seed=6)
    s = _solver(m, "D", coarse_max=64)
    top = np.asarray(m.top, dtype=bool)
    B = np.stack([s.rhs(fourier_field(m.xyz, 1e-2, 950 + k)) for k in range(nrhs)])
    single = [s.solve(b, rtol=1e-9) for b in B]
    B[:, top] = np.nan  # ignored
    x, its, _, st = s.solve(B, rtol=1e-9)
    assert st == 0 and x[:, torch.as_tensor(top, device=x.device)].abs().max().item() == 0.0
    for k in range(nrhs):
        assert its[k] == single[k][1][0] and torch.equal(x[k], single[k][0]), k


@pytest.mark.parametrize("precision", ["fp64", "mixed_pc"])
def test_a_column_of_nan_or_infinity_stays_alone(precision):
    m = _hub(41, 41, 2)
    s = _solver(m, "N", coarse_max=16, precision=precision)
    B = np.stack([s.rhs(fourier_field(m.xyz, 0.05, 980 + k)) for k in range(4)])
    single = [s.solve(b, rtol=1e-9) for b in B]
    B[1, 700], B[2] = np.nan, np.inf
    b = torch.as_tensor(B, device="cuda")
    x, its, rel = torch.empty_like(b), (C.c_int * 4)(), (C.c_double * 4)()
    st = s._lib.vemg_solve(s._h, 4, C.c_void_p(b.data_ptr()), C.c_void_p(x.data_ptr()), 1e-9, 1000, its, rel)
    assert st == -6
    for k in (0, 3):
        assert its[k] == single[k][1][0] and torch.equal(x[k], single[k][0]), k


@pytest.mark.parametrize("precision", ["fp64", "mixed_pc", "mixed_ir"])
@pytest.mark.parametrize("poll", [8, 5, 40])
def test_only_the_first_solve_captures(precision, poll):
    # the lengths of the chunks follow the residuals, so each tolerance takes others
    m = box_mesh(21, 13, 6, 1e-2, jitter=0.3, seed=2, bathymetry=True)
    s = _solver(m, "N", poll_every=poll, precision=precision, coarse_max=64)
    b = s.rhs(fourier_field(m.xyz, 1e-2, 970))
    s.solve(b, rtol=0.5)
    first = s.export("graphs", np.int64)[0]
    assert first > 0
    for rtol in 10.0 ** -np.arange(1, 11):
        s.solve(b, rtol=rtol)
        assert s.export("graphs", np.int64)[0] == first, rtol
    s.solve(np.stack([b, b]), rtol=1e-6)
    assert s.export("graphs", np.int64)[0] > first  # another width


@pytest.mark.parametrize("pc", ["vl_as", "vl_add", "sa"])
@pytest.mark.parametrize("coarse_max", [64, 8192])  # 8192: A_bar is one dense level
def test_calls_of_every_precision_share_vectors_and_keep_apart(pc, coarse_max):
    # the precisions' vectors overlap in memory; whatever ran before, in any
    # precision, width or operator, a call gives what a fresh handle does
    m = box_mesh(21, 13, 6, 1e-2, jitter=0.3, seed=2, bathymetry=True)
    kw = dict(coarse_max=coarse_max, pc=pc)
    s = _solver(m, "N", **kw)
    n, nt = s.info()["n"], s.info()["n_top"]
    B = np.stack([s.rhs(fourier_field(m.xyz, 1e-2, 990 + k)) for k in range(8)])
    r = np.random.default_rng(6).standard_normal(n)
    xn = np.random.default_rng(7).standard_normal(m.n)

    def calls(h):
        return {"solve 1": lambda: h.solve(B[0], rtol=1e-9)[0], "solve 8": lambda: h.solve(B, rtol=1e-9)[0],
                "solve 2": lambda: h.solve(B[:2], rtol=1e-9)[0], "matvec": lambda: h.matvec(xn),
                "precond": lambda: h.apply(lib.OP_PRECOND, r, n),
                "vcycle": lambda: h.apply(lib.OP_VCYCLE_ABAR, r[nt:], n - nt),
                "time": lambda: torch.tensor(h.time_op(lib.OP_A, nrhs=8, reps=1)[1])}

    want = {}
    for precision in ("fp64", "mixed_pc", "mixed_ir"):
        for name in calls(s):
            f = _solver(m, "N", precision=precision, **kw)
            want[precision, name] = calls(f)[name]()
            f.close()
    order = [(p, c) for p in ("fp64", "mixed_pc", "mixed_ir") for c in calls(s)]
    for k in range(3):
        for i in np.random.default_rng(20 + k).permutation(len(order)):
            precision, name = order[i]
            s.set_precision(precision)
            assert torch.equal(calls(s)[name](), want[precision, name]), (precision, name)


# where the sweeps form r.z again
@pytest.mark.parametrize("nx,ny,nz", [(101, 99, 100), (100, 100, 100)])
def test_sums_of_a_million_rows_do_not_depend_on_the_batch_width(nx, ny, nz):
    test_scalar_steps_do_not_depend_on_the_batch_width(nx, ny, nz)

"""The merged fine sweeps of the VL + additive smoother preconditioner (one
pair of sweeps for the SOR cycle and the smoother) against the oracle's two
separate cycles, where the extended rows are everything, a few rows or none:
one layer of cells (every row below the top is extended), few layers, odd
sizes, and the whole top fixed (no extended row); and every batch width
against the single column."""
import numpy as np
import pytest

from inputs import box_mesh, fourier_field

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_0912_1976_amd as lib  # noqa: E402  (a missing package fails, never skips)

from oracle import precond, solver as osolver  # noqa: E402


def _build(nx, ny, nz, mode, precision="fp64"):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case merged", nx, ny, nz, mode, precision, flush=True)
    m = box_mesh(nx, ny, nz, 1e-2, jitter=0.3, seed=nx + nz, bathymetry=True)
    alpha = 20.0 if mode == "R" else 0.0
    s = lib.Solver(m.xyz, m.tets, m.top, top_bc=mode, device=0, coarse_max=16, robin_alpha=alpha, precision=precision)
    return m, s, osolver.setup(m, mode, coarse_max=16, alpha=alpha)


@pytest.mark.parametrize("nx,ny,nz,mode", [(9, 7, 2, "N"), (21, 5, 3, "R"), (12, 11, 4, "N"), (19, 14, 8, "N"),
                                           (17, 13, 7, "D")])
def test_merged_cycles_match_the_two_cycles(nx, ny, nz, mode):
    m, s, o = _build(nx, ny, nz, mode)
    assert len(o.Abar_levels) > 1  # a single dense level takes the separate form
    r = np.random.default_rng(3).standard_normal(o.n)
    z = s.apply(lib.OP_PRECOND, r, o.n).cpu().numpy()
    ref = precond.make(o, "vl_as")(r)
    # the coarse operators are summed in another order than the oracle's, which
    # the exact coarsest solves amplify by their condition numbers
    c = max(np.linalg.cond(L[-1].A.toarray()) for L in (o.S_levels, o.Abar_levels) if L)
    tol = max(1e-12, 50 * np.finfo(float).eps * c)
    err = np.linalg.norm(z - ref) / np.linalg.norm(ref)
    print("rel", err, "tol", tol, flush=True)
    assert err < tol


@pytest.mark.parametrize("precision", ["fp64", "mixed_pc"])
def test_merged_cycles_do_not_depend_on_the_batch_width(precision):
    m, s, o = _build(21, 13, 6, "N", precision)
    B = np.stack([s.rhs(fourier_field(m.xyz, 1e-2, 600 + k)) for k in range(8)])
    single = [s.solve(b, rtol=1e-9) for b in B]
    for K in (2, 4, 8):
        x, its, _, st = s.solve(B[:K], rtol=1e-9)
        assert st == 0
        for k in range(K):
            assert its[k] == single[k][1][0] and torch.equal(x[k], single[k][0]), (K, k)


@pytest.mark.parametrize("nx,ny,nz,mode", [(9, 7, 2, "N"), (21, 5, 3, "R"), (19, 14, 8, "N"), (17, 13, 7, "D")])
@pytest.mark.parametrize("precision", ["fp64", "mixed_pc"])
def test_the_merged_cycles_are_the_sum_of_the_separate_ones(nx, ny, nz, mode, precision):
    # the SOR cycle and the smoother's each with fine sweeps of its own, as the
    # other preconditioners run them
    m, s, o = _build(nx, ny, nz, mode, precision)
    r = np.random.default_rng(5).standard_normal(o.n)
    z = s.apply(lib.OP_PRECOND, r, o.n).cpu().numpy()
    s.set_preconditioner("vl_sor")
    ref = s.apply(lib.OP_PRECOND, r, o.n).cpu().numpy()
    ref[o.n_top:] += s.apply(lib.OP_VCYCLE_ABAR, r[o.n_top:], o.n - o.n_top).cpu().numpy()
    # the same terms summed in another order: some 15 a row, through the colours of two sweeps
    eps = np.finfo(np.float64 if precision == "fp64" else np.float32).eps
    colours = len(np.unique(s.export("colour", np.int32)))
    err, tol = np.linalg.norm(z - ref) / np.linalg.norm(ref), 2 * 15 * colours * eps
    print("separate", err, "tol", tol, flush=True)
    assert err < tol
    if precision != "fp64":  # FP32 operators against the oracle's
        want = precond.make(o, "vl_as")(r)
        err = np.linalg.norm(z - want) / np.linalg.norm(want)
        print("oracle", err, flush=True)
        assert err < 1e-4


@pytest.mark.parametrize("mode", ["N", "D"])
@pytest.mark.parametrize("precision", ["fp64", "mixed_ir"])
def test_the_merged_steps_are_timed(mode, precision):
    m, s, o = _build(17, 13, 7, mode, precision)
    colours = max(s.info()["fine_colours_top"], s.info()["fine_colours_bar"])
    b = s.rhs(fourier_field(m.xyz, 1e-2, 650))
    x = s.solve(b, rtol=1e-8)[0]
    for K in (1, 8):
        for op, launches in ((lib.OP_MERGED_FWD, colours), (lib.OP_MERGED_RES, 1), (lib.OP_MERGED_PROLONG, 1),
                             (lib.OP_MERGED_BWD, colours)):
            ms, nl = s.time_op(op, reps=3, nrhs=K)
            assert ms > 0 and nl == launches
    assert torch.equal(s.solve(b, rtol=1e-8)[0], x)
    f = lib.Solver(m.xyz, m.tets, m.top, top_bc=mode, device=0)  # A_bar is one dense level
    assert f.info()["abar_levels"] == 1
    with pytest.raises(lib.VemgError) as e:
        f.time_op(lib.OP_MERGED_BWD)
    assert e.value.status == -7

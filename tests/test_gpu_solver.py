"""GPU parity of gmresdr_solve (GMRES-DR + GMRES-Proj, Sec. 7) against the oracle.

Solutions are compared with dense LU (|x - x_LU| / |x_LU| <= 1e-10 in
FP64), converged harmonic Ritz values with the dense spectrum of the
even/odd operator, hermitian Rayleigh-Ritz pairs with dense eigh (through
the projector sum_q e e^+ / lambda, since phases and degenerate rotations
are free).  Iteration counts are not compared.  The full-size case checks
the true residual recomputed by the oracle.
"""
import numpy as np
import pytest

from tests.gpu_common import require_gpu, context, to_gpu, to_host, say, rel_err
from oracle import lattice as L
from oracle import wilson as W
from oracle import krylov as K
from oracle.noise import z4_noise

pytestmark = pytest.mark.gpu


def _dense_solve(U, kappa, dims, eta):
    M = W.dense_M(U, kappa, dims)
    n = eta.shape[0]
    return np.linalg.solve(M, eta.reshape(n, -1).T).T.reshape(eta.shape), M


@pytest.mark.parametrize("dims,kappa,nrhs,block", [((4, 4, 4, 4), 0.12, 4, 2),
                                                    ((6, 4, 2, 8), 0.13, 5, 3),
                                                    ((4, 4, 4, 4), 0.12, 13, 13)])
def test_schur_solve_fp64(dims, kappa, nrhs, block):
    """Blocks of 13 right-hand sides take the matrix-core projection in tiles
    of 8 + 5 columns."""
    require_gpu()
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2001, dims, 0, nrhs)
    say("solve schur f64", dims, kappa, nrhs, block)
    x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=20, k=10, tol=1e-12,
                                    tol_super=1e-13, rhs_block=block)
    x = to_host(x)
    xref, _ = _dense_solve(U, kappa, dims, eta)
    for r in range(nrhs):
        assert rel_err(x[r], xref[r]) < 1e-10, r
        assert st[r]["true_resid"] < 1e-11, st[r]
    # a second call reuses the deflation space (GMRES-Proj for every rhs)
    say("solve schur f64 reuse", dims)
    x2, _, st2 = ctx.gmresdr_solve(to_gpu(eta[1:2]), op="schur", m=20, k=10, tol=1e-12, defl=defl)
    assert rel_err(to_host(x2)[0], xref[1]) < 1e-10


@pytest.mark.parametrize("m", [90, 100])
def test_schur_solve_large_basis(m):
    """Restarts of bases of m + 1 = 91 vectors (recombination by the
    persistent kernel with 64-element tiles and the coefficients in LDS) and
    of 101 vectors (the general LDS-staged form): same solution as dense LU.
    On this lattice and kappa the oracle's GMRES-DR(m, 40) takes 3 cycles."""
    require_gpu()
    dims, kappa = (4, 4, 4, 4), 0.19
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2001, dims, 0, 1)
    say("solve schur f64 large basis", dims, kappa, "m", m)
    x, _, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=m, k=40, tol=1e-12, tol_super=1e-13,
                                 max_cycles=200)
    assert st[0]["cycles"] >= 2, st[0]  # at least one restart
    xref, _ = _dense_solve(U, kappa, dims, eta)
    assert rel_err(to_host(x)[0], xref[0]) < 1e-10
    assert st[0]["true_resid"] < 1e-11, st[0]


def test_harmonic_ritz_values_gpu():
    """Super-converged GMRES-DR: converged harmonic Ritz values are
    eigenvalues of Mhat (dense), like the oracle's."""
    require_gpu()
    dims, kappa = (4, 4, 2, 4), 0.13
    ctx, U = context(dims, 0.3, 31, kappa)
    eta = z4_noise(5, dims, 0, 1)
    say("ritz", dims)
    _, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=14, k=7, tol=1e-13, tol_super=1e-13,
                                    eig_tol=1e-11, n_eig=3, max_cycles=400)
    theta = defl.ritz()
    ev, od = L.eo_tables(dims)
    M = W.dense_M(U, kappa, dims)
    ie = np.concatenate([np.arange(12 * s, 12 * s + 12) for s in ev])
    io = np.concatenate([np.arange(12 * s, 12 * s + 12) for s in od])
    Mhat = np.eye(ie.size) - M[np.ix_(ie, io)] @ M[np.ix_(io, ie)]
    lam = np.linalg.eigvals(Mhat)
    # oracle run on the same problem
    shape = eta[0].shape
    A = lambda v: W.apply_Mhat(U, kappa, v.reshape(shape), dims).ravel()
    src = W.eo_source(U, kappa, eta[0], dims).ravel()
    _, oinfo = K.gmres_dr(A, src, 14, 7, 1e-13, max_cycles=400, eig_tol=1e-11, n_eig=3)
    for t in theta[:3]:
        assert np.min(np.abs(lam - t)) < 1e-9
        assert np.min(np.abs(oinfo["theta"] - t)) < 1e-9


def test_hermitian_solve_and_eigpairs():
    require_gpu()
    dims, kappa = (4, 4, 2, 4), 0.125
    ctx, U = context(dims, 0.3, 31, kappa)
    eta = z4_noise(5, dims, 0, 2)
    say("solve MG5", dims)
    x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="MG5", m=40, k=20, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-11, n_eig=8, max_cycles=300)
    M = W.dense_M(U, kappa, dims)
    Mp = M @ W.dense_gamma(L.GAMMA5, L.volume(dims))
    xref = np.linalg.solve(Mp, eta.reshape(2, -1).T).T
    x = to_host(x).reshape(2, -1)
    for r in range(2):
        assert rel_err(x[r], xref[r]) < 1e-10
    Q = 6
    lam, res = defl.eigpairs(Q)
    lam_d, E_d = K.hermitian_eigpairs_dense(Mp, Q)
    assert (res < 1e-9).all()
    assert np.abs(lam - lam_d).max() < 1e-9


def _near_critical_kappa(U, dims):
    """kappa in [0.13, 0.26] where M' = M g5 of this small lattice has its
    smallest |eigenvalue| on a coarse grid (an eigenvalue crossing zero)."""
    best = None
    for kappa in np.linspace(0.13, 0.26, 27):
        M = W.dense_M(U, kappa, dims)
        lam = np.linalg.eigvalsh(M @ W.dense_gamma(L.GAMMA5, L.volume(dims)))
        v = np.abs(lam).min()
        if best is None or v < best[1]:
            best = (kappa, v)
    return best


@pytest.mark.parametrize("near_critical", [False, True])
def test_minres_dr_hermitian(near_critical):
    """MINRES-DR on M' = M g5 (full lattice): solutions vs dense LU, Ritz
    pairs vs dense eigh, harmonic Ritz values vs the oracle's MINRES-DR, at
    a moderate kappa and at a kappa where an eigenvalue of M' is near zero
    (the regime where the hermitian system needs MINRES-DR)."""
    require_gpu()
    dims = (4, 4, 2, 4)
    ctx, U = context(dims, 0.3, 31, 0.125)
    kappa = 0.125
    if near_critical:
        kappa, lmin = _near_critical_kappa(U, dims)
        ctx.set_kappa(kappa)
    eta = z4_noise(5, dims, 0, 2)
    say("MINRES-DR MG5", dims, "kappa", kappa)
    x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="MG5", m=40, k=20, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-11, n_eig=8, max_cycles=400, method="minres-dr")
    M = W.dense_M(U, kappa, dims)
    Mp = M @ W.dense_gamma(L.GAMMA5, L.volume(dims))
    xref = np.linalg.solve(Mp, eta.reshape(2, -1).T).T
    xg = to_host(x).reshape(2, -1)
    cond = np.linalg.cond(Mp)
    for r in range(2):
        assert rel_err(xg[r], xref[r]) < 1e-13 * cond + 1e-10
        assert st[r]["true_resid"] < 1e-11
    Q = 6
    lam, res = defl.eigpairs(Q)
    lam_d, E_d = K.hermitian_eigpairs_dense(Mp, Q)
    assert (res < 1e-9).all()
    assert np.abs(lam - lam_d).max() < 1e-9
    # the oracle's MINRES-DR reaches the same harmonic Ritz values
    shape = eta[0].shape
    Ap = lambda v: W.apply_Mprime(U, kappa, v.reshape(shape)).ravel()
    _, info = K.minres_dr(Ap, eta[0].ravel(), 40, 20, 1e-13, max_cycles=400, eig_tol=1e-11, n_eig=8)
    th_o = np.sort(info["theta"][:6].real)
    th_g = np.sort(defl.ritz()[:6].real)
    assert np.abs(th_g - th_o).max() < 1e-9 * np.abs(th_o).max()


def test_gamma5_matches_oracle():
    require_gpu()
    dims = (4, 4, 2, 4)
    ctx, U = context(dims, 0.3, 31, 0.125)
    rng = np.random.default_rng(4)
    x = rng.standard_normal((3,) + ctx.shape) + 1j * rng.standard_normal((3,) + ctx.shape)
    y = to_host(ctx.gamma5(to_gpu(x)))
    assert np.array_equal(y, W.g5(x))
    xg = to_gpu(x)
    ctx.gamma5(xg, out=xg)  # in place
    assert np.array_equal(to_host(xg), W.g5(x))


def test_single_special_rhs_production():
    """Sec. 10's production setup: the hermitian modes of one MINRES-DR solve
    deflate every later solve of M' (GMRES-Proj on LQCD_OP_MG5, mixed
    precision), and x = g5 y solves M x = eta (compared with dense LU)."""
    require_gpu()
    dims, kappa = (4, 4, 2, 4), 0.125
    ctx, U = context(dims, 0.3, 31, kappa)
    eta0 = z4_noise(5, dims, 0, 1)
    say("production: MINRES-DR modes", dims)
    _, hdefl, _ = ctx.gmresdr_solve(to_gpu(eta0), op="MG5", m=40, k=20, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-10, n_eig=10, max_cycles=300, method="minres-dr")
    eta = z4_noise(6, dims, 0, 4)
    say("production: deflated MG5 solves")
    y, _, st = ctx.gmresdr_solve(to_gpu(eta), op="MG5", m=40, k=20, tol=1e-11, defl=hdefl, inner="f32",
                                 inner_tol=1e-4, rhs_block=4)
    x = to_host(ctx.gamma5(y))
    xref, _ = _dense_solve(U, kappa, dims, eta)
    for r in range(4):
        assert rel_err(x[r], xref[r]) < 1e-9
        assert st[r]["true_resid"] < 1e-11


def test_minres_dr_rejects_non_hermitian_operator():
    require_gpu()
    from paper_1903_06986_amd.lqcd import LqcdError
    dims = (4, 4, 2, 4)
    ctx, U = context(dims, 0.3, 31, 0.125)
    eta = z4_noise(5, dims, 0, 1)
    with pytest.raises(LqcdError):
        ctx.gmresdr_solve(to_gpu(eta), op="schur", m=20, k=10, method="minres-dr")


@pytest.mark.parametrize("op,method", [("schur", "gmres-dr"), ("MG5", "gmres-dr"), ("MG5", "minres-dr")])
def test_first_rhs_cut_off_by_max_cycles_is_enoconv(op, method):
    """Two cycles of GMRES-DR(8,4) / MINRES-DR(8,4) cannot reach 1e-12 on
    a 4^4 lattice near kappa 0.13: the call must report ENOCONV (with the
    deflation space still handed back), not LQCD_OK."""
    require_gpu()
    import ctypes
    from paper_1903_06986_amd import lqcd
    dims = (4, 4, 4, 4)
    ctx, U = context(dims, 0.3, 33, 0.13)
    eta = to_gpu(z4_noise(6, dims, 0, 2))
    say("solve cut off", op, method)
    x = eta.clone()
    p = lqcd.SolveParams(8, 4, 2, 1e-12, 1e-12, 0.0, 0, lqcd.F64, 1e-5, 1, 0, lqcd._METHODS[method])
    st = (lqcd.SolveStats * 2)()
    h = ctypes.c_void_p(None)
    code = lqcd.lib().gmresdr_solve(ctx.handle, lqcd._OPS[op], ctypes.byref(p), lqcd._ptr(eta),
                                    lqcd._ptr(x), 2, ctypes.byref(h), st)
    assert code == 4, code                       # LQCD_ENOCONV
    assert h.value is not None                   # the deflation space is returned
    assert st[0].cycles == 2 and st[0].true_resid > 1e-12
    lqcd.lib().lqcd_defl_free(h)


@pytest.mark.parametrize("dims,kappa,nrhs,block", [((4, 4, 4, 4), 0.12, 5, 4), ((6, 4, 2, 8), 0.13, 5, 4),
                                                    ((4, 4, 4, 4), 0.12, 12, 12)])
def test_mixed_precision_solve(dims, kappa, nrhs, block):
    require_gpu()
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2001, dims, 0, nrhs)
    say("solve mixed", dims, nrhs, block)
    x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=20, k=10, tol=1e-11, tol_super=1e-13,
                                    inner="f32", inner_tol=1e-5, rhs_block=block)
    x = to_host(x)
    xref, _ = _dense_solve(U, kappa, dims, eta)
    for r in range(nrhs):
        assert rel_err(x[r], xref[r]) < 1e-9
        assert st[r]["true_resid"] < 1e-11
    assert all(s["refinements"] >= 1 for s in st[1:])


def test_full_size_true_residual_16x32():
    require_gpu()
    dims, kappa = (16, 16, 16, 32), 0.12
    ctx, U = context(dims, 0.25, 1002, kappa)
    eta = z4_noise(2002, dims, 0, 3)
    say("solve full size", dims)
    x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=50, k=30, tol=1e-10, tol_super=1e-12,
                                    rhs_block=2)
    x = to_host(x)
    for r in range(3):
        res = np.linalg.norm(eta[r] - W.apply_M(U, kappa, x[r])) / np.linalg.norm(eta[r])
        assert res < 1.5e-10, (r, res)
        assert abs(res - st[r]["true_resid"]) < 1e-12


@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_matrix_core_deflation_products(inner):
    """The deflation products V C with one shared basis (GMRES-Proj's
    x += V_k d and r -= V_{k+1} Hbar d for a block of right-hand sides, the
    Rayleigh-Ritz eigenvectors, the hermitian projections) run on the
    matrix cores; the FMA kernel is the reference.  Both give the LU
    solution to 1e-9 (their iterates differ by rounding only, so the two
    solutions agree to the solver tolerance), and the Rayleigh-Ritz
    eigenvalues of the same hermitian space agree to 1e-12."""
    require_gpu()
    dims, kappa = (6, 4, 2, 8), 0.13
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2001, dims, 0, 13)
    xs = []
    for mfma in (0, 1):
        ctx.tune(gemm_mfma=mfma)
        say("solve gemm_mfma", mfma, inner)
        x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=20, k=10, tol=1e-11, tol_super=1e-13,
                                        inner=inner, inner_tol=1e-5, rhs_block=13)
        assert max(s["true_resid"] for s in st) < 1e-11
        xs.append(to_host(x))
        _, hdefl, _ = ctx.gmresdr_solve(to_gpu(eta[:1]), op="MG5", m=30, k=18, tol=1e-12, tol_super=1e-13,
                                        eig_tol=1e-11, n_eig=12, max_cycles=400)
        lam, res = hdefl.eigpairs(12)
        if mfma == 0:
            lam0 = lam
        else:
            assert np.abs(lam - lam0).max() < 1e-10
    ctx.tune(gemm_mfma=1)
    xref, _ = _dense_solve(U, kappa, dims, eta)
    for x in xs:
        for r in range(13):
            assert rel_err(x[r], xref[r]) < 1e-9
    assert rel_err(xs[0], xs[1]) < 1e-9


@pytest.mark.parametrize("method,op", [("gmres-dr", "schur"), ("minres-dr", "MG5")])
def test_recombination_forms_agree(method, op):
    """The restart recombination V_{k+1} = V_{m+1} P in its two forms
    (outputs in registers with P in LDS, and the LDS-tiled form) gives the
    same first-right-hand-side solve: solutions and harmonic Ritz values
    agree to rounding, and the solution reaches LU."""
    require_gpu()
    dims, kappa = (6, 4, 2, 8), 0.13
    ctx, U = context(dims, 0.3, 31, kappa)
    eta = z4_noise(5, dims, 0, 1)
    out = {}
    try:
        for regs in (1, 0):
            ctx.tune(recombine_regs=regs)
            say("recombination form", regs, method)
            x, defl, st = ctx.gmresdr_solve(to_gpu(eta), op=op, m=16, k=8, tol=1e-12, tol_super=1e-13,
                                            max_cycles=400, method=method)
            assert st[0]["cycles"] > 2, st[0]  # several restarts ran
            out[regs] = (to_host(x), np.sort_complex(defl.ritz()[:10]), st[0]["matvecs"])
    finally:
        ctx.tune(recombine_regs=1)
    M = W.dense_M(U, kappa, dims)
    if op == "MG5":
        M = M @ W.dense_gamma(L.GAMMA5, L.volume(dims))
        xref = np.linalg.solve(M, eta.reshape(1, -1).T).T.reshape(eta.shape)
    else:
        xref = np.linalg.solve(M, eta.reshape(1, -1).T).T.reshape(eta.shape)
    assert rel_err(out[1][0], xref) < 1e-9
    assert rel_err(out[1][0], out[0][0]) < 1e-11
    assert np.abs(out[1][1] - out[0][1]).max() < 1e-9 * np.abs(out[0][1]).max()
    assert abs(out[1][2] - out[0][2]) <= 8


@pytest.mark.parametrize("m", [19, 20, 21])
@pytest.mark.parametrize("forced", [0, 1])
@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_sstep_arnoldi_plain_basis(inner, forced, m):
    """Several Arnoldi steps per pass over an FP64 or FP32 basis span the same
    Krylov space as single ones: solutions reach LU and the true residual in
    about as many matrix-vector products, with the second pass forced on every
    block and with last blocks of 1 to 3 steps (p = 9, 10, 11)."""
    require_gpu()
    dims, kappa = (6, 4, 2, 8), 0.13
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2003, dims, 0, 4)
    xref, _ = _dense_solve(U, kappa, dims, eta)
    st = {}
    for steps in (1, 2, 3, 4, 6):  # 6: blocks of 4, the longest on these bases
        ctx.tune(arnoldi_steps=steps, cycle_reorth=forced)
        say("solve s-step", inner, forced, m, steps)
        x, _, s = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=m, k=10, tol=1e-12, tol_super=1e-13, inner=inner,
                                    inner_tol=1e-4, rhs_block=3)
        x = to_host(x)
        for r in range(4):
            assert rel_err(x[r], xref[r]) < (1e-10 if inner == "f64" else 1e-9), (steps, r)
            assert s[r]["true_resid"] < 1e-11, (steps, r)
        st[steps] = s
    for steps in (2, 3, 4, 6):
        for r in range(1, 4):
            assert st[steps][r]["matvecs"] <= st[1][r]["matvecs"] + (m - 10 + 1), (steps, r)
            assert (st[steps][r]["reorth"] > 0) == bool(forced), (steps, r)


@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_sstep_arnoldi_plain_basis_two_units_per_lane(inner):
    """A field large enough for two 16-byte units per lane and the separate
    sums, plan and finish launches: same solution as single steps."""
    require_gpu()
    dims, kappa, nrhs = (16, 12, 12, 24), 0.124, 6
    ctx, _ = context(dims, 0.25, 1004, kappa)
    eta = to_gpu(z4_noise(2004, dims, 0, nrhs))
    kw = dict(op="schur", m=30, k=10, tol=1e-12, inner=inner, inner_tol=1e-4, rhs_block=nrhs)
    _, defl, _ = ctx.gmresdr_solve(eta[0:1], op="schur", m=30, k=10, tol=1e-10)
    xs = {}
    for steps in (1, 4):
        ctx.tune(arnoldi_steps=steps)
        say("solve s-step", inner, dims, steps)
        xs[steps], _, st = ctx.gmresdr_solve(eta, defl=defl, **kw)
        for s in st:
            assert s["true_resid"] <= 1.05e-12, s
    a, b = to_host(xs[1]), to_host(xs[4])
    # both within 1e-12 / lambda_min(M) of the solution, lambda_min > 0.05 here
    assert np.linalg.norm(a - b) < 4e-11 * np.linalg.norm(a)


@pytest.mark.parametrize("zeros", [(), (1,), (2, 4), (1, 2, 3), (5,), (1, 2, 3, 4, 5)])
@pytest.mark.parametrize("inner", ["f64", "f32", "f16"])
def test_finished_right_hand_sides_change_places(zeros, inner):
    """A block whose right-hand sides finish at different times: zero sources,
    finished before the first cycle, at the front, middle and end of a block of
    five, and one eigenvector-like source among noise.  Every solution belongs
    to its own source (LU, 1e-9, the bar of the solver's other tests) and the
    sources stay as they were."""
    require_gpu()
    dims, kappa = (4, 4, 2, 4), 0.13
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2003, dims, 0, 6).astype(np.complex128)
    eta[3] *= 1e-3
    for z in zeros:
        eta[z] = 0
    M = W.dense_M(U, kappa, dims)
    xref = np.linalg.solve(M, eta.reshape(6, -1).T).T.reshape(eta.shape)
    say("solve swaps", zeros, inner)
    eg = to_gpu(eta)
    x, _, st = ctx.gmresdr_solve(eg, op="schur", m=20, k=10, tol=1e-11, tol_super=1e-13, inner=inner,
                                 inner_tol=1e-3, rhs_block=5)
    x = to_host(x)
    np.testing.assert_array_equal(to_host(eg), eta)
    for r in range(6):
        if r in zeros:
            np.testing.assert_array_equal(x[r], 0)
        else:
            assert rel_err(x[r], xref[r]) < 1e-9, r
            assert st[r]["true_resid"] < 1e-11, r


@pytest.mark.parametrize("m,k", [(5, 2), (8, 3), (13, 6), (34, 17)])
@pytest.mark.parametrize("dims", [(2, 2, 2, 4), (6, 4, 4, 4)])
def test_dots_split_over_the_basis(dims, m, k):
    """Single Arnoldi steps on small lattices, whose dot passes split the basis
    into groups of two or more vectors (1 to 35 of them here: one vector, odd
    and even counts, ragged last groups): solutions against LU (1e-9) and the
    true residual, FP64 and FP32 bases, one and three right-hand sides at once."""
    require_gpu()
    kappa = 0.12
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2003, dims, 0, 4).astype(np.complex128)
    xref, _ = _dense_solve(U, kappa, dims, eta)
    ctx.tune(arnoldi_steps=1)
    for inner in ("f64", "f32"):
        say("dot groups", dims, m, k, inner)
        x, _, st = ctx.gmresdr_solve(to_gpu(eta), op="schur", m=m, k=k, tol=1e-11, tol_super=1e-12, inner=inner,
                                     inner_tol=1e-3, rhs_block=3, max_cycles=400)
        x = to_host(x)
        for r in range(4):
            assert rel_err(x[r], xref[r]) < 1e-9, (inner, r)
            assert st[r]["true_resid"] < 1e-11, (inner, r)


@pytest.mark.parametrize("inner", ["f64", "f32"])
def test_sstep_blocks_need_no_vectors_beside_the_basis(inner):
    """Device memory of a solve with four Arnoldi steps per basis pass against
    single steps: the powers of a block lie in the basis, so the two differ by
    sums (16 MB here) and not by four vectors of every right-hand side (404 MB
    in FP64, 202 MB in FP32): a solve that fits with single steps fits."""
    require_gpu()
    import torch
    dims, nrhs = (16, 16, 16, 32), 9
    half = 12 * int(np.prod(dims)) // 2 * (16 if inner == "f64" else 8)
    used = {}
    for steps in (1, 1, 4):  # the first pass fills torch's pool
        torch.cuda.synchronize()
        ctx, _ = context(dims, 0.25, 1002, 0.11)
        free0 = torch.cuda.mem_get_info()[0]
        ctx.tune(arnoldi_steps=steps)
        say("solver memory", inner, steps)
        x, _, st = ctx.gmresdr_solve(ctx.noise_z4(7, 0, nrhs), op="schur", m=30, k=10, tol=1e-8, inner=inner,
                                     rhs_block=nrhs - 1)
        torch.cuda.synchronize()
        used[steps] = free0 - torch.cuda.mem_get_info()[0]
        assert max(s["true_resid"] for s in st) < 2e-8
        del x
        ctx.close()
    assert used[4] - used[1] < (nrhs - 1) * half, used


@pytest.mark.parametrize("inner", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(6, 4, 2, 8), (16, 12, 12, 24)])
def test_second_passes_are_counted_in_steps(inner, dims):
    """With the second pass forced, every step of every cycle counts, also where
    a block of steps takes it together (a last block of one, short sums in one
    launch on the first lattice, the separate launches on the second)."""
    require_gpu()
    ctx, _ = context(dims, 0.3, 1001, 0.12)
    eta = ctx.noise_z4(9, 0, 4)
    for steps in (1, 2, 3, 4):
        ctx.tune(arnoldi_steps=steps, cycle_reorth=1)
        say("second passes", inner, dims, steps)
        _, _, st = ctx.gmresdr_solve(eta, op="schur", m=23, k=10, tol=1e-8, inner=inner, inner_tol=1e-4, rhs_block=3)
        for s in st[1:]:
            assert s["reorth"] == 13 * s["cycles"] > 0, (steps, s)


@pytest.mark.parametrize("p", [24, 60, 120])
def test_one_long_cycle_of_blocks_reaches_the_residual_of_single_steps(p):
    """One GMRES cycle of p steps on an FP64 basis, in blocks and step by step
    from the same start: the residual is the smallest in the same Krylov space.
    A basis orthonormal to d leaves it larger by d of itself (d <= 1e-11 p where a
    block is stored without its second pass), and an Arnoldi relation off by 1e-15
    per product, times 1e3 for the pivot bound, by 1e-12 of the source."""
    require_gpu()
    dims, kappa = (6, 4, 2, 8), 0.13
    ctx, _ = context(dims, 0.3, 1001, kappa)
    eta = to_gpu(z4_noise(2003, dims, 0, 4))
    _, defl, _ = ctx.gmresdr_solve(eta[:1], op="schur", m=20, k=10, tol=1e-12, tol_super=1e-13)
    res = {}
    for steps in (1, 2, 3, 4):
        ctx.tune(arnoldi_steps=steps)
        say("one cycle", p, steps)
        _, _, st = ctx.gmresdr_solve(eta, op="schur", m=20, k=10, tol=0.05, rhs_block=4, defl=defl, proj_m=p)
        assert all(s["cycles"] == 1 and s["reorth"] == 0 for s in st), st
        res[steps] = np.array([s["true_resid"] for s in st])
    print("residuals after one cycle", res)
    for steps in (2, 3, 4):
        assert np.all(np.abs(res[steps] - res[1]) <= 1e-8 * res[1] + 1e-12), (steps, res)


@pytest.mark.parametrize("steps", [1, 2, 3, 4])
@pytest.mark.parametrize("inner", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(2, 2, 2, 4), (4, 4, 2, 4)])
def test_sstep_blocks_in_small_invariant_subspaces(dims, inner, steps):
    """Sources whose Krylov space ends inside a block (the free operator on a
    constant field, and on one that differs between the parities: exact
    eigenvectors; a sum of eigenvectors of a random field: dimension 1 to 6), beside
    noise in the same block: a Cholesky pivot vanishes and the rest of the block's
    vectors are zero.  Solutions against LU, and eigenvectors take no more
    cycles than noise."""
    require_gpu()
    kappas = (0.0625, 0.03125, 0.11)
    for kappa in kappas:
        for free in (True, False):
            ctx, U = context(dims, 0.3, 1001, kappa, unit=free)
            eta = z4_noise(3, dims, 0, 8).astype(np.complex128)
            par = np.broadcast_to(W.parity_mask(dims) == 0, ctx.shape)
            M = W.dense_M(U, kappa, dims)
            if free:
                eta[1] = 1.0
                eta[2] = np.where(par, 1.0, 2.0)
                eta[2][..., 0, 0] *= 3
                eta[4] = np.where(par, 1.0, 0.0)
                eta[5] = 0.0
                eta[5][..., 1, 2] = 1.0
                eta[6] = eta[4] + 1e-6 * eta[6]
            else:
                flat = par.reshape(-1)
                E, O = np.flatnonzero(flat), np.flatnonzero(~flat)
                lam, vec = np.linalg.eig(M[np.ix_(E, E)] - M[np.ix_(E, O)] @ M[np.ix_(O, E)])
                order = np.argsort(-np.abs(lam))
                for r, count in ((1, 1), (2, 2), (4, 3), (5, 4), (6, 6)):
                    e = np.zeros(M.shape[0], complex)
                    e[E] = vec[:, order[:count]].sum(1)
                    eta[r] = e.reshape(ctx.shape)
            xref = np.linalg.solve(M, eta.reshape(8, -1).T).T.reshape(eta.shape)
            say("invariant subspaces", dims, inner, steps, kappa, "free" if free else "random")
            _, defl, _ = ctx.gmresdr_solve(to_gpu(eta[:1]), op="schur", m=20, k=10, tol=1e-12)
            ctx.tune(arnoldi_steps=steps)
            x, _, st = ctx.gmresdr_solve(to_gpu(eta[1:]), op="schur", m=20, k=10, tol=1e-11, inner=inner,
                                         inner_tol=1e-4, rhs_block=7, defl=defl, max_cycles=200)
            x = to_host(x)
            for r in range(7):
                assert rel_err(x[r], xref[r + 1]) < 1e-9, (kappa, free, r)
                assert st[r]["true_resid"] < 1e-11, (kappa, free, r, st[r])
            assert st[0]["cycles"] <= st[2]["cycles"], (kappa, free, st)


@pytest.mark.parametrize("quick", [(1,), (3,), (5,), (1, 2), (2, 4), (1, 2, 3, 4)])
@pytest.mark.parametrize("inner", ["f64", "f32", "f16"])
def test_right_hand_sides_that_finish_cycles_apart_change_places(quick, inner):
    """Some right-hand sides of a block of five are eigenvectors of Mhat that the
    deflation space holds to 1e-9, so the first projection leaves them little to
    do, at the front, middle and end among noise that goes on: finished slots change places with active ones that have run cycles.
    Every solution belongs to its own source (LU, 1e-9), the sources stay as they
    were, and the counts are each right-hand side's own."""
    require_gpu()
    dims, kappa = (4, 4, 2, 4), 0.13
    ctx, U = context(dims, 0.3, 1001, kappa)
    M = W.dense_M(U, kappa, dims)
    par = np.broadcast_to(W.parity_mask(dims) == 0, ctx.shape).reshape(-1)
    E, O = np.flatnonzero(par), np.flatnonzero(~par)
    lam, vec = np.linalg.eig(M[np.ix_(E, E)] - M[np.ix_(E, O)] @ M[np.ix_(O, E)])
    order = np.argsort(np.abs(lam))
    eta = z4_noise(2003, dims, 0, 6).astype(np.complex128)
    for r in quick:
        e = np.zeros(M.shape[0], complex)
        e[E] = vec[:, order[r]]
        eta[r] = 3.0 ** r * e.reshape(ctx.shape)
    xref = np.linalg.solve(M, eta.reshape(6, -1).T).T.reshape(eta.shape)
    say("solve swaps", quick, inner)
    eg = to_gpu(eta)
    x, _, st = ctx.gmresdr_solve(eg, op="schur", m=30, k=16, tol=1e-11, tol_super=1e-13, eig_tol=1e-9, n_eig=8,
                                 max_cycles=400, inner=inner, inner_tol=1e-3, rhs_block=5)
    x = to_host(x)
    np.testing.assert_array_equal(to_host(eg), eta)
    for r in range(6):
        assert rel_err(x[r], xref[r]) < 1e-9, r
        assert st[r]["true_resid"] < 1e-11, r
    slow = [r for r in range(1, 6) if r not in quick]
    assert max(st[r]["cycles"] for r in quick) < min([st[r]["cycles"] for r in slow] + [99]), st
    if inner == "f64":
        assert all(st[r]["matvecs"] == 15 * st[r]["cycles"] for r in range(1, 6)), st

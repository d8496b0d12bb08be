"""GPU parity of pert_subtract, poly_subtract, deflate_project and
loop_estimate against the oracle, plus closed-form pins of the exact trace
corrections (the GPU computes them by closed-walk enumeration, the oracle
by dense powers / unit probes).

Tolerances: subtraction vectors 1e-12 relative (FP64 stencil chains),
trace corrections 1e-10 relative, Min-Res coefficients 1e-8 relative
(normal equations on the GPU vs Householder QR in the oracle), estimates
1e-9 * max(|T|, sigma) as the path's target states.
"""
import itertools

import numpy as np
import pytest

from tests.gpu_common import require_gpu, context, to_gpu, to_host, say, rel_err
from oracle import lattice as L
from oracle import wilson as W
from oracle import subtract as S
from oracle import estimate as E
from oracle import krylov as K
from oracle.noise import z4_noise

pytestmark = pytest.mark.gpu
THETAS = (0, 1, 2, 3, 4)


def _oracle_corr(U, kappa, coeffs, dims):
    if L.volume(dims) <= 256:
        A = S.poly_dense(W.dense_P(U, dims), kappa, coeffs)
        return S.trace_correction_dense(A, dims, THETAS)
    return S.trace_correction_probe(U, kappa, coeffs, dims, THETAS)


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 4, 4, 4), (6, 4, 2, 8)])
@pytest.mark.parametrize("order", [4, 7])
def test_pert_subtract(dims, order):
    require_gpu()
    kappa = 0.12
    ctx, U = context(dims, 0.3, 77, kappa)
    eta = z4_noise(9, dims, 0, 3)
    say("pert", dims, order)
    xt, corr = ctx.pert_subtract(order, to_gpu(eta), THETAS)
    ref = S.pert_vector(U, kappa, eta, order)
    assert rel_err(to_host(xt), ref) < 1e-12
    cref = _oracle_corr(U, kappa, S.pert_coeffs(order), dims)
    assert np.abs(corr - cref).max() < 1e-10 * np.abs(cref).max()


def _single_power_trace(ctx, j, n_t):
    """Tr_t(Theta P^j) from poly_subtract with coefficients e_j at kappa = 1."""
    import torch
    c = np.zeros(j + 1, dtype=np.complex128)
    c[j] = 1.0
    eta = torch.zeros((1,) + ctx.shape, dtype=torch.complex128, device="cuda")
    _, corr, _, _ = ctx.poly_subtract(j, eta, b=None, coeffs=c, thetas=THETAS)
    return corr


def test_trace_closed_forms_free_field_8():
    """Free field, extents >= 7: Tr P^4 / V = -1152, Tr P^6 / V = -50688,
    Tr P^2 = 0, and every g_mu trace vanishes."""
    require_gpu()
    dims = (8, 8, 8, 8)
    ctx, _ = context(dims, 0.0, 0, 1.0, unit=True)
    V = L.volume(dims)
    say("free-field walk traces", dims)
    for j, ref in ((2, 0.0), (4, -1152.0), (6, -50688.0)):
        corr = _single_power_trace(ctx, j, dims[3])
        assert abs(corr[0].sum() / V - ref) < 1e-9
        assert np.abs(corr[1:]).max() < 1e-9
        # translation invariance: equal timeslices
        assert np.abs(corr[0] - corr[0].mean()).max() < 1e-8


def test_trace_plaquette_form_L6():
    """Random links, extents >= 5: Tr P^4 = -64 sum_plaq Re tr U_P and
    Tr g4 P^4 = 0 (only plaquettes close in four hops)."""
    require_gpu()
    from tests.test_oracle_wilson import plaquette_sum
    dims = (6, 6, 6, 6)
    ctx, U = context(dims, 0.3, 12, 1.0)
    say("plaquette walk traces", dims)
    corr = _single_power_trace(ctx, 4, dims[3])
    ref = -64.0 * plaquette_sum(U)
    assert abs(corr[0].sum() - ref) < 1e-11 * abs(ref)
    assert abs(corr[4].sum()) < 1e-10 * abs(ref)


def test_poly_subtract():
    require_gpu()
    dims, kappa, d = (4, 4, 4, 4), 0.12, 7
    ctx, U = context(dims, 0.3, 1001, kappa)
    eta = z4_noise(2001, dims, 0, 4)
    say("poly", dims, d)
    xt, corr, c, a = ctx.poly_subtract(d, to_gpu(eta), b=to_gpu(eta[0:1]), thetas=THETAS)
    c_ref, a_ref = S.poly_coeffs(U, kappa, eta[0], d)
    assert np.abs(c - c_ref).max() < 1e-8 * np.abs(c_ref).max()
    assert np.abs(a - a_ref).max() < 1e-7 * np.abs(a_ref).max()
    # with the GPU's coefficients the vectors and corrections match to rounding
    assert rel_err(to_host(xt), S.horner(U, kappa, eta, c)) < 1e-12
    cref = _oracle_corr(U, kappa, c, dims)
    assert np.abs(corr - cref).max() < 1e-10 * np.abs(cref).max()


def test_deflate_project_vs_dense_eigenpairs():
    require_gpu()
    dims, kappa, Q = (4, 4, 2, 4), 0.125, 6
    ctx, U = context(dims, 0.3, 31, kappa)
    eta = z4_noise(5, dims, 0, 3)
    say("deflate_project", dims)
    _, hdefl, _ = ctx.gmresdr_solve(to_gpu(eta[0:1]), op="MG5", m=40, k=20, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-11, n_eig=Q + 2, max_cycles=300)
    M = W.dense_M(U, kappa, dims)
    Mp = M @ W.dense_gamma(L.GAMMA5, L.volume(dims))
    lam, Ev = K.hermitian_eigpairs_dense(Mp, Q)
    shape = eta[0].shape
    Et = Ev.T.reshape((Q,) + shape)
    # HFES
    import torch
    xt, corr, _ = ctx.deflate_project(hdefl, Q, to_gpu(eta), xt=torch.zeros((3,) + shape, dtype=torch.complex128,
                                                                               device="cuda"))
    inv = 1.0 / lam + 0j
    assert rel_err(to_host(xt), S.eig_vector(Et, inv, eta)) < 1e-9
    assert np.abs(corr - S.site_bilinear(Et, THETAS, dims, inv)).max() < 1e-9 * np.abs(corr).max()
    # EIGPOLY with the perturbative polynomial: weights 1/lambda - 1/xi
    cp = S.pert_coeffs(6)
    xi = S.xi_inverse(U, kappa, Et, cp)
    xt2, corr2, xi_gpu = ctx.deflate_project(hdefl, Q, to_gpu(eta), xt=torch.zeros_like(xt),
                                             mode=1, coeffs=cp)
    assert np.abs(xi_gpu - xi).max() < 1e-9 * np.abs(xi).max()
    assert rel_err(to_host(xt2), S.eig_vector(Et, inv - xi, eta)) < 1e-9


def test_loop_estimate_function():
    require_gpu()
    dims = (4, 2, 6, 4)
    ctx, U = context(dims, 0.3, 3, 0.1)
    rng = np.random.default_rng(8)
    shape = (5,) + ctx.shape
    eta = z4_noise(4, dims, 0, 5)
    x = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    xt = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    corr = rng.standard_normal((5, dims[3])) + 1j * rng.standard_normal((5, dims[3]))
    say("loop_estimate", dims)
    est, err, smp = ctx.loop_estimate(to_gpu(eta), to_gpu(x), to_gpu(xt), corr, THETAS, samples=True)
    t = E.samples(eta, x, xt, THETAS, dims)
    e_ref, s_ref = E.estimate(t, corr)
    assert np.abs(smp - t).max() < 1e-12 * np.abs(t).max()
    assert np.abs(est - e_ref).max() < 1e-12 * np.abs(e_ref).max()
    assert np.abs(err - s_ref).max() < 1e-12 * np.abs(s_ref).max()


def test_deflate_project_multi_equals_single_calls():
    """deflate_project_multi: each variant equals deflate_project with the
    same mode, coefficients, vector and correction bit for bit (overlaps
    formed once); modes other than HFES / EIGPOLY and more than four
    variants are rejected."""
    require_gpu()
    import torch
    from paper_1903_06986_amd import lqcd
    from paper_1903_06986_amd.lqcd import LqcdError
    dims, kappa, Q = (4, 4, 2, 4), 0.125, 6
    ctx, U = context(dims, 0.3, 31, kappa)
    n = 18  # a full block of 16 right-hand sides and a ragged one
    eta = to_gpu(z4_noise(5, dims, 0, n))
    say("deflate_project_multi", dims, n)
    _, hdefl, _ = ctx.gmresdr_solve(eta[0:1], op="MG5", m=40, k=20, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-11, n_eig=Q + 2, max_cycles=300)
    rng = np.random.default_rng(4)
    bases = [torch.from_numpy(rng.standard_normal((n,) + ctx.shape) + 0j).cuda() for _ in range(2)]
    corrs = [rng.standard_normal((5, dims[3])) + 1j * rng.standard_normal((5, dims[3])) for _ in range(2)]
    cp = S.pert_coeffs(6)
    cq = rng.standard_normal(4) + 1j * rng.standard_normal(4)
    variants = [(lqcd.DEFL_HFES, None, None, None),
                (lqcd.DEFL_EIGPOLY, cp, bases[0].clone(), corrs[0]),
                (lqcd.DEFL_EIGPOLY, cq, bases[1].clone(), corrs[1])]
    multi = ctx.deflate_project_multi(hdefl, Q, eta, variants, THETAS)
    refs = [ctx.deflate_project(hdefl, Q, eta, xt=torch.zeros_like(eta), mode=lqcd.DEFL_HFES, thetas=THETAS),
            ctx.deflate_project(hdefl, Q, eta, xt=bases[0].clone(), corr=corrs[0], mode=lqcd.DEFL_EIGPOLY,
                                coeffs=cp, thetas=THETAS),
            ctx.deflate_project(hdefl, Q, eta, xt=bases[1].clone(), corr=corrs[1], mode=lqcd.DEFL_EIGPOLY,
                                coeffs=cq, thetas=THETAS)]
    for (xt, corr), (xr, cr, _) in zip(multi, refs):
        np.testing.assert_array_equal(to_host(xt), to_host(xr))
        np.testing.assert_array_equal(corr, cr)
    with pytest.raises(LqcdError):
        ctx.deflate_project_multi(hdefl, Q, eta, [(lqcd.DEFL_ES, None, None, None)], THETAS)
    with pytest.raises(LqcdError):
        ctx.deflate_project_multi(hdefl, Q, eta, [(lqcd.DEFL_HFES, None, None, None)] * 5, THETAS)


@pytest.mark.parametrize("Q", [1, 15, 16, 17, 33])
def test_projection_on_the_matrix_cores_equals_the_other_form(Q):
    """V^H X and V C of the projection on the matrix cores (rows and columns
    in tiles of 16) against the FMA form, for one mode up to three tiles of
    them and 1, 15 and 18 right-hand sides, in one variant and in three, on
    given fields and on fresh ones (written, not added to).  Sums of 1536
    terms in another order: 1e-12 of the largest element."""
    require_gpu()
    import torch
    from paper_1903_06986_amd import lqcd
    dims, kappa = (4, 4, 2, 4), 0.125
    ctx, U = context(dims, 0.3, 31, kappa)
    eta = to_gpu(z4_noise(5, dims, 0, 18))
    say("projection tiles", Q)
    _, hdefl, _ = ctx.gmresdr_solve(eta[0:1], op="MG5", m=90, k=50, tol=1e-12, tol_super=1e-13,
                                    eig_tol=1e-8, n_eig=35, max_cycles=300)
    rng = np.random.default_rng(4)
    cp = S.pert_coeffs(6)
    base = torch.from_numpy(rng.standard_normal((18,) + ctx.shape) + 0j).cuda()
    for n in (1, 15, 18):
        out = {}
        for mfma in (1, 0):
            ctx.tune(gemm_mfma=mfma)
            try:
                out[mfma] = ctx.deflate_project_multi(
                    hdefl, Q, eta[:n].contiguous(),
                    [(lqcd.DEFL_HFES, None, None, None), (lqcd.DEFL_EIGPOLY, cp, base[:n].clone(), None),
                     (lqcd.DEFL_EIGPOLY, cp, None, None)], THETAS)
            finally:
                ctx.tune(gemm_mfma=1)
        for v in range(3):
            a, b = to_host(out[1][v][0]), to_host(out[0][v][0])
            assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max(), (n, v)
            np.testing.assert_array_equal(out[1][v][1], out[0][v][1])
        one = ctx.deflate_project(hdefl, Q, eta[:n].contiguous(), thetas=THETAS)
        np.testing.assert_array_equal(to_host(one[0]), to_host(out[1][0][0]))


@pytest.mark.parametrize("dims", [(10, 14, 14, 16), (10, 2, 4, 6)])
def test_trace_corrections_double_with_a_periodic_copy(dims):
    """Links repeated once along x: no loop of length <= 8 winds round an
    extent of 10 or 20, so every timeslice sum doubles.  The first lattice's
    timeslices (1960 and 3920 sites) are more chunks of sites than a launch
    has workgroups for and end in a ragged one; the second has windings in
    y, z and t, in both lattices alike.  Sums of 4e3 sites times 4e4 walks in
    two orders: 1e-12 of the largest is five digits above their rounding."""
    require_gpu()
    ctx, U = context(dims, 0.3, 29, 0.12)
    U2 = np.ascontiguousarray(np.concatenate([U, U], axis=3))
    from paper_1903_06986_amd import Context
    ctx2 = Context((2 * dims[0],) + tuple(dims[1:]), U2, 0.12)
    ops = tuple(range(9))
    say("trace corrections of a doubled lattice", dims)
    _, a = ctx.pert_subtract(7, ctx.empty(0), ops)
    _, b = ctx2.pert_subtract(7, ctx2.empty(0), ops)
    for op in ops:
        scale = max(np.abs(a[op]).max(), 1e-4 * np.abs(a).max())  # some rows cancel to nothing
        assert np.abs(b[op] - 2 * a[op]).max() <= 1e-12 * 2 * scale, op


@pytest.mark.parametrize("dims", [(4, 4, 2, 4), (2, 2, 2, 4), (2, 4, 2, 6)])
@pytest.mark.parametrize("links", ["perturbed", "float32"])
def test_trace_corrections_of_links_that_are_not_unitary(dims, links):
    """The corrections are the traces of the operator as its links are, also
    where U U^+ is not 1: links off by 5 %, and rounded to FP32 (a walk whose
    last step undoes its first keeps both links).  Dense traces, orders 6 and 7
    of PS and a polynomial, all nine operators, at 1e-10 as for unitary links;
    without those links' U U^+ the vector currents are off by 5 % and 1e-8."""
    require_gpu()
    from oracle import pointsplit as PSO
    from paper_1903_06986_amd import Context
    from synth import random_su3_links
    kappa = 0.12
    U = random_su3_links(dims, 0.3, 77)
    rng = np.random.default_rng(4)
    if links == "perturbed":
        U = U + 0.05 * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape))
    else:
        U = U.astype(np.complex64).astype(np.complex128)
    ctx = Context(dims, U, kappa)
    Pd = W.dense_P(U, dims)
    for order in (6, 7):
        c = rng.standard_normal(order + 1) + 1j * rng.standard_normal(order + 1)
        for coeffs in (S.pert_coeffs(order), c):
            say("trace corrections of non-unitary links", dims, links, order)
            _, corr, _, _ = ctx.poly_subtract(order, ctx.empty(0), coeffs=coeffs, thetas=range(9))
            A = S.poly_dense(Pd, kappa, coeffs)
            ref = np.concatenate([S.trace_correction_dense(A, dims, THETAS),
                                  np.stack([PSO.trace_ps_dense(U, kappa, dims, mu, A) for mu in range(4)])])
            for op in range(9):
                assert np.abs(corr[op] - ref[op]).max() < 1e-10 * np.abs(ref[1:]).max(), (order, op)


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 12, 16)])
def test_projections_of_several_columns_equal_single_ones(dims):
    """V^H X of 2 to 16 columns at once (matrix cores; 49 and more vectors of a
    large field in two halves for up to four columns) against one column at a
    time (dot passes over V), through the projection on 1 to 64 modes: the same
    sums in another order, 1e-12."""
    require_gpu()
    ctx, _ = context(dims, 0.25, 17, 0.12)
    eta = ctx.noise_z4(5, 0, 16)
    say("deflation modes", dims)
    _, hdefl, _ = ctx.gmresdr_solve(eta[:1].contiguous(), op="MG5", m=80, k=66, tol=0.3, tol_super=0.3,
                                    method="minres-dr")
    for Q in (1, 16, 17, 33, 48, 49, 56, 64):
        ones = [to_host(ctx.deflate_project(hdefl, Q, eta[r:r + 1].contiguous(), thetas=(0,))[0])[0] for r in range(16)]
        for n in (2, 4, 5, 16):
            say("columns at once", dims, Q, n)
            xt = to_host(ctx.deflate_project(hdefl, Q, eta[:n].contiguous(), thetas=(0,))[0])
            for r in range(n):
                assert np.abs(xt[r] - ones[r]).max() <= 1e-12 * np.abs(ones[r]).max(), (Q, n, r)

"""FP64 products on both tile sizes (32 x 32 and 64 x 64) and their Hermitian
form (unitarity of U_T, upper tiles only), at sizes on either side of the
choice between them, against plain FP64 matrix products.

Tolerances: a step's Chebyshev sum has L terms of products over n columns; in
FP64 with n <= 1100 their rounding stays below 1e-13 in a column's 2-norm.
"""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from workloads import gue

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


# padded size 64 .. 1152; 64 x 64 tiles make 1, 4, 9, 100, 256 (exactly one per
# CU) and 324 of them
@pytest.mark.parametrize("n", [64, 65, 192, 640, 1024, 1100])
def test_fp64_products_on_both_tiles(fl, n):
    print("[case] products", n, flush=True)
    rng = np.random.default_rng(90 + n)
    H0, V = gue(n, rng), gue(n, rng)
    T, M = 0.3, 3
    f = np.cos(fl.node_times(T, M))
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f)
    U = ctx.build_ut()
    rep = ctx.last_report
    cols = np.unique(np.array([0, 1, n // 2, n - 1]))
    X = np.eye(n, dtype=complex)[:, cols]
    a, b = orc.magnus4_weights(f, T / M)
    K = orc.commutator(H0, V)
    for k in range(M):
        H = H0 + a[k] * V + b[k] * K
        w, Q = np.linalg.eigh(H)
        X = Q @ (np.exp(-1j * (T / M) * w)[:, None] * (Q.conj().T @ X))
    err = orc.column_error(U.cpu().numpy()[:, cols], X)
    G = U.conj().T @ U - torch.eye(n, dtype=U.dtype, device=U.device)
    print("[case] e_col", err, "unitarity", rep["unitarity_max"], rep["unitarity_fro"], flush=True)
    # truncation 1e-12 a step beside rounding
    assert err < M * 1e-12 + 1e-13
    assert abs(rep["unitarity_max"] - G.abs().max().item()) < 1e-13
    assert abs(rep["unitarity_fro"] - torch.linalg.norm(G).item()) < 1e-13 * math.sqrt(n)


def _build_and_block(fl, n, M, L, T=1.2):
    """U_T by build_ut and by propagating the identity block, and the oracle's."""
    rng = np.random.default_rng(7 * n + L)
    H0, V = gue(n, rng), gue(n, rng)
    f = np.cos(fl.node_times(T, M))
    a, b = orc.magnus4_weights(f, T / M)
    lo, hi = orc.weyl_cover(H0, V, orc.commutator(H0, V), a, b)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f, e_min=lo, e_max=hi, L=L)
    U = ctx.build_ut().cpu().numpy()
    X = ctx.propagate(np.eye(n, dtype=complex)).cpu().numpy()
    ref = orc.build_ut(H0, V, f, T, M, route="cheb", e_min=lo, e_max=hi, L=L)
    return U, X, ref


# every block length and block count of the polynomial form (2 .. 20 terms in
# a build's segments, 2 .. 12 for a single step), the term-by-term form on
# either side of it, and a top block of one coefficient (L a multiple of s).
# All factors have norm at most 1 (|c_l| <= 1, |T_l| <= 1), so rounding is of
# the order of L M n eps < 1e-12 in the worst column.
@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 15, 16, 17, 20, 21])
def test_step_polynomials_of_every_order(fl, L):
    print("[case] polynomial order", L, flush=True)
    U, X, ref = _build_and_block(fl, 70, 5, L)
    eu, ex = orc.column_error(U, ref), orc.column_error(X, ref)
    print("[case] build", eu, "block", ex, flush=True)
    assert eu < 1e-12 and ex < 1e-12


# segments of unequal length (512 padded states run 8 segments), one segment
# per step and odd segment counts in the product of the segments
@pytest.mark.parametrize("n,M", [(500, 11), (500, 8), (130, 7), (130, 2), (130, 1), (50, 130),
                                 (50, 3)])
def test_segmented_builds(fl, n, M):
    print("[case] segments", n, M, flush=True)
    U, X, ref = _build_and_block(fl, n, M, 9, T=0.1 * M)
    eu, ex = orc.column_error(U, ref), orc.column_error(X, ref)
    print("[case] build", eu, "block", ex, flush=True)
    assert eu < 1e-12 and ex < 1e-12


# 1, 2, 4, 8 and 16 rows on the vector units, 32, 48 and 64 on the matrix cores
# in blocks of 16 and (2500 states) 32 rows, each with and without remainder,
# with fewer and more columns than the waves of a workgroup cover; 65 states
# take whole tiles, 50 the one-launch chain
@pytest.mark.parametrize("n,ncols", [(50, 3), (100, 1), (100, 16), (500, 2), (500, 17), (700, 4),
                                     (700, 33), (1100, 8), (1100, 9), (1100, 48), (1100, 49),
                                     (2000, 3), (2000, 64), (2000, 65), (2500, 48), (2500, 60)])
def test_few_states(fl, n, ncols):
    print("[case] few states", n, ncols, flush=True)
    rng = np.random.default_rng(n + ncols)
    H0, V = gue(n, rng), gue(n, rng)
    T, M = 0.4, 3
    f = np.cos(fl.node_times(T, M))
    X0 = rng.standard_normal((n, ncols)) + 1j * rng.standard_normal((n, ncols))
    X0 /= np.linalg.norm(X0, axis=0)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f)
    U = ctx.build_ut().cpu().numpy()
    for _ in range(2):
        X, snaps = ctx.propagate(X0, snap_every=2)
        err = orc.column_error(X.cpu().numpy(), U @ X0)
        print("[case] e_col", err, flush=True)
        # both carry at most the truncation of 1e-12 a step
        assert err < 2 * M * 1e-12
    assert snaps.shape == (1, n, ncols)
    fg = np.cos(np.arange(M) * T / M)
    e = ctx.period_average(X0, fg)
    a, b = orc.magnus4_weights(f, T / M)
    K = orc.commutator(H0, V)
    Y, ref = X0, 0.0
    for k in range(M):
        H = H0 + fg[k] * V
        ref = ref + np.real(np.sum(Y.conj() * (H @ Y), axis=0)) / np.linalg.norm(Y, axis=0) ** 2
        w, Q = np.linalg.eigh(H0 + a[k] * V + b[k] * K)
        Y = Q @ (np.exp(-1j * (T / M) * w)[:, None] * (Q.conj().T @ Y))
    assert np.max(np.abs(e - ref / M)) < 1e-11


# products that share their reduction between waves: blocks of 16 rows up to one
# per CU (128 rows at 512 padded states), of 32 rows up to one per CU (256 rows at
# 512), tiles beyond; conjugated, transposed and Hermitian operands through a
# whole block's step polynomials and the segments of a build (16 rows up to 256
# padded states, Hermitian up to 320, 32 rows up to 320); two members in a batch
@pytest.mark.parametrize("n,ncols", [(128, 128), (256, 65), (256, 256), (300, 300), (320, 320),
                                     (321, 321), (500, 128), (500, 129), (500, 250), (500, 300),
                                     (700, 100), (1000, 128), (1000, 129)])
def test_products_with_shared_reduction(fl, n, ncols):
    print("[case] shared reduction", n, ncols, flush=True)
    rng = np.random.default_rng(3 * n + ncols)
    H0, V = gue(n, rng), gue(n, rng)
    T, M = 0.4, 3
    f = np.cos(fl.node_times(T, M))
    X0 = rng.standard_normal((n, ncols)) + 1j * rng.standard_normal((n, ncols))
    X0 /= np.linalg.norm(X0, axis=0)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f)
    U = ctx.build_ut().cpu().numpy()
    X = ctx.propagate(X0).cpu().numpy()
    a, b = orc.magnus4_weights(f, T / M)
    K = orc.commutator(H0, V)
    R, Y = np.eye(n, dtype=complex), X0
    for k in range(M):
        w, Q = np.linalg.eigh(H0 + a[k] * V + b[k] * K)
        E = (Q * np.exp(-1j * (T / M) * w)) @ Q.conj().T
        R, Y = E @ R, E @ Y
    eu, ex = orc.column_error(U, R), orc.column_error(X, Y)
    print("[case] build", eu, "block", ex, flush=True)
    # truncation 1e-12 a step beside rounding
    assert eu < M * 1e-12 + 1e-13 and ex < M * 1e-12 + 1e-13


# the cover's Lanczos on the device: one, four and sixteen elements per thread
# (up to 256, 1024 and 4096 states) and vectors in memory beyond; fewer states
# than steps; one row per workgroup and blocks of four. With a zero drive the
# cover is H0's Ritz hull widened by 1 % of its spread, and 200 steps leave an
# extreme Ritz value less than 1 % of the spread inside the spectrum.
@pytest.mark.parametrize("n", [1, 2, 7, 200, 256, 257, 515, 1024, 1025, 4096, 4100])
def test_cover_of_a_known_spectrum(fl, n):
    print("[case] cover", n, flush=True)
    rng = np.random.default_rng(n)
    lam = np.sort(rng.uniform(-3.0, 5.0, n))
    # Householder reflection of diag(lam): dense, spectrum known
    v = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    v /= np.linalg.norm(v)
    lv = lam * v
    H0 = np.diag(lam).astype(complex) - 2.0 * np.outer(v, lv.conj()) - 2.0 * np.outer(lv, v.conj()) \
        + 4.0 * np.real(np.vdot(v, lv)) * np.outer(v, v.conj())
    H0 = 0.5 * (H0 + H0.conj().T)
    Hm = np.diag(rng.uniform(-1.0, 1.0, n)).astype(complex)
    ctx = fl.FloquetContext(h0=H0, hmod=Hm, T=0.1, M=1, f_nodes=np.zeros((1, 2)))
    rep = ctx.report
    w = lam[-1] - lam[0]
    print("[case] interval", rep["e_min"], rep["e_max"], "spectrum", lam[0], lam[-1], flush=True)
    slack = 1e-7 if w == 0.0 else 1e-12 * w
    assert lam[0] - 0.01 * w - slack <= rep["e_min"] <= lam[0] + slack
    assert lam[-1] - slack <= rep["e_max"] <= lam[-1] + 0.01 * w + slack
    # the same interval given by hand passes its check, one that cuts the spectrum fails
    kw = dict(h0=H0, hmod=Hm, T=0.1, M=1, f_nodes=np.zeros((1, 2)))
    fl.FloquetContext(e_min=rep["e_min"], e_max=rep["e_max"], **kw)
    if w > 0.0:
        from paper_1508_07621_amd._abi import FQ_ERR_SPECTRUM, FloquetError
        with pytest.raises(FloquetError) as e:
            fl.FloquetContext(e_min=lam[0] - 0.01 * w, e_max=lam[0] + 0.5 * w, **kw)
        assert e.value.status == FQ_ERR_SPECTRUM


# which precision a mixed context's calls run in, on both sides of every rule:
# FP64 up to 512 padded states and for few states, else the context's own
# products; FP32 also runs builds in FP64. Errors: truncation 1e-12 a step for
# FP64 runs, the library's bar of 1e-6 for the others.
@pytest.mark.parametrize("precision,n,ncols,f64", [
    ("bf16x3", 64, 0, True), ("bf16x3", 512, 0, True), ("bf16x3", 512, 200, True),
    ("bf16x3", 513, 0, False), ("bf16x3", 513, 65, False), ("bf16x3", 1100, 48, True),
    ("bf16x3", 1100, 64, False), ("bf16x3", 2000, 32, True), ("bf16x3", 2000, 33, False),
    ("fp32", 513, 0, True), ("fp32", 1100, 0, True), ("fp32", 1100, 1000, True),
    ("fp32", 1100, 192, True), ("fp32", 1100, 257, False), ("fp32", 2000, 128, True)])
def test_mixed_context_runs_in_fp64_where_faster(fl, precision, n, ncols, f64):
    print("[case] route", precision, n, ncols, flush=True)
    rng = np.random.default_rng(n + ncols)
    H0, V = gue(n, rng), gue(n, rng)
    T, M = 0.4, 2
    f = np.cos(fl.node_times(T, M))
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f, precision=precision)
    cols = np.arange(min(n, ncols)) if ncols else np.array([0, n // 2, n - 1])
    if ncols:
        X = ctx.propagate(np.eye(n, ncols, dtype=complex)).cpu().numpy()
    else:
        X = ctx.build_ut().cpu().numpy()[:, cols]
        rep = ctx.last_report
        assert all(t == 0 for t in rep["term_format"][:rep["L"]]) == f64
        assert (rep["mixed_err_est"] == 0.0) == f64
    a, b = orc.magnus4_weights(f, T / M)
    K = orc.commutator(H0, V)
    Y = np.eye(n, dtype=complex)[:, cols]
    for k in range(M):
        w, Q = np.linalg.eigh(H0 + a[k] * V + b[k] * K)
        Y = Q @ (np.exp(-1j * (T / M) * w)[:, None] * (Q.conj().T @ Y))
    err = orc.column_error(X, Y)
    print("[case] e_col", err, flush=True)
    if f64:
        assert err < M * 1e-12 + 1e-13
    else:
        assert err < 1e-6
        if precision == "bf16x3":   # not in FP64
            assert err > 1e-11


# propagations that form the propagators of a batch of steps at once: more steps
# than a batch holds (192 at 128 padded states, 30 at 320), remainders, one-launch
# chain sizes, snapshots between, both schemes with one and two exponentials a step,
# and energy averages; against U_T, against single steps (which go term by term), and
# against their energies. All carry the same truncation; rounding is below 1e-13 a step.
@pytest.mark.parametrize("n,ncols,M,scheme", [(30, 5, 9, "magnus4"), (64, 64, 2, "cf4"),
                                              (100, 3, 300, "magnus4"), (100, 100, 7, "magnus6"),
                                              (300, 9, 70, "cf4"), (300, 130, 31, "magnus4"),
                                              (500, 200, 9, "magnus4"), (900, 100, 5, "cf4")])
def test_batches_of_step_propagators(fl, n, ncols, M, scheme):
    print("[case] batches", n, ncols, M, scheme, flush=True)
    rng = np.random.default_rng(n + M)
    H0, V = gue(n, rng), gue(n, rng)
    T = 0.2 * M
    f = np.cos(fl.node_times(T, M, scheme))
    X0 = rng.standard_normal((n, ncols)) + 1j * rng.standard_normal((n, ncols))
    X0 /= np.linalg.norm(X0, axis=0)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f, scheme=scheme)
    U = ctx.build_ut().cpu().numpy()
    every = max(1, M // 3)
    X, snaps = ctx.propagate(X0, snap_every=every)
    tol = M * 2e-12
    assert orc.column_error(X.cpu().numpy(), U @ X0) < tol
    fg = np.cos(np.arange(M) * T / M)
    H0d, Vd = torch.from_numpy(H0).cuda(), torch.from_numpy(V).cuda()
    Y, ref = torch.from_numpy(X0).cuda(), 0.0
    for k in range(M):
        H = H0d + fg[k] * Vd
        ref = ref + torch.sum(Y.conj() * (H @ Y), dim=0).real / torch.sum(Y.abs() ** 2, dim=0)
        Y = ctx.propagate(Y, k, k + 1)
        if (k + 1) % every == 0:
            err = (snaps[(k + 1) // every - 1] - Y).abs().max().item()
            assert err < tol, (k, err)
    assert torch.linalg.vector_norm(X - Y, dim=0).max().item() < tol
    e = ctx.period_average(X0, fg)
    err = float(np.max(np.abs(np.asarray(e) - (ref / M).cpu().numpy())))
    print("[case] average", err, flush=True)
    assert err < 1e-11

"""Per-step setup of the tridiagonal layout on the GPU: the extreme eigenvalues
of every step's H_eff and the gauge factors, against the host bisection of the
same matrices and (through U_T) the oracle, at the edges of the kernels' chunks.

Tolerances: both searches end within a few spacings of doubles at the scale of
the spectrum; U_T against the oracle at the library's FP64 bar.
"""
import numpy as np
import pytest

import oracle as orc
from workloads import dimer_tridiag

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


def _problem(n, seed):
    rng = np.random.default_rng(seed)
    d = rng.standard_normal(n) * 3.0
    e = rng.standard_normal(max(n - 1, 0)) + 1j * rng.standard_normal(max(n - 1, 0))
    if n > 4:
        e[n // 2] = 0.0                 # a chain in two pieces
    v = rng.standard_normal(n)
    return d, e, v


# one row, a few, the ends of 64-lane and 256-thread runs, one LDS chunk of 2048
# rows and the next
@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 256, 257, 2047, 2048, 2049, 4100])
def test_extremes_of_every_step(fl, n):
    print("[case] extremes", n, flush=True)
    T, M = 0.7, 3
    d, e, v = _problem(n, 300 + n)
    f = np.random.default_rng(n).uniform(-2, 2, (M, 2))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f)
    a, b = orc.magnus4_weights(f, T / M)
    lo, hi = np.inf, -np.inf
    for k in range(M):
        ek = np.abs(e * (1.0 - 1j * b[k] * np.diff(v)))
        l, h = fl.tridiag_extremes(d + a[k] * v, ek)
        lo, hi = min(lo, l), max(hi, h)
    rep = ctx.report
    scale = max(abs(lo), abs(hi))
    if n == 1:  # a constant H widens its interval
        assert rep["e_min"] <= lo <= hi <= rep["e_max"]
        return
    print("[case]", rep["e_min"] - lo, rep["e_max"] - hi, flush=True)
    assert abs(rep["e_min"] - lo) < 1e-13 * scale and abs(rep["e_max"] - hi) < 1e-13 * scale


def test_vanishing_pivots(fl):
    """Zero diagonal: pivots that vanish exactly at the middle of the interval."""
    n, T, M = 201, 1.0, 2
    e = np.ones(n - 1)
    ctx = fl.FloquetContext(h0_diag=np.zeros(n), h0_off=e, hmod_diag=np.zeros(n), T=T, M=M,
                            f_nodes=np.zeros((M, 2)))
    x = 2.0 * np.cos(np.pi / (n + 1))
    rep = ctx.report
    assert abs(rep["e_min"] + x) < 1e-14 and abs(rep["e_max"] - x) < 1e-14


@pytest.mark.parametrize("n", [2, 130, 257, 700])
def test_complex_couplings_through_the_gauge(fl, n):
    """U_T for random complex couplings with b_k != 0: the gauge factors of
    every step against the oracle, which has no gauge."""
    print("[case] gauge", n, flush=True)
    T, M = 0.9, 6
    d, e, v = _problem(n, 500 + n)
    f = np.random.default_rng(n).uniform(-2, 2, (M, 2))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f)
    U = ctx.build_ut().cpu().numpy()
    rep = ctx.report
    ref = orc.build_ut_tridiag(d, e, v, f, T, M, route="cheb", e_min=rep["e_min"],
                               e_max=rep["e_max"], L=rep["L"])
    err = orc.column_error(U, ref)
    print("[case] e_col", err, flush=True)
    assert err < 1e-12


# ---- the chain kernel at every number of rows per lane --------------------------------------------

# 1, 2, 4, 8 and 16 rows per lane at their first and last sizes, two waves per part from
# 1025 rows on; M = 40 steps make short columns run in segments
@pytest.mark.parametrize("scheme", ["magnus4", "cf4"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025])
def test_chain_at_every_row_count(fl, n, scheme):
    print("[case] chain", n, scheme, flush=True)
    rng = np.random.default_rng(900 + n)
    if n <= 129:                        # complex couplings, b_k != 0
        d, e, v = _problem(n, 900 + n)
        T, M = 2.0, 40
    else:
        d, e, v = dimer_tridiag(n - 1, 1.0, 0.01)
        T, M = 0.05, 5
    f = rng.uniform(-1, 1, (M, 2))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f, scheme=scheme)
    U = ctx.build_ut().cpu().numpy()
    rep = ctx.last_report
    kw = dict(route="cheb", e_min=rep["e_min"], e_max=rep["e_max"], L=rep["L"], scheme=scheme)
    cols = np.unique([0, n // 3, n - 1])
    X0 = np.eye(n, dtype=complex)[:, cols]
    ref = orc.build_ut_tridiag(d, e, v, f, T, M, X0=X0, **kw)
    err = orc.column_error(U[:, cols], ref)
    print("[case] build", err, "unitarity", rep["unitarity_max"], flush=True)
    # every factor is bounded by 1: rounding of the order of L M eps
    assert err < 1e-11
    # a few states over a step range with snapshots, then the rest of the range
    X = rng.standard_normal((n, min(n, 3))) + 1j * rng.standard_normal((n, min(n, 3)))
    X /= np.linalg.norm(X, axis=0)
    Y, snaps = ctx.propagate(X, 0, 3, snap_every=2)
    Z = ctx.propagate(snaps[0].contiguous(), 2, M)
    assert orc.column_error(Z.cpu().numpy(), U @ X) < 1e-11
    assert orc.column_error(ctx.propagate(Y, 3, M).cpu().numpy(), U @ X) < 1e-11
    # energies along the way (relative to the spectrum's scale)
    fg = rng.uniform(-1, 1, M)
    got = ctx.period_average(X, fg)
    H0, V, _ = orc.tridiag_matrices(d, e, v)
    want, Xk = 0.0, X
    for k in range(M):
        E = np.real(np.sum(Xk.conj() * (H0 @ Xk + fg[k] * (V @ Xk)), axis=0))
        want = want + E / np.sum(np.abs(Xk) ** 2, axis=0) / M
        Xk = orc.build_ut_tridiag(d, e, v, f, T, M, X0=Xk, k_range=(k, k + 1), **kw)
    scale = max(abs(rep["e_min"]), abs(rep["e_max"]))
    print("[case] average", np.max(np.abs(got - want)) / scale, flush=True)
    assert np.max(np.abs(got - want)) < 1e-11 * scale


# streamed columns: windows of 8 and 16 rows per lane, one to several passes a step,
# against the same columns of a wider block (which takes other windows) and, for the
# norm, against 1. Rounding grows with the terms: 1e-12 holds 20000 terms' worth.
@pytest.mark.parametrize("n,M,T", [(4097, 6, 0.02), (4100, 3, 0.2), (4099, 2, 0.6), (9001, 2, 0.1)])
def test_streamed_windows(require_gpu, n, M, T):
    from paper_1508_07621_amd import floquet as fl
    print("[case] streamed windows", n, M, T, flush=True)
    i = np.arange(n, dtype=float)
    nb = n - 1
    d = 0.5 * 0.01 * (i * (i - 1.0) + (nb - i) * (nb - i - 1.0))
    e = -np.sqrt((i[:-1] + 1.0) * (nb - i[:-1])).astype(complex)
    f = 0.5 + np.cos(fl.node_times(T, M))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=2.0 * i - nb, T=T, M=M, f_nodes=f)
    rng = np.random.default_rng(n)
    X0 = rng.standard_normal((n, 700)) + 1j * rng.standard_normal((n, 700))
    X0 /= np.linalg.norm(X0, axis=0)
    print("[case] L", ctx.report["L"], flush=True)
    wide = ctx.propagate(X0).cpu().numpy()
    assert np.max(np.abs(np.linalg.norm(wide, axis=0) - 1.0)) < 1e-11
    for c in (1, 3, 40, 200):
        X = ctx.propagate(np.ascontiguousarray(X0[:, :c])).cpu().numpy()
        err = np.max(np.linalg.norm(X - wide[:, :c], axis=0))
        print("[case] columns", c, "difference", err, flush=True)
        assert err < 1e-12


# several waves per part: two with their last ghost group (2016 rows) and three (2017),
# four with the last (4000 rows), and the form without ghost lanes beyond
@pytest.mark.parametrize("scheme", ["magnus4", "cf4"])
@pytest.mark.parametrize("n", [2016, 2017, 4000, 4001])
def test_chain_of_several_waves(fl, n, scheme):
    test_chain_at_every_row_count(fl, n, scheme)

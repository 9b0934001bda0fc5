"""Resident tridiagonal columns where an order of events or a value is extreme:
period averages whose steps hold fewer terms than the waves' exchange interval,
couplings below the normal numbers, checked against the oracle.

Tolerances: the library's FP64 bar for U_T; energies relative to the spectrum's
scale, where a mixed-up row would show at the size of the commutator's share.
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


# several waves per part: two, three and four with ghost lanes, which exchange every 16
# terms, and the form with a barrier every term; b_k != 0 and at most 16 terms a step
@pytest.mark.parametrize("n", [1025, 2017, 4000, 4001])
def test_period_average_of_short_steps(fl, n):
    print("[case] short steps", n, flush=True)
    M, T = 12, 12 * 0.3 / n
    rng = np.random.default_rng(n)
    d, e, v = dimer_tridiag(n - 1, 1.0, 0.01)
    e = e * np.exp(1j * rng.uniform(0, 2 * np.pi, n - 1))
    h = T / M
    # node differences of the order 1 / h: b_k dv_i up to one, a_k small
    u = rng.uniform(0.5, 3.0, M) / h * rng.choice([-1.0, 1.0], M)
    f = np.stack([u, -u], axis=1) + rng.uniform(-0.1, 0.1, (M, 2))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f)
    rep = ctx.report
    assert 4 <= rep["L"] <= 16
    X = rng.standard_normal((n, 5)) + 1j * rng.standard_normal((n, 5))
    X /= np.linalg.norm(X, axis=0)
    fg = rng.uniform(-1, 1, M)
    kw = dict(route="cheb", e_min=rep["e_min"], e_max=rep["e_max"], L=rep["L"])
    want, Xk = 0.0, X
    for k in range(M):
        dk = (d + fg[k] * v)[:, None]
        y = dk * Xk
        y[:-1] += e[:, None] * Xk[1:]
        y[1:] += e.conj()[:, None] * Xk[:-1]
        want = want + np.real(np.sum(Xk.conj() * y, axis=0)) / np.sum(np.abs(Xk) ** 2, axis=0) / M
        Xk = orc.build_ut_tridiag(d, e, v, f, T, M, X0=Xk, k_range=(k, k + 1), **kw)
    scale = max(abs(rep["e_min"]), abs(rep["e_max"]))
    for _ in range(3):
        got = ctx.period_average(X, fg)
        err = np.max(np.abs(got - want)) / scale
        print("[case] L", rep["L"], "average", err, flush=True)
        assert err < 1e-12


# couplings among and next to the subnormal numbers (2.2e-308 down to 4.9e-324): they
# vanish in H_eff, and the gauge factors beyond them stay unit numbers
@pytest.mark.parametrize("tiny", [5e-324, 1e-310, 5.6e-309, 3e-308])
@pytest.mark.parametrize("n", [3, 70, 1100, 4100])
def test_subnormal_coupling(fl, n, tiny):
    print("[case] subnormal coupling", n, tiny, flush=True)
    rng = np.random.default_rng(n)
    M, T = 3, 0.3
    d, v = rng.standard_normal(n), rng.standard_normal(n)
    e = rng.standard_normal(n - 1) + 1j * rng.standard_normal(n - 1)
    e[n // 2 - 1] = tiny * (1.0 if n % 2 else 1.0j)
    f = rng.uniform(-2, 2, (M, 2))
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f)
    rep = ctx.report
    cols = np.unique([0, n // 2 - 1, n // 2, n - 1])
    X0 = np.eye(n, dtype=complex)[:, cols]
    got = ctx.propagate(X0).cpu().numpy()
    ref = orc.build_ut_tridiag(d, e, v, f, T, M, route="cheb", e_min=rep["e_min"],
                               e_max=rep["e_max"], L=rep["L"], X0=X0)
    err = orc.column_error(got, ref)
    print("[case] e_col", err, flush=True)
    assert err < 1e-12


def _chain_80bit(d, e, v, f, T, M, e_max, L, coef):
    """U_T of the same truncated series on [-e_max, e_max], in 80-bit arithmetic."""
    ld = np.longdouble
    n, h = len(d), T / M
    a, b = orc.magnus4_weights(f, h)
    X = np.eye(n, dtype=np.clongdouble)
    inv = ld(1.0 / e_max)
    dv = np.diff(v.astype(ld))
    for k in range(M):
        dd = ((d.astype(ld) + ld(a[k]) * v.astype(ld)) * inv)[:, None]
        up = (e.astype(np.clongdouble) * (1 - 1j * (ld(b[k]) * dv)) * inv)[:, None]

        def mv(x):
            y = dd * x
            y[:-1] += up * x[1:]
            y[1:] += up.conj() * x[:-1]
            return y
        p0, p1 = X, mv(X)
        Y = ld(coef[0]) * p0 + (-1j) * (ld(coef[1]) * p1)
        for l in range(2, L + 1):
            p0, p1 = p1, 2 * mv(p1) - p0
            Y = Y + np.array((-1j) ** l, dtype=np.clongdouble) * (ld(coef[l]) * p1)
        X = Y
    return X


# Random node differences in every step: correctly rounded gauge factors deviate from
# unit numbers independently of each other, so the error of U_T walks at random: a step's
# (four roundings of a rotation, about L / 2 of the sum) stays below 12 roundings of 53
# bits, and M steps below that times sqrt(M). A deviation common to all steps would grow
# with M. The interval is symmetric: the step phase is exactly 1.
@pytest.mark.parametrize("n", [3, 21, 90])
def test_gauge_factors_round_once(fl, n):
    print("[case] long chain", n, flush=True)
    rng = np.random.default_rng(40 + n)
    M = 1000
    T = 0.1 * M
    d, v = rng.standard_normal(n), rng.standard_normal(n)
    e = rng.standard_normal(n - 1) + 1j * rng.standard_normal(n - 1)
    f = rng.uniform(-2, 2, (M, 2))
    e_max = 16.0
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f, e_min=-e_max,
                            e_max=e_max)
    rep = ctx.report
    L = rep["L"]
    assert L < 24
    ref = _chain_80bit(d, e, v, f, T, M, e_max, L, fl.bessel_weights(T / M * e_max, L))
    U = ctx.build_ut().cpu().numpy()
    X = ctx.propagate(np.eye(n, dtype=complex)).cpu().numpy()
    bound = 12 * 2.0 ** -53 * np.sqrt(M)
    for name, A in (("build", U), ("states", X)):
        err = float(np.max(np.sqrt(np.sum(np.abs(A.astype(np.clongdouble) - ref) ** 2, axis=0))))
        print("[case]", name, "L", L, "e_col", err, "bound", bound, flush=True)
        assert err < bound


# Real couplings and a drive constant over each step: the device and the host bisection
# take the same pivots, operation by operation, and both end between neighbouring doubles
@pytest.mark.parametrize("scale", [1.0, 1e-100, 1e-145, 1e100])
@pytest.mark.parametrize("n", [2, 17, 300, 3000])
def test_extremes_as_the_host_finds_them(fl, n, scale):
    print("[case] extremes", n, scale, flush=True)
    rng = np.random.default_rng(60 + n)
    d, e = rng.standard_normal(n) * scale, rng.standard_normal(n - 1) * scale
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=np.zeros(n), T=0.01 / scale, M=1,
                            f_nodes=np.zeros((1, 2)))
    lo, hi = fl.tridiag_extremes(d, np.abs(e))
    rep = ctx.report
    print("[case]", (rep["e_min"] - lo) / np.spacing(abs(lo)),
          (rep["e_max"] - hi) / np.spacing(abs(hi)), flush=True)
    assert abs(rep["e_min"] - lo) <= np.spacing(abs(lo))
    assert abs(rep["e_max"] - hi) <= np.spacing(abs(hi))


# Commutator-free steps: the gauge stays, so that a step ends with the bare phase in every
# row and step. Rounded alike each time, that alone would put U_T off by up to one rounding per
# exponential, 1000 of them here; by turns it stays within one, and the rest walks as above
@pytest.mark.parametrize("n", [2, 4, 33])
def test_step_phase_rounds_by_turns(fl, n):
    print("[case] phase by turns", n, flush=True)
    rng = np.random.default_rng(70 + n)
    ld, M = np.longdouble, 500
    T = 0.2 * M
    d, v = rng.standard_normal(n), rng.standard_normal(n)
    e = rng.standard_normal(n - 1) + 1j * rng.standard_normal(n - 1)
    f = rng.uniform(-2, 2, (M, 2))
    lo, hi = -15.0, 16.4
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f, scheme="cf4",
                            e_min=lo, e_max=hi)
    L, beta, dE, h = ctx.report["L"], 0.5 * (hi + lo), 0.5 * (hi - lo), T / (2 * M)
    assert L < 24
    coef = fl.bessel_weights(h * dE, L)
    arg = ld(beta) * ld(h)
    phase = np.cos(arg) - 1j * np.sin(arg)
    p, q = 0.5 + 0.57735026918962576451, 0.5 - 0.57735026918962576451
    X = np.eye(n, dtype=np.clongdouble)
    inv = ld(1.0 / dE)
    up = (e.astype(np.clongdouble) * inv)[:, None]
    for f1, f2 in f:
        for a in (p * f1 + q * f2, q * f1 + p * f2):
            dd = ((d.astype(ld) + ld(a) * v.astype(ld) - ld(beta)) * inv)[:, None]

            def mv(x):
                y = dd * x
                y[:-1] += up * x[1:]
                y[1:] += up.conj() * x[:-1]
                return y
            p0, p1 = X, mv(X)
            Y = ld(coef[0]) * p0 + (-1j) * (ld(coef[1]) * p1)
            for l in range(2, L + 1):
                p0, p1 = p1, 2 * mv(p1) - p0
                Y = Y + np.array((-1j) ** l, dtype=np.clongdouble) * (ld(coef[l]) * p1)
            X = phase * Y
    bound = 12 * 2.0 ** -53 * np.sqrt(2 * M)
    for name, A in (("build", ctx.build_ut()), ("states", ctx.propagate(np.eye(n, dtype=complex)))):
        A = A.cpu().numpy().astype(np.clongdouble)
        err = float(np.max(np.sqrt(np.sum(np.abs(A - X) ** 2, axis=0))))
        print("[case]", name, "L", L, "e_col", err, "bound", bound, flush=True)
        assert err < bound

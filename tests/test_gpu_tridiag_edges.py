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

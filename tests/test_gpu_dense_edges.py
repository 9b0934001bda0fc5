"""Dense builds at the ends of what the library takes: results that are no numbers."""
import numpy as np
import pytest

from workloads import gue

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


# A caller's interval is checked at the steps with the smallest and the largest weight of
# Hmod; the step between them here has its spectrum far outside through the commutator, and
# T_300 overflows there: inf - inf leaves no number in U_T
@pytest.mark.parametrize("n", [5, 64, 150])
def test_unitarity_of_no_numbers_is_reported(fl, n):
    print("[case] no numbers", n, flush=True)
    rng = np.random.default_rng(n)
    f = np.array([[-1.0, -1.0], [2e4, -2e4], [1.0, 1.0]])
    ctx = fl.FloquetContext(h0=gue(n, rng), hmod=gue(n, rng), T=3.0, M=3, f_nodes=f, e_min=-20.0,
                            e_max=20.0, L=300)
    U = ctx.build_ut().cpu().numpy()
    rep = ctx.last_report
    print("[case] unitarity", rep["unitarity_max"], rep["unitarity_fro"], flush=True)
    assert np.isnan(U).any()
    assert rep["diverged"] == 1 and np.isnan(rep["unitarity_max"])


# Orders that no step polynomial serves (1, and beyond 36), and the least workspace with two
# steps between checkpoints: the reverse products of FP32 contexts run on FP32 matrix cores.
# Their operands are rounded to 24 bits and their sums over n products round in FP32: some
# sqrt(n L M) 2^-24 of the derivative, 1e-5 with an ample factor
@pytest.mark.parametrize("n,M,L,T,lean", [(70, 9, 1, 0.02, False), (70, 4, 37, 6.0, False),
                                          (300, 4, 37, 6.0, False), (70, 9, 8, 1.5, True),
                                          (300, 6, 9, 1.2, True)])
def test_fp32_gradient_term_by_term(fl, monkeypatch, n, M, L, T, lean):
    print("[case] fp32 reverse products", n, M, L, lean, flush=True)
    rng = np.random.default_rng(n + L)
    f = rng.uniform(-1, 1, (M, 2))
    kw = dict(h0=gue(n, rng), hmod=gue(n, rng), T=T, M=M, f_nodes=f, e_min=-6.0, e_max=6.0, L=L,
              checkpoint_every=2)
    W = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    exact = fl.FloquetContext(precision="fp64", **kw)
    exact.build_ut()
    g0 = exact.grad(W)
    if lean:
        monkeypatch.setattr(fl, "_free_bytes", lambda device: 0)
        monkeypatch.setattr(fl, "_UNASKED_SCRATCH", 0)
    ctx = fl.FloquetContext(precision="fp32", profile=True, **kw)
    ctx.build_ut()
    g = ctx.grad(W)
    rep = ctx.report
    err = np.max(np.abs(g - g0)) / np.max(np.abs(g0))
    print("[case] rel err", err, "reverse launches", rep["n_kernel"][7], flush=True)
    assert rep["n_kernel"][7] == M * L      # one reverse product per term and step
    assert 0.0 < err < 1e-5

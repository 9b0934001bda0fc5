"""Split-BF16 builds by step polynomials: how far they are from the FP64 build, against the
estimate that their formats were chosen for."""
import math

import numpy as np
import pytest

from workloads import gue

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


def _build(fl, n, M, omega, tol):
    import torch
    rng = np.random.default_rng(n + M)
    T = 2.0 * math.pi / omega
    kw = dict(h0=gue(n, rng), hmod=gue(n, rng), T=T, M=M,
              f_nodes=np.cos(omega * fl.node_times(T, M)))
    exact = fl.FloquetContext(precision="fp64", **kw).build_ut()
    ctx = fl.FloquetContext(precision="bf16x3", mixed_tol=tol, **kw)
    terms = ctx.report["mixed_err_est"]  # of the schedule of terms, before a build
    U = ctx.build_ut()
    rep = ctx.last_report
    err = torch.linalg.vector_norm(U - exact, dim=0).max().item()
    print("[case] L", rep["L"], "e_col", err, "estimates", terms, rep["mixed_err_est"],
          "formats", rep["term_format"][:8], flush=True)
    return err, terms, rep["mixed_err_est"]


# steps of small R, whose terms stay well below the target: a polynomial is taken only at
# an estimate no larger than theirs, and stays below that estimate
@pytest.mark.parametrize("tol", [0.0, 1e-6])
@pytest.mark.parametrize("n,M,omega", [(520, 200, 1.0), (1030, 200, 1.0), (1500, 100, 1.0)])
def test_polynomial_no_further_off_than_the_terms(fl, n, M, omega, tol):
    print("[case] split-BF16 estimate", n, M, omega, tol, flush=True)
    err, terms, est = _build(fl, n, M, omega, tol)
    assert est <= terms * (1 + 1e-12)
    assert err < terms


# Few long steps: the product with X, three pieces and FP32 sums, carries the whole error.
# The estimate's constant was fitted to sums of Ar B and Ai B apart; in one running sum each
# element rounds on partial sums sqrt(2) larger on average, and comes to the estimate
@pytest.mark.parametrize("n", [1030, 1500, 1984])
def test_three_piece_products_sum_parts_apart(fl, n):
    print("[case] split-BF16 three pieces", n, flush=True)
    err, terms, est = _build(fl, n, 20, 10.0, 0.0)
    assert err < 0.85 * est


# Hermitian products on both sides of their tile choice: the largest states on 64 x 64 tiles
# (padded to 4480) and the first on 128 x 128 (4608), below the estimate
@pytest.mark.parametrize("n", [4225, 4480, 4481])
def test_hermitian_products_on_either_tile(fl, n):
    print("[case] split-BF16 tiles", n, flush=True)
    err, terms, est = _build(fl, n, 3, 20.0, 0.0)
    assert err < est <= terms * (1 + 1e-12)

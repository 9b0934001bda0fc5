"""Adjoint gradient (floquet_grad) against the oracle and finite differences."""
import math

import numpy as np
import pytest

import oracle as orc
from workloads import dimer_tridiag, drive_cos, gue, haar_unitary, workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)
    return floquet


def _say(*a):
    print("[case]", *a, flush=True)


def _trace_loss_and_bar(U, W):
    """loss = 1 - |Tr(W^dagger U)|^2 / N^2 and Ubar = dL/dRe U + i dL/dIm U."""
    n = U.shape[0]
    tau = np.vdot(W, U)
    return 1.0 - abs(tau) ** 2 / n ** 2, -(2.0 / n ** 2) * tau * W


def _problem(n, M, seed):
    rng = np.random.default_rng(seed)
    H0, V = gue(n, rng), gue(n, rng)
    f = rng.uniform(-1, 1, M)
    W = haar_unitary(n, rng)
    return H0, V, f, W


@pytest.mark.parametrize("n,M,ckpt,precision,tol", [(48, 24, 5, "fp64", 1e-9), (64, 20, 16, "fp64", 1e-9),
                                                    (130, 12, 4, "fp64", 1e-9), (64, 20, 8, "fp32", 1e-5),
                                                    (64, 20, 8, "bf16x3", 1e-5)])
def test_piecewise_gradient_matches_oracle(fl, n, M, ckpt, precision, tol):
    """Piecewise-constant drive: the oracle's exact (Daleckii-Krein) derivative
    of the Chebyshev chain with the same interval and order."""
    _say("grad piecewise", n, M, ckpt, precision)
    H0, V, f, W = _problem(n, M, 40 + n)
    T = 2.0
    lo, hi = orc.weyl_cover(H0, V, np.zeros_like(H0), f, np.zeros(M))
    L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-13)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=np.stack([f, f], 1), e_min=lo,
                            e_max=hi, L=L, precision=precision, checkpoint_every=ckpt)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar)
    g_f = g.sum(axis=1)
    ref = orc.grad_piecewise(H0, V, f, T, W, route="cheb", e_min=lo, e_max=hi, L=L)
    err = np.max(np.abs(g_f - ref)) / np.max(np.abs(ref))
    _say("rel err", err, "max|g|", np.max(np.abs(ref)))
    assert err < tol


def test_smooth_drive_gradient_matches_oracle_differences(fl):
    """Smooth drive (b_k != 0 exercises the commutator contraction): every
    node derivative against central differences of the oracle."""
    n, M = 24, 8
    rng = np.random.default_rng(77)
    H0, V = gue(n, rng), gue(n, rng)
    W = haar_unitary(n, rng)
    T = 2 * math.pi
    f = drive_cos(orc.node_times(T, M), 0.2, 1.1, 1.0)
    lo, hi = -5.0, 5.0
    L = 30
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=f, e_min=lo, e_max=hi, L=L,
                            checkpoint_every=3)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar)

    def loss(ff):
        Uo = orc.build_ut(H0, V, ff, T, M, route="cheb", e_min=lo, e_max=hi, L=L)
        return _trace_loss_and_bar(Uo, W)[0]

    eps = 1e-5
    fd = np.zeros_like(f)
    for k in range(M):
        for i in range(2):
            fp, fm = f.copy(), f.copy()
            fp[k, i] += eps
            fm[k, i] -= eps
            fd[k, i] = (loss(fp) - loss(fm)) / (2 * eps)
    err = np.max(np.abs(g - fd)) / np.max(np.abs(fd))
    _say("smooth rel err", err)
    assert err < 1e-6
    assert np.max(np.abs(g[:, 0] - g[:, 1])) > 1e-6 * np.max(np.abs(g))  # nodes differ


@pytest.mark.parametrize("layout", ["dense", "tridiag"])
def test_constant_drive_node_derivatives(fl, layout):
    """A drive constant over every step (b_k = 0 throughout): each node's own
    derivative still has the commutator part (moving one node makes b_k
    nonzero), against central differences of the oracle node by node; with
    grad_pair_sums only the node sums are kept, as equal halves."""
    M = 6
    rng = np.random.default_rng(91)
    T = 2.0
    f = rng.uniform(-1, 1, M)
    nodes = np.stack([f, f], 1)
    if layout == "dense":
        n = 20
        H0, V = gue(n, rng), gue(n, rng)
        sysk = dict(h0=H0, hmod=V)
        lo, hi, L = -8.0, 8.0, 40

        def build(ff):
            return orc.build_ut(H0, V, ff, T, M, route="cheb", e_min=lo, e_max=hi, L=L)
    else:
        d, e, v = dimer_tridiag(19, 1.0, 0.3)
        n = 20
        sysk = dict(h0_diag=d, h0_off=e, hmod_diag=v)
        a, b = orc.magnus4_weights(nodes, T / M)
        lo, hi = orc.tridiag_cover(d, e, v, a, b)
        lo, hi = lo - 1.0, hi + 1.0
        L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-14)

        def build(ff):
            return orc.build_ut_tridiag(d, e, v, ff, T, M, route="cheb", e_min=lo, e_max=hi, L=L)
    W = haar_unitary(n, rng)
    kw = dict(T=T, M=M, f_nodes=nodes, e_min=lo, e_max=hi, L=L, checkpoint_every=2, **sysk)
    ctx = fl.FloquetContext(**kw)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar)
    eps = 1e-5
    fd = np.zeros_like(nodes)
    for k in range(M):
        for i in range(2):
            fp, fm = nodes.copy(), nodes.copy()
            fp[k, i] += eps
            fm[k, i] -= eps
            fd[k, i] = (_trace_loss_and_bar(build(fp), W)[0] -
                        _trace_loss_and_bar(build(fm), W)[0]) / (2 * eps)
    err = np.max(np.abs(g - fd)) / np.max(np.abs(fd))
    _say(layout, "constant-drive node derivatives rel err", err)
    assert err < 1e-6
    assert np.max(np.abs(g[:, 0] - g[:, 1])) > 1e-4 * np.max(np.abs(g))  # the K part is there
    cp = fl.FloquetContext(grad_pair_sums=True, **kw)
    cp.build_ut()
    gp = cp.grad(Ubar)
    assert np.array_equal(gp[:, 0], gp[:, 1])
    err = np.max(np.abs(gp.sum(axis=1) - g.sum(axis=1))) / np.max(np.abs(g.sum(axis=1)))
    _say(layout, "pair sums rel diff", err)
    assert err < 1e-10


@pytest.mark.parametrize("where", ["cpu", "cuda"])
def test_autograd_function(fl, where):
    """The gradient comes back on the device (and in the dtype) of f_nodes."""
    import torch
    n, M = 40, 10
    H0, V, f, W = _problem(n, M, 5)
    T = 1.5
    lo, hi = -5.0, 5.0
    fn = torch.tensor(np.stack([f, f], 1), dtype=torch.float64, device=where, requires_grad=True)
    U = fl.FloquetUT.apply(fn, h0=H0, hmod=V, T=T, M=M, e_min=lo, e_max=hi, tol=1e-13,
                           checkpoint_every=4)
    Wt = torch.from_numpy(W).to(U.device)
    loss = 1.0 - torch.abs(torch.sum(torch.conj(Wt) * U)) ** 2 / n ** 2
    loss.backward()
    assert fn.grad.device == fn.device and fn.grad.dtype == fn.dtype
    g = fn.grad.cpu().numpy().sum(axis=1)
    ref = orc.grad_piecewise(H0, V, f, T, W, route="cheb", e_min=lo, e_max=hi, tol=1e-13)
    assert np.max(np.abs(g - ref)) / np.max(np.abs(ref)) < 1e-8


def test_grad_error_paths(fl):
    from paper_1508_07621_amd._abi import FQ_ERR_STATE, FloquetError
    n, M = 32, 4
    H0, V, f, W = _problem(n, M, 6)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=1.0, M=M, f_nodes=np.stack([f, f], 1), e_min=-5,
                            e_max=5)
    with pytest.raises(FloquetError) as e:
        ctx.grad(np.zeros((n, n), complex))
    assert e.value.status == FQ_ERR_STATE
    ctx2 = fl.FloquetContext(h0=H0, hmod=V, T=1.0, M=M, f_nodes=np.stack([f, f], 1), e_min=-5,
                             e_max=5, checkpoint_every=2)
    with pytest.raises(FloquetError) as e:
        ctx2.grad(np.zeros((n, n), complex))   # no build yet
    assert e.value.status == FQ_ERR_STATE


def test_adjoint_config_full_size_against_fd(fl):
    """The 1024-state adjoint workload: complex64 forward (FP32 products,
    complex64 U_T and U_bar), checkpoint every 16 steps, against central
    differences (h = 1e-4) of the FP64 forward on 8 seeded amplitudes."""
    wl = workload("adjoint1024")
    H0, V, W, f = wl.arrays["h0"], wl.arrays["v"], wl.arrays["w"], wl.amplitudes
    T, M, n = wl.T, wl.M, wl.n
    lo, hi = orc.weyl_cover(np.diag(np.linalg.eigvalsh(H0)), np.diag(np.linalg.eigvalsh(V)),
                            np.zeros((1, 1)), f, np.zeros(M))
    _say("adjoint1024", n, M, lo, hi)
    nodes = np.stack([f, f], 1)
    ctx = fl.FloquetContext(h0=H0, hmod=V, T=T, M=M, f_nodes=nodes, e_min=lo, e_max=hi, tol=1e-12,
                            precision="fp32", checkpoint_every=16, dtype="complex64")
    U = ctx.build_ut().cpu().numpy().astype(complex)
    L = ctx.report["L"]
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar).sum(axis=1)
    ref_ctx_kw = dict(h0=H0, hmod=V, T=T, M=M, e_min=lo, e_max=hi, L=L)
    rng = np.random.default_rng(1508 + 30)
    ks = rng.choice(M, size=8, replace=False)
    eps = 1e-4
    for k in ks:
        vals = []
        for sgn in (+1, -1):
            ff = f.copy()
            ff[k] += sgn * eps
            Uf = fl.FloquetContext(f_nodes=np.stack([ff, ff], 1), **ref_ctx_kw).build_ut().cpu().numpy()
            vals.append(_trace_loss_and_bar(Uf, W)[0])
        fd = (vals[0] - vals[1]) / (2 * eps)
        _say("k", k, "adjoint", g[k], "fd", fd)
        assert abs(g[k] - fd) <= 1e-3 * abs(fd) + 1e-9


# ---- tridiagonal (dimer) gradient ---------------------------------------------------------------

def _dimer_problem(nb, M, seed, U_int=0.01):
    d, e, v = dimer_tridiag(nb, 1.0, U_int)
    rng = np.random.default_rng(seed)
    f = rng.uniform(-1, 1, M)
    W = haar_unitary(nb + 1, rng)
    return d, e, v, f, W


@pytest.mark.parametrize("nb,M,ckpt", [(39, 24, 5), (199, 16, 16), (700, 12, 4), (1499, 6, 2)])
def test_tridiag_piecewise_gradient_matches_oracle(fl, nb, M, ckpt):
    """Piecewise-constant drive on the dimer: the per-column reverse sweep
    against the oracle's exact derivative of the same Chebyshev chain (dense
    copies of the tridiagonal operators)."""
    _say("tridiag grad piecewise", nb + 1, M, ckpt)
    d, e, v, f, W = _dimer_problem(nb, M, 90 + nb)
    T = 2.0
    nodes = np.stack([f, f], 1)
    a, b = orc.magnus4_weights(nodes, T / M)
    lo, hi = orc.tridiag_cover(d, e, v, a, b)
    L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-13)
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=nodes, e_min=lo,
                            e_max=hi, L=L, checkpoint_every=ckpt)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar)
    H0s, Vs, _ = orc.tridiag_matrices(d, e, v)
    ref = orc.grad_piecewise(H0s.toarray(), Vs.toarray(), f, T, W, route="cheb", e_min=lo, e_max=hi,
                             L=L)
    err = np.max(np.abs(g.sum(axis=1) - ref)) / np.max(np.abs(ref))
    _say("rel err", err, "L", L, "max|g|", np.max(np.abs(ref)))
    assert err < 1e-9
    # b_k = 0, but each node's own derivative keeps its commutator part
    assert np.max(np.abs(g[:, 0] - g[:, 1])) > 1e-6 * np.max(np.abs(g))


def test_tridiag_smooth_drive_gradient_matches_oracle_differences(fl):
    """Smooth drive on an interacting dimer (b_k != 0: the K contraction):
    every node derivative against central differences of the oracle."""
    nb, M = 23, 8
    d, e, v = dimer_tridiag(nb, 1.0, 0.3)
    W = haar_unitary(nb + 1, np.random.default_rng(78))
    T = 2 * math.pi
    f = drive_cos(orc.node_times(T, M), 0.5, 1.5, 1.0)
    a, b = orc.magnus4_weights(f, T / M)
    lo, hi = orc.tridiag_cover(d, e, v, a, b)
    lo, hi = lo - 1.0, hi + 1.0   # room for the perturbed drives
    L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-14)
    ctx = fl.FloquetContext(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=f, e_min=lo,
                            e_max=hi, L=L, checkpoint_every=3)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar)

    def loss(ff):
        Uo = orc.build_ut_tridiag(d, e, v, ff, T, M, route="cheb", e_min=lo, e_max=hi, L=L)
        return _trace_loss_and_bar(Uo, W)[0]

    eps = 1e-5
    fd = np.zeros_like(f)
    for k in range(M):
        for i in range(2):
            fp, fm = f.copy(), f.copy()
            fp[k, i] += eps
            fm[k, i] -= eps
            fd[k, i] = (loss(fp) - loss(fm)) / (2 * eps)
    err = np.max(np.abs(g - fd)) / np.max(np.abs(fd))
    _say("tridiag smooth rel err", err)
    assert err < 1e-6
    assert np.max(np.abs(g[:, 0] - g[:, 1])) > 1e-6 * np.max(np.abs(g))


def test_tridiag_dimer1000_256_amplitudes_against_fd(fl):
    """The 999-boson dimer with 256 piecewise-constant amplitudes (checkpoint
    every 16 steps): the adjoint against central differences (h = 1e-4) of the
    library's own FP64 build on 8 seeded amplitudes."""
    nb, M = 999, 256
    d, e, v, f, W = _dimer_problem(nb, M, 1508 + 50)
    T = 2 * math.pi
    nodes = np.stack([f, f], 1)
    a, b = orc.magnus4_weights(nodes, T / M)
    lo, hi = orc.tridiag_cover(d, e, v, a, b)
    lo, hi = lo - 10.0, hi + 10.0
    L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-13)
    kw = dict(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, e_min=lo, e_max=hi, L=L)
    ctx = fl.FloquetContext(f_nodes=nodes, checkpoint_every=16, **kw)
    U = ctx.build_ut().cpu().numpy()
    _, Ubar = _trace_loss_and_bar(U, W)
    g = ctx.grad(Ubar).sum(axis=1)
    _say("dimer1000 grad L", L, "max|g|", np.max(np.abs(g)))
    ks = np.random.default_rng(1508 + 51).choice(M, size=8, replace=False)
    eps = 1e-4
    for k in ks:
        vals = []
        for sgn in (+1, -1):
            ff = f.copy()
            ff[k] += sgn * eps
            Uf = fl.FloquetContext(f_nodes=np.stack([ff, ff], 1), **kw).build_ut().cpu().numpy()
            vals.append(_trace_loss_and_bar(Uf, W)[0])
        fd = (vals[0] - vals[1]) / (2 * eps)
        _say("k", k, "adjoint", g[k], "fd", fd)
        assert abs(g[k] - fd) <= 1e-5 * abs(fd) + 1e-9


def test_tridiag_gradient_complex64_ubar(fl):
    """The tridiagonal reverse sweep reads a complex64 U_bar when the context
    stores its state blocks in complex64."""
    d, e, v, f, W = _dimer_problem(60, 10, 321)
    T = 2.0
    nodes = np.stack([f, f], 1)
    a, b = orc.magnus4_weights(nodes, T / 10)
    lo, hi = orc.tridiag_cover(d, e, v, a, b)
    L = orc.choose_L(orc.rescale(lo, hi, T / 10)[2], 1e-13)
    kw = dict(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=10, f_nodes=nodes, e_min=lo, e_max=hi, L=L,
              checkpoint_every=3)
    c128 = fl.FloquetContext(**kw)
    c64 = fl.FloquetContext(dtype="complex64", **kw)
    U = c128.build_ut().cpu().numpy()
    c64.build_ut()
    _, Ubar = _trace_loss_and_bar(U, W)
    g1 = c128.grad(Ubar)
    g2 = c64.grad(Ubar.astype(np.complex64))
    err = np.max(np.abs(g1 - g2)) / np.max(np.abs(g1))
    _say("c64 ubar rel", err)
    assert err < 1e-5


# ---- streamed reverse sweep (columns longer than one workgroup holds) --------------------------

def _dimer_kw(d, e, v, nodes, T, M, margin):
    a, b = orc.magnus4_weights(nodes, T / M)
    lo, hi = orc.tridiag_cover(d, e, v, a, b)
    lo, hi = lo - margin, hi + margin
    L = orc.choose_L(orc.rescale(lo, hi, T / M)[2], 1e-13)
    return dict(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, e_min=lo, e_max=hi, L=L)


@pytest.mark.parametrize("nb,M,ckpt,smooth,dtype,pair", [(299, 10, 3, False, "complex128", False),
                                                         (299, 10, 3, False, "complex128", True),
                                                         (299, 8, 3, True, "complex128", False),
                                                         (299, 8, 3, True, "complex128", True),
                                                         (1999, 6, 4, False, "complex128", True),
                                                         (1999, 6, 4, True, "complex128", False),
                                                         (299, 7, 2, False, "complex64", False),
                                                         (779, 5, 5, False, "complex128", True),
                                                         (15, 4, 2, True, "complex128", False)])
def test_tridiag_streamed_sweep_matches_per_column_sweep(fl, monkeypatch, nb, M, ckpt, smooth,
                                                         dtype, pair):
    """The streamed reverse sweep (selected for n <= 2048 by the environment
    switch) against the per-column sweep on the same problem: one block per
    column (n = 16, 300, 780 with a column end inside the last lane group)
    and three (n = 2000, blocks of 768 owned rows), with the K contraction
    (the default) and without it (node-pair sums), for piecewise-constant and
    smooth drives, one checkpoint segment and several, and with complex64
    state blocks (U_bar read as complex64)."""
    _say("streamed vs per-column sweep", nb + 1, M, ckpt, smooth, dtype, "pair sums", pair)
    rng = np.random.default_rng(400 + nb)
    if smooth:
        d, e, v = dimer_tridiag(nb, 1.0, 0.3)
        T = 2.0
        nodes = drive_cos(orc.node_times(T, M), 0.5, 1.5, 1.0)
    else:
        d, e, v = dimer_tridiag(nb, 1.0, 0.01)
        T = 2.0
        f = rng.uniform(-1, 1, M)
        nodes = np.stack([f, f], 1)
    kw = _dimer_kw(d, e, v, nodes, T, M, 0.0)
    W = haar_unitary(nb + 1, rng)
    per_col = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, dtype=dtype,
                                grad_pair_sums=pair, **kw)
    monkeypatch.setenv("FQ_TRIDIAG_STREAMED_ADJOINT", "1")
    streamed = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, dtype=dtype,
                                 grad_pair_sums=pair, **kw)
    monkeypatch.delenv("FQ_TRIDIAG_STREAMED_ADJOINT")
    U = per_col.build_ut().cpu().numpy()
    streamed.build_ut()
    _, Ubar = _trace_loss_and_bar(U.astype(np.complex128), W)
    Ubar = Ubar.astype(U.dtype)
    g1 = per_col.grad(Ubar)
    g2 = streamed.grad(Ubar)
    err = np.max(np.abs(g1 - g2)) / np.max(np.abs(g1))
    _say("L", kw["L"], "max|g|", np.max(np.abs(g1)), "rel diff", err)
    assert err < 1e-10
    if not pair:
        assert np.max(np.abs(g2[:, 0] - g2[:, 1])) > 1e-6 * np.max(np.abs(g2))


@pytest.mark.parametrize("pair", [True, False])
def test_tridiag_streamed_sweep_short_expansion(fl, monkeypatch, pair):
    """A deliberately short expansion (L from a 1e-4 truncation tolerance, so the
    last weight |c_L| is near 1e-5 instead of 1e-13): the reverse sweep starts
    from Pbar_L = conj(c_L) Lambda, in the streamed passes as in the per-column
    sweep, so the two agree to rounding; a first pass that dropped or misread
    c_L would differ at about |c_L| relative."""
    nb, M, ckpt = 299, 4, 2
    _say("streamed vs per-column sweep, short expansion, pair sums", pair)
    rng = np.random.default_rng(4242)
    d, e, v = dimer_tridiag(nb, 1.0, 0.01)
    T = 2.0
    f = rng.uniform(-1, 1, M)
    nodes = np.stack([f, f], 1)
    kw = _dimer_kw(d, e, v, nodes, T, M, 0.0)
    R = orc.rescale(kw["e_min"], kw["e_max"], T / M)[2]
    kw["L"] = orc.choose_L(R, 1e-4)
    cL = abs(orc.bessel_coefficients(R, kw["L"])[-1])
    assert cL > 1e-8
    W = haar_unitary(nb + 1, rng)
    per_col = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, grad_pair_sums=pair, **kw)
    monkeypatch.setenv("FQ_TRIDIAG_STREAMED_ADJOINT", "1")
    streamed = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, grad_pair_sums=pair, **kw)
    monkeypatch.delenv("FQ_TRIDIAG_STREAMED_ADJOINT")
    U = per_col.build_ut().cpu().numpy()
    streamed.build_ut()
    _, Ubar = _trace_loss_and_bar(U, W)
    g1 = per_col.grad(Ubar)
    g2 = streamed.grad(Ubar)
    err = np.max(np.abs(g1 - g2)) / np.max(np.abs(g1))
    _say("L", kw["L"], "R", R, "|c_L|", cL, "rel diff", err)
    assert err < 1e-10


@pytest.mark.parametrize("nb,M,ckpt,pair", [(2499, 6, 2, True), (4499, 6, 2, False)])
def test_tridiag_long_column_gradient_against_fd(fl, nb, M, ckpt, pair):
    """Columns beyond the per-column sweep (n > 2048; for n > 4096 the forward
    build streams too and records its checkpoints through the snapshot store):
    the streamed reverse sweep against central differences (h = 1e-5) of the
    library's own builds on three amplitudes. Loss 1 - |Tr(W^dagger U)|^2/N^2
    with the target W = U_T of a slightly perturbed drive, so that the loss is
    well below one. A unit of drive turns the phases by up to h_t |V| ~ 20 rad
    here (|V| ~ N), which sets the difference step."""
    import torch
    T = 0.05
    d, e, v = dimer_tridiag(nb, 1.0, 0.01)
    n = nb + 1
    rng = np.random.default_rng(500 + nb)
    f = rng.uniform(-1, 1, M)
    fw = f + 0.02 * rng.uniform(-1, 1, M)
    kw = _dimer_kw(d, e, v, np.stack([f, f], 1), T, M, 10.0)
    _say("long-column gradient", n, "M", M, "L", kw["L"])
    sys_kw = {k: kw[k] for k in ("h0_diag", "h0_off", "hmod_diag", "T", "M")}
    W = fl.FloquetContext(f_nodes=np.stack([fw, fw], 1), **sys_kw).build_ut()
    ctx = fl.FloquetContext(f_nodes=np.stack([f, f], 1), checkpoint_every=ckpt,
                            grad_pair_sums=pair, **kw)
    U = ctx.build_ut()

    def loss_of(Ut):
        tau = torch.sum(torch.conj(W) * Ut).item()
        return 1.0 - abs(tau) ** 2 / n ** 2, tau

    loss, tau = loss_of(U)
    ubar = (-2.0 / n ** 2) * tau * W
    g = ctx.grad(ubar).sum(axis=1)
    _say("loss", loss, "max|g|", np.max(np.abs(g)))
    eps = 1e-5
    for k in (0, M // 2, M - 1):
        vals = []
        for sgn in (+1, -1):
            ff = f.copy()
            ff[k] += sgn * eps
            c = fl.FloquetContext(f_nodes=np.stack([ff, ff], 1), **kw)
            vals.append(loss_of(c.build_ut())[0])
            del c
        fd = (vals[0] - vals[1]) / (2 * eps)
        _say("k", k, "adjoint", g[k], "fd", fd)
        assert abs(g[k] - fd) <= 1e-5 * abs(fd) + 1e-9


def test_tridiag_long_column_complex64_tape(fl):
    """n > 4096 with complex64 state blocks: the streamed build records its
    checkpoints in complex64 (entries of half the size), which the reverse
    sweep reads back for every segment; against the complex128 gradient."""
    import torch
    nb, M, ckpt = 4199, 6, 2
    d, e, v = dimer_tridiag(nb, 1.0, 0.01)
    n = nb + 1
    rng = np.random.default_rng(600)
    f = rng.uniform(-1, 1, M)
    kw = _dimer_kw(d, e, v, np.stack([f, f], 1), 0.05, M, 10.0)
    W = torch.from_numpy(haar_unitary(n, rng)).to("cuda")
    gs = []
    for dtype in ("complex128", "complex64"):
        _say("long-column tape", n, dtype)
        ctx = fl.FloquetContext(f_nodes=np.stack([f, f], 1), checkpoint_every=ckpt, dtype=dtype,
                                **kw)
        U = ctx.build_ut()
        Wd = W.to(U.dtype)
        tau = torch.sum(torch.conj(Wd) * U)
        gs.append(ctx.grad((-2.0 / n ** 2) * tau * Wd))
        del ctx, U
    err = np.max(np.abs(gs[0] - gs[1])) / np.max(np.abs(gs[0]))
    _say("complex64 tape rel diff", err)
    assert err < 1e-5


# ---- dense sweep through the step polynomials ----------------------------------------------------

@pytest.mark.parametrize("n,M,ckpt,L,T", [
    (70, 9, 2, 1, 0.02), (70, 9, 2, 2, 0.1), (70, 9, 2, 3, 0.3), (70, 9, 4, 5, 0.8),
    (70, 9, 9, 6, 1.0), (70, 9, 2, 7, 1.2), (70, 9, 2, 8, 1.5), (70, 9, 2, 9, 1.8),
    (70, 9, 2, 12, 3.0), (70, 9, 2, 15, 4.0), (70, 9, 2, 25, 9.0), (70, 4, 2, 36, 6.0),
    (70, 4, 2, 37, 6.0), (500, 11, 3, 8, 1.8), (1030, 5, 2, 8, 0.8), (1030, 3, 3, 9, 0.6)])
def test_dense_gradient_of_every_order(fl, n, M, ckpt, L, T):
    """The sweep in segments (n = 70, and 500 with unequal ones), from the tape one
    step at a time (n = 1030) and, for L = 1 and L = 37, term by term, at every
    block count: the derivative of the truncated map itself, against the
    oracle's derivative of the same chain (n = 70) or against differences of
    the library's own builds along a seeded direction. Both differ from the
    derivative by rounding (1e-13 of the largest entry a step) or by the
    difference quotient (its step 1e-5: 1e-10 by truncation, 1e-10 by rounding
    of a loss of order one)."""
    _say("dense gradient order", n, M, ckpt, L)
    rng = np.random.default_rng(n + L)
    H0, V = gue(n, rng), gue(n, rng)
    f = rng.uniform(-1, 1, M)
    nodes = np.stack([f, f], 1)
    W = haar_unitary(n, rng)
    a, b = orc.magnus4_weights(nodes, T / M)
    lo, hi = orc.weyl_cover(H0, V, np.zeros_like(H0), a, b)
    lo, hi = 1.05 * lo, 1.05 * hi
    kw = dict(h0=H0, hmod=V, T=T, M=M, e_min=lo, e_max=hi, L=L)
    ctx = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, **kw)
    U = ctx.build_ut().cpu().numpy()
    if n == 70:
        _, Ubar = _trace_loss_and_bar(U, W)
        g = ctx.grad(Ubar)
        ref = orc.grad_piecewise(H0, V, f, T, W, route="cheb", e_min=lo, e_max=hi, L=L)
        err = np.max(np.abs(g.sum(axis=1) - ref)) / np.max(np.abs(ref))
        _say("rel err", err)
        assert err < 1e-9
        pair = fl.FloquetContext(f_nodes=nodes, checkpoint_every=ckpt, grad_pair_sums=True, **kw)
        pair.build_ut()
        gp = pair.grad(Ubar)
        assert np.max(np.abs(gp.sum(axis=1) - g.sum(axis=1))) < 1e-12 * max(1.0, np.max(np.abs(ref)))
        return
    # a reachable loss of order one: Re Tr(W^dagger U) / sqrt(n)
    w = W / math.sqrt(n)
    g = ctx.grad(w)
    u = rng.standard_normal((M, 2))
    u /= np.linalg.norm(u)
    eps, vals = 1e-5, []
    for s in (1, -1):
        Us = fl.FloquetContext(f_nodes=nodes + s * eps * u, **kw).build_ut().cpu().numpy()
        vals.append(np.sum(w.conj() * Us).real)
    fd = (vals[0] - vals[1]) / (2 * eps)
    _say("direction", np.sum(g * u), "difference", fd)
    assert abs(np.sum(g * u) - fd) < 1e-8 * max(1.0, abs(fd))


# ---- resident sweep in the gauge frame: every row count, segments, both drives ------------------

@pytest.mark.parametrize("pair", [True, False])
@pytest.mark.parametrize("n,L", [(2, 0), (64, 0), (65, 1), (128, 2), (129, 3), (256, 0), (257, 0),
                                 (512, 0), (513, 0), (1024, 0)])
def test_tridiag_resident_sweep_at_every_row_count(fl, monkeypatch, n, L, pair):
    """1, 2, 4, 8 and 16 rows per lane at their first and last sizes, unequal
    segments, one to three terms, against the streamed sweep, which contracts
    with the commutator term by term instead of at the step's ends: complex
    couplings with one zero among them, a drive with b_k != 0 and a step with
    b_k = 0. Both sum some n M L products of order one in FP64."""
    _say("resident sweep", n, L, "pair sums", pair)
    rng = np.random.default_rng(600 + n)
    d = rng.standard_normal(n)
    e = rng.standard_normal(n - 1) + 1j * rng.standard_normal(n - 1)
    if n > 4:
        e[n // 2] = 0.0
    v = rng.standard_normal(n)
    T, M = (0.02 if L else 1.5), 9
    nodes = rng.uniform(-1, 1, (M, 2))
    nodes[4, 1] = nodes[4, 0]
    kw = dict(h0_diag=d, h0_off=e, hmod_diag=v, T=T, M=M, f_nodes=nodes, checkpoint_every=2, L=L,
              grad_pair_sums=pair)
    res = fl.FloquetContext(**kw)
    monkeypatch.setenv("FQ_TRIDIAG_STREAMED_ADJOINT", "1")
    streamed = fl.FloquetContext(**kw)
    monkeypatch.delenv("FQ_TRIDIAG_STREAMED_ADJOINT")
    U = res.build_ut().cpu().numpy()
    Us = streamed.build_ut().cpu().numpy()
    assert np.max(np.abs(U - Us)) < 1e-12
    w = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    g1, g2 = res.grad(w), streamed.grad(w)
    err = np.max(np.abs(g1 - g2)) / np.max(np.abs(g2))
    _say("rel diff", err, "max|g|", np.max(np.abs(g2)))
    assert err < 1e-10

"""Rounding of FP64 builds and propagations against the same truncated series in about
100 bits: what the library's operation order costs, apart from the series itself.

The reference splits every real matrix into slices of 20 bits, whose products torch's
float64 matmul sums exactly (20 + 20 bits and 2^11 terms stay below 2^53), and adds them as
pairs of doubles.

Tolerances, u = 2^-53: a step of norm-one columns adds a few elementwise roundings (the sum,
the step phase; 3 u) and the rounding of one sum over N products of the size of the step's
change, R / sqrt(N) each: at most u R sqrt(N) / 2 for a column of N elements; coefficients
rounded alike in every step add u R / 2 each time. Steps add in quadrature otherwise.
"""
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


# ---- pairs of doubles on the GPU: real arrays (high, low), complex ones (re, im) ----------------

def _two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def _add(x, y):
    s, e = _two_sum(x[0], y[0])
    return _two_sum(s, e + (x[1] + y[1]))


def _neg(x):
    return -x[0], -x[1]


def _halves(a):
    t = 134217729.0 * a
    h = t - (t - a)
    return h, a - h


def _scale(x, c):
    """x times the number c = (high, low)."""
    ch, cl = _halves(c[0])
    p = x[0] * c[0]
    ah, al = _halves(x[0])
    e = ((ah * ch - p) + ah * cl + al * ch) + al * cl
    return _two_sum(p, e + (x[0] * c[1] + x[1] * c[0]))


def _slices(x):
    import torch
    hi, lo = x
    m = torch.max(torch.abs(hi)).item()
    top = 2.0 ** math.ceil(math.log2(m)) if m > 0 else 1.0
    out = []
    for i in range(4):
        q = top * 2.0 ** (-20 * (i + 1))
        s = torch.round(hi / q) * q
        out.append(s)
        hi, lo = _two_sum(hi - s, lo)
    return out


def _mm(x, y):
    import torch
    a, b = _slices(x), _slices(y)
    acc = None
    for w in range(3, -1, -1):
        for i in range(w, -1, -1):
            p = a[i] @ b[w - i]
            z = (p, torch.zeros_like(p))
            acc = z if acc is None else _add(acc, z)
    return acc


def _cmm(X, Y):
    return (_add(_mm(X[0], Y[0]), _neg(_mm(X[1], Y[1]))), _add(_mm(X[0], Y[1]), _mm(X[1], Y[0])))


def _cadd(X, Y):
    return _add(X[0], Y[0]), _add(X[1], Y[1])


def _cscale(X, c):
    return _scale(X[0], c), _scale(X[1], c)


def _minus_i(X):
    return X[1], _neg(X[0])


def _pair(v):
    v = np.longdouble(v)
    return float(v), float(v - np.longdouble(float(v)))


def _lift(a):
    import torch
    t = [torch.from_numpy(np.ascontiguousarray(p)).to("cuda") for p in (a.real, a.imag)]
    return tuple((p, torch.zeros_like(p)) for p in t)


def _reference(fl, kw, L, X):
    """E_M ... E_1 X with the library's step weights, interval and Bessel weights."""
    M, f, cf4 = kw["M"], np.asarray(kw["f_nodes"]), kw["scheme"] == "cf4"
    h = kw["T"] / (M * (2 if cf4 else 1))
    beta, dE = 0.5 * (kw["e_max"] + kw["e_min"]), 0.5 * (kw["e_max"] - kw["e_min"])
    c = fl.bessel_weights(h * dE, L)
    H0, V = _lift(kw["h0"]), _lift(kw["hmod"])
    K = _minus_i(_cadd(_cmm(H0, V), _cscale(_cmm(V, H0), (-1.0, 0.0))))
    one = _lift(np.eye(len(kw["h0"]), dtype=complex))
    s3 = math.sqrt(3.0)
    p, q = 0.5 + 0.57735026918962576451, 0.5 - 0.57735026918962576451
    arg = np.longdouble(beta) * np.longdouble(h)
    phr, phi = _pair(np.cos(arg)), _pair(-np.sin(arg))
    X = _lift(X)
    for f1, f2 in f:
        subs = ([(p * f1 + q * f2, 0.0), (q * f1 + p * f2, 0.0)] if cf4 else
                [(0.5 * (f1 + f2), s3 * h * (f1 - f2) / 12.0)])
        for a, b in subs:
            Ht = _cadd(_cadd(H0, _cscale(V, (a, 0.0))), _cscale(K, (b, 0.0)))
            Ht = _cadd(Ht, _cscale(one, (-beta, 0.0)))
            Ht = _cscale(Ht, (1.0 / dE, 0.0))
            Y, p0, p1 = _cscale(X, (float(c[0]), 0.0)), X, _cmm(Ht, X)
            for l in range(1, L + 1):
                if l > 1:
                    t = _cscale(_cmm(Ht, p1), (2.0, 0.0))
                    p0, p1 = p1, _cadd(t, _cscale(p0, (-1.0, 0.0)))
                t = _cscale(p1, (float(c[l]), 0.0))
                for _ in range(l % 4):
                    t = _minus_i(t)
                Y = _cadd(Y, t)
            t = _cscale(_minus_i(Y), (-phi[0], -phi[1]))      # i phi Y
            X = _cadd(_cscale(Y, phr), t)
    return X


def _worst_column(U, ref):
    import torch
    d = 0.0
    for u, r in ((U.real, ref[0]), (U.imag, ref[1])):
        e = (u.contiguous() - r[0]) - r[1]
        d = d + torch.sum(e * e, dim=0)
    return torch.sqrt(torch.max(d)).item()


def _problem(n, M, T, scheme):
    rng = np.random.default_rng(7 * n + M)
    t = (np.arange(M)[:, None] + np.array([0.5 - math.sqrt(3) / 6, 0.5 + math.sqrt(3) / 6])) * T / M
    f = 0.85 * np.cos(2 * math.pi / T * t) + 0.1 * rng.uniform(-1, 1, (M, 2))
    return dict(h0=gue(n, rng), hmod=gue(n, rng), T=T, M=M, f_nodes=f, scheme=scheme, e_min=-5.3,
                e_max=5.7)


def _bound(ctx, n, M, scheme):
    subs = M * (2 if scheme == "cf4" else 1)
    R, u = ctx.report["R"], 2.0 ** -53
    return u * math.sqrt(subs) * (3.0 + 0.5 * R * math.sqrt(n)) + 0.5 * u * R * subs


# steps through their propagators one by one: the whole build, and single steps of it
@pytest.mark.parametrize("scheme,T", [("magnus4", 0.9), ("cf4", 0.3)])
@pytest.mark.parametrize("n", [1030, 1100])
def test_steps_one_by_one(fl, n, scheme, T):
    print("[case] rounding, steps", n, scheme, T, flush=True)
    M = 4
    kw = _problem(n, M, T, scheme)
    ctx = fl.FloquetContext(**kw)
    ref = _reference(fl, kw, ctx.report["L"], np.eye(n, dtype=complex))
    err, bound = _worst_column(ctx.build_ut(), ref), _bound(ctx, n, M, scheme)
    print("[case] L", ctx.report["L"], "e_col", err, "bound", bound, flush=True)
    assert err < bound


# propagators of a batch of steps at once, applied to a few states and to many
@pytest.mark.parametrize("scheme", ["magnus4", "cf4"])
@pytest.mark.parametrize("n,M", [(64, 60), (100, 60), (256, 40)])
def test_batches_of_steps(fl, n, M, scheme):
    print("[case] rounding, batches", n, M, scheme, flush=True)
    kw = _problem(n, M, 4.0, scheme)
    ctx = fl.FloquetContext(**kw)
    ref = _reference(fl, kw, ctx.report["L"], np.eye(n, dtype=complex))
    for cols in (4, n):
        X = ctx.propagate(np.ascontiguousarray(np.eye(n, dtype=complex)[:, :cols]))
        part = tuple(tuple(t[:, :cols] for t in z) for z in ref)
        err, bound = _worst_column(X, part), _bound(ctx, n, M, scheme)
        print("[case] states", cols, "e_col", err, "bound", bound, flush=True)
        assert err < bound


# Builds cut into segments whose operators are multiplied up. A product A B of the operators
# of len steps each rounds three times elementwise, and sums the change of B, min(1, R len),
# with eight or N / 16 partial sums: sqrt(12 + N / 10) u for a whole column (u^2 (4 / 3)
# (8.5 + N / 32) in blocks of 16, u^2 N / 12 + 6 in eight parts)
@pytest.mark.parametrize("n,M,T,segments", [(40, 60, 1.2, 30), (64, 100, 2.0, 50), (100, 100, 2.0, 100),
                                            (199, 50, 1.0, 32), (256, 64, 1.28, 32), (500, 40, 0.8, 8)])
def test_segments_multiplied_up(fl, n, M, T, segments):
    print("[case] rounding, segments", n, M, T, flush=True)
    kw = _problem(n, M, T, "magnus4")
    ctx = fl.FloquetContext(**kw)
    ref = _reference(fl, kw, ctx.report["L"], np.eye(n, dtype=complex))
    R, u = ctx.report["R"], 2.0 ** -53
    products, cnt, length = 0.0, segments, M / segments
    while cnt > 1:
        products += cnt // 2 * (9.0 + (12.0 + n / 10) * min(1.0, R * length) ** 2)
        cnt, length = (cnt + 1) // 2, 2 * length
    steps = M * (3.0 + 0.5 * R * math.sqrt(n)) ** 2
    bound = u * math.sqrt(steps + products) + 0.5 * u * R * M
    err = _worst_column(ctx.build_ut(), ref)
    print("[case] L", ctx.report["L"], "e_col", err, "bound", bound, flush=True)
    assert err < bound

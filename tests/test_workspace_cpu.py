"""Device workspace on the CPU (no GPU needed): problems whose planes and step tables fit the
static array of the one-shot build are accepted by it, whatever scratch a larger workspace
would add."""
import ctypes
import math

import numpy as np
import pytest

from paper_1508_07621_amd import _abi

FAKE = ctypes.c_void_p(0x1000)
STATIC = 256 << 20


def _system(n, layout=_abi.FQ_DENSE, drives=1):
    s = _abi.FqSystem()
    s.n, s.layout, s.n_drive = n, layout, drives
    s.h0 = s.hmod = FAKE
    s.h0_diag = s.h0_off = s.hmod_diag = FAKE
    if drives > 1:
        s._arr = (ctypes.c_void_p * drives)(*[FAKE] * drives)
        s.hmods = ctypes.cast(s._arr, ctypes.POINTER(ctypes.c_void_p))
    return s


def _params(M, scheme=_abi.FQ_MAGNUS4, drives=1, precision=0, checkpoint_every=0, reortho=0):
    f = np.zeros((3 if scheme == _abi.FQ_MAGNUS6 else 2) * M * drives)
    p = _abi.FqParams()
    p.T, p.M, p.L, p.tol = 1.0, M, 0, 1e-12
    p.f_nodes = _abi.dptr(f)
    p.e_min = p.e_max = math.nan
    p.precision, p.checkpoint_every, p.scheme = precision, checkpoint_every, scheme
    p.reorthonormalize = reortho
    p._keep = f
    return p


def _bytes(s, p):
    n = ctypes.c_size_t(0)
    assert _abi.lib().fq_workspace_bytes(ctypes.byref(s), ctypes.byref(p), ctypes.byref(n)) == 0
    return n.value


def _pad(x, t):
    return -(-x // t) * t


def _tables(n, steps):
    """Reduction scratch, averages, step scalars and Bessel coefficients, 256-byte aligned."""
    return sum(_pad(b, 256) for b in (512, 24 * n, 16 * steps, 16 * 65536))


def _dense_needs(n, M, scheme, drives, precision):
    """H0, the drive block, Ht, X, Y and two P (two more in mixed precision, nine
    commutators in the sixth-order scheme), and the tables."""
    steps = M * (2 if scheme == _abi.FQ_CF4 else 1)
    J = 2 if drives == 1 else drives if scheme == _abi.FQ_CF4 else 2 * drives + drives * (drives - 1) // 2
    planes = 6 + J + (2 if precision else 0) + (9 if scheme == _abi.FQ_MAGNUS6 else 0)
    np_ = _pad(n, 128 if n > 1984 else 64)
    return planes * 16 * np_ * np_ + _tables(n, steps)


def _tridiag_needs(n, M, scheme, reortho):
    """X (and three more for the re-orthonormalisation), gauge factors, and the tables."""
    steps = M * (2 if scheme == _abi.FQ_CF4 else 1)
    np_ = _pad(n, 128 if n > 1984 else 64)
    return (1 + 3 * reortho) * 16 * np_ * np_ + _pad(16 * n * steps, 256) + _tables(n, steps)


def _check(s, p, needs, label):
    got = _bytes(s, p)
    assert got >= needs, label
    if needs <= STATIC:
        assert got <= STATIC, (label, needs, got)
    # the one-shot entry point checks the size before any device work
    rep = _abi.FqReport()
    if needs > STATIC:
        st = _abi.lib().floquet_build_UT_static(ctypes.byref(s), ctypes.byref(p), None, FAKE,
                                                ctypes.byref(rep))
        assert st == _abi.FQ_ERR_ARG, label


# the last megabytes of the array: four drive terms between 250 and 256 MiB, long drives
# whose step tables fill what the planes leave, and both sides of the limit
@pytest.mark.parametrize("scheme", [_abi.FQ_MAGNUS4, _abi.FQ_MAGNUS6, _abi.FQ_CF4])
@pytest.mark.parametrize("drives", [1, 2, 4])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_dense_problems_that_fit_the_static_array(scheme, drives, precision):
    if drives > 1 and scheme == _abi.FQ_MAGNUS6:
        pytest.skip("one drive term")
    for n in (1, 64, 300, 700, 900, 960, 1024, 1217, 1280, 1344, 1400, 1408):
        for M in (1, 100, 30000, 55000, 400000, 700000):
            needs = _dense_needs(n, M, scheme, drives, precision)
            _check(_system(n, drives=drives), _params(M, scheme, drives, precision), needs,
                   (n, M, scheme, drives, precision))


@pytest.mark.parametrize("scheme", [_abi.FQ_MAGNUS4, _abi.FQ_CF4])
@pytest.mark.parametrize("reortho", [0, 1])
def test_tridiagonal_problems_that_fit_the_static_array(scheme, reortho):
    for n, steps in ((1, 7_000_000), (2, 4_500_000), (21, 700_000), (64, 240_000), (1000, 15_000),
                     (1025, 14_000), (2000, 5_000), (3000, 2_000), (3900, 30), (3968, 1)):
        for M in (1, 40, max(1, steps // 2), steps):
            needs = _tridiag_needs(n, M, scheme, reortho)
            _check(_system(n, _abi.FQ_TRIDIAG), _params(M, scheme, reortho=reortho), needs,
                   (n, M, scheme, reortho))


# ---- gradients -----------------------------------------------------------------------------------

def _least(s, p):
    n = ctypes.c_size_t(0)
    assert _abi.lib().fq_workspace_min_bytes(ctypes.byref(s), ctypes.byref(p), ctypes.byref(n)) == 0
    return n.value


def _grad_needs(n, M, scheme, every, tridiag):
    """The tape and three matrices per step of a checkpoint segment; dense also the two
    stacks of the term-by-term sweep, Lambda and the accumulators."""
    sub = 2 if scheme == _abi.FQ_CF4 else 1
    steps, seg = M * sub, every * sub
    tape = -(-steps // seg) + 1
    np_ = _pad(n, 128 if n > 1984 else 64)
    if tridiag:
        return _tridiag_needs(n, M, scheme, 0) + 16 * n * n * (tape + 3 * seg) + 16 * steps
    return _dense_needs(n, M, scheme, 1, 0) + 16 * np_ * np_ * (tape + 3 * seg + 5) + 16 * steps


# the least workspace follows the caller's checkpoint spacing; the recommended one adds at
# most the scratch that the header names
@pytest.mark.parametrize("scheme", [_abi.FQ_MAGNUS4, _abi.FQ_CF4])
@pytest.mark.parametrize("tridiag", [False, True])
def test_gradient_workspace_follows_the_checkpoints(scheme, tridiag):
    layout = _abi.FQ_TRIDIAG if tridiag else _abi.FQ_DENSE
    for n in (16, 256, 400, 960, 1000, 1500, 2048) + (() if tridiag else (10000,)):
        for M, every in ((64, 1), (64, 8), (128, 16), (100, 100), (5000, 16), (5000, 100)):
            s, p = _system(n, layout), _params(M, scheme, checkpoint_every=every)
            label = (n, M, every, scheme, tridiag)
            needs, least, full = _grad_needs(n, M, scheme, every, tridiag), _least(s, p), _bytes(s, p)
            assert least <= min(needs + 4096, full), label
            np_ = _pad(n, 128 if n > 1984 else 64)
            scratch = (144 << 20) + (2 << 30) + (5 << 30) + 26 * 16 * np_ * np_
            if tridiag:  # four matrices per segment in the place of the tape
                scratch += max(0, needs - 3 * 16 * n * n * every)
            assert full <= needs + scratch, (label, needs, full)

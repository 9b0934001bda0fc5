"""Contexts with the least workspace, and between that and the recommended one: the same
results as with all the scratch, by the step-by-step forms."""
import ctypes

import numpy as np
import pytest

from workloads import dimer_tridiag, gue

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


def _dense(n, M, scheme="magnus4", drives=1, **kw):
    rng = np.random.default_rng(n + 10 * M)
    nodes = 3 if scheme == "magnus6" else 2
    V = [gue(n, rng) for _ in range(drives)]
    f = rng.uniform(-1, 1, (M, nodes) + ((drives,) if drives > 1 else ()))
    return dict(h0=gue(n, rng), hmod=V if drives > 1 else V[0], T=0.1 * M, M=M, f_nodes=f,
                scheme=scheme, **kw)


def _tridiag(n, M, **kw):
    d, e, v = dimer_tridiag(n - 1, 1.0, 0.01)
    f = np.random.default_rng(n).uniform(-1, 1, (M, 2))
    return dict(h0_diag=d, h0_off=e, hmod_diag=v, T=2.0 * M / n, M=M, f_nodes=f, **kw)


def _lean(fl, monkeypatch, kw):
    """A context where almost nothing is free beyond the least workspace."""
    with monkeypatch.context() as m:
        m.setattr(fl, "_free_bytes", lambda device: 0)
        m.setattr(fl, "_UNASKED_SCRATCH", 0)
        ctx = fl.FloquetContext(**kw)
    return ctx


def _results(fl, ctx, n, S, M, grad):
    rng = np.random.default_rng(5)
    X = rng.standard_normal((n, 3)) + 1j * rng.standard_normal((n, 3))
    X /= np.linalg.norm(X, axis=0)
    W = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    fg = rng.uniform(-1, 1, (M, S))
    out = [ctx.build_ut().cpu().numpy()]
    if grad:
        out.append(ctx.grad(W) / np.linalg.norm(W))
        out.append(ctx.grad(W) / np.linalg.norm(W))     # again from the same build
    out.append(ctx.propagate(X).cpu().numpy())
    out.append(ctx.period_average(X, fg))
    return out


CASES = [("dense 40", _dense(40, 20)), ("dense 200", _dense(200, 12)),
         ("dense cf4 two drives", _dense(130, 6, "cf4", 2)), ("dense magnus6", _dense(100, 6, "magnus6")),
         ("dense 1030", _dense(1030, 4)), ("bf16x3 600", _dense(600, 4, precision="bf16x3")),
         ("fp32 300", _dense(300, 4, precision="fp32")),
         ("tridiagonal 21", _tridiag(21, 50)), ("tridiagonal 700", _tridiag(700, 6)),
         ("tridiagonal 1500", _tridiag(1500, 3, scheme="cf4")),
         ("gradient 64", _dense(64, 12, checkpoint_every=5)),
         ("gradient 200 cf4", _dense(200, 8, "cf4", checkpoint_every=8)),
         ("gradient 150 two drives", _dense(150, 6, drives=2, checkpoint_every=2)),
         ("gradient 1030", _dense(1030, 3, checkpoint_every=2)),
         ("gradient tridiagonal 33", _tridiag(33, 40, checkpoint_every=6)),
         ("gradient tridiagonal 700", _tridiag(700, 5, checkpoint_every=2))]


@pytest.mark.parametrize("name,kw", CASES, ids=[c[0] for c in CASES])
def test_least_workspace(fl, monkeypatch, name, kw):
    print("[case] lean", name, flush=True)
    S = len(kw["hmod"]) if isinstance(kw.get("hmod"), list) else 1
    full = fl.FloquetContext(**kw)
    lean = _lean(fl, monkeypatch, kw)
    assert lean.workspace.numel() < full.workspace.numel()
    grad = kw.get("checkpoint_every", 0) > 0
    a = _results(fl, full, full.n, S, kw["M"], grad)
    b = _results(fl, lean, lean.n, S, kw["M"], grad)
    tol = 5e-7 if kw.get("precision") == "bf16x3" else 1e-11
    scale = [1.0] * len(a)
    scale[-1] = max(abs(full.report["e_min"]), abs(full.report["e_max"]))
    for x, y, s in zip(a, b, scale):
        err = np.max(np.abs(x - y)) / s
        print("[case] difference", err, flush=True)
        assert err < tol


# sizes between the two: each context takes what fits, and one byte less than the least is refused
def test_workspaces_in_between(fl):
    import torch
    from paper_1508_07621_amd import _abi
    kw = _dense(150, 16, checkpoint_every=4)
    ref = fl.FloquetContext(**kw)
    U0 = ref.build_ut()
    W = torch.ones_like(U0)
    g0 = ref.grad(W)
    L = _abi.lib()
    least = ctypes.c_size_t(0)
    _abi.check(L.fq_workspace_min_bytes(ctypes.byref(ref._sys), ctypes.byref(ref._par),
                                        ctypes.byref(least)))
    full = ref.workspace.numel()
    stream = torch.cuda.current_stream().cuda_stream
    for size in (least.value - 1, least.value, (least.value + full) // 2, full - 1, full):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        h = ctypes.c_void_p()
        st = L.fq_create(ctypes.byref(h), ctypes.byref(ref._sys), ctypes.byref(ref._par),
                         ws.data_ptr(), size, stream)
        if size < least.value:
            assert st == _abi.FQ_ERR_ARG
            continue
        _abi.check(st)
        U, g = torch.empty_like(U0), np.empty_like(g0)
        rep = _abi.FqReport()
        _abi.check(L.floquet_build_UT(h, U.data_ptr(), ctypes.byref(rep)))
        _abi.check(L.floquet_grad(h, W.data_ptr(), _abi.dptr(g)))
        L.fq_destroy(h)
        print("[case] workspace", size, (U - U0).abs().max().item(), np.max(np.abs(g - g0)), flush=True)
        assert (U - U0).abs().max().item() < 1e-12
        assert np.max(np.abs(g - g0)) < 1e-10 * np.max(np.abs(g0))


# an allocation that fails for the scratch falls back to the least, one that fails for that raises
def test_out_of_memory_falls_back(fl, monkeypatch):
    import torch
    kw = _dense(100, 8, checkpoint_every=4)
    full = fl.FloquetContext(**kw)
    limit = [full.workspace.numel() - 1]
    empty = torch.empty

    def short(*size, **k):
        if k.get("dtype") == torch.uint8 and size[0] > limit[0]:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(*size, **k)
    monkeypatch.setattr(torch, "empty", short)
    lean = fl.FloquetContext(**kw)
    assert lean.workspace.numel() < full.workspace.numel()
    assert (lean.build_ut() - full.build_ut()).abs().max().item() < 1e-13
    limit[0] = lean.workspace.numel() - 1
    with pytest.raises(torch.cuda.OutOfMemoryError):
        fl.FloquetContext(**kw)

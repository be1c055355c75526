"""Views on the smallest workspace they take (test_workspace_sizes.py pins
those sizes) and batches on the smallest, a part and all of the memory that a
view would like to borrow: the oracle's values, batches equal to single updates
bit for bit, and no byte outside the buffers touched."""

from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle as O
import synth
from tests.gpu_util import dev, host, need_gpu, note, storage_inputs

pytestmark = pytest.mark.gpu

GUARD = 1 << 16


def _guarded(torch, nbytes):
    buf = torch.full((nbytes + 2 * GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    return buf, buf[GUARD:GUARD + nbytes]


def _intact(buf):
    return bool((buf[:GUARD] == 0x5A).all()) and bool((buf[-GUARD:] == 0x5A).all())


def _read(lv, h, p, n, td):
    import torch
    out = torch.empty(n, n, dtype=td, device="cuda")
    lv.lv_view_read(h, p, out, td)
    return out


@pytest.mark.parametrize("mode,n,k,r_max,r", [
    ("fp64", 256, 16, 1, 1), ("fp64", 300, 2, 8, 3), ("fp64", 512, 4, 1, 1), ("fp64", 700, 8, 3, 2),
    ("fp64", 1030, 16, 2, 2), ("fp64", 300, 4, 64, 33), ("fp32", 256, 16, 1, 1), ("fp32", 512, 16, 1, 1),
    ("fp32", 1300, 8, 8, 4), ("fp32", 300, 256, 2, 2), ("fp32", 260, 4, 128, 100), ("shadow", 256, 16, 4, 4),
    ("shadow", 700, 16, 1, 1), ("shadow", 600, 4, 128, 70), ("shadow", 1100, 16, 32, 20)])
def test_plain_views(mode, n, k, r_max, r):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd, td = (np.float64, torch.float64) if mode == "fp64" else (np.float32, torch.float32)
    code = {"fp64": lv.LV_FP64, "fp32": lv.LV_FP32, "shadow": lv.LV_FP32_BF16SHADOW}[mode]
    counts = [2, 9, 5]
    A64 = synth.gaussian_matrix(n, seed=n + k, config=2)
    Us, Vs = synth.update_factors(n, r, sum(counts), seed=n + r, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, nd)
    U, V = dev(Us, td), dev(Vs, td)
    bufs, handles = [], []
    for _ in range(4):   # single updates; batches on the workspace, on a part and on all of the lent memory
        buf, ws = _guarded(torch, lv.lv_view_footprint(n, k, r_max, code))
        handles.append(lv.lv_view_create(dev(A, td), k, r_max, code, ws))
        bufs.append(buf)
    want = lv.lv_view_batch_bytes(handles[0])
    for h, part in ((handles[2], want // 512 * 256), (handles[3], want)):
        if part:
            buf, ws = _guarded(torch, part)
            lv.lv_view_set_batch_workspace(h, ws)
            bufs.append(buf)
    t = 0
    P = O.reeval(A, k)
    for c in counts:
        for s in range(t, t + c):
            lv.lv_view_update(handles[0], U[s], V[s], td)
        for h in handles[1:]:
            lv.lv_view_update_batch(h, U[t:t + c], V[t:t + c], td)
        t += c
        for p in P:
            one = _read(lv, handles[0], p, n, td)
            for h in handles[1:]:
                assert torch.equal(one, _read(lv, h, p, n, td)), f"P_{p} after {t} updates"
    if k <= 16:
        P = O.apply_updates(P, Us, Vs)
        tol = {"fp64": 1e-10, "fp32": 1e-4, "shadow": 5e-3}[mode]
        err = max(O.maxrel(host(_read(lv, handles[0], p, n, td)), P[p]) for p in P)
        note(f"{mode} n={n} k={k} r={r}/{r_max}: lent {want} bytes, maxrel {err:.2e}")
        assert err < tol
    for buf in bufs:
        assert _intact(buf)
    for h in handles:
        lv.lv_view_destroy(h)


@pytest.mark.parametrize("mode,n,k,r,p,strategy,s", [
    ("fp64", 300, 4, 2, 7, 0, 0), ("fp64", 300, 2, 16, 1, 1, 0), ("fp64", 520, 16, 1, 40, 1, 4),
    ("fp32", 300, 8, 2, 64, 0, 0), ("fp32", 513, 16, 1, 130, 1, 0), ("shadow", 300, 16, 1, 5, 1, 8)])
def test_general_form_views(mode, n, k, r, p, strategy, s):
    """Against the same view on a workspace with room to spare."""
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd, td = (np.float64, torch.float64) if mode == "fp64" else (np.float32, torch.float32)
    code = {"fp64": lv.LV_FP64, "fp32": lv.LV_FP32, "shadow": lv.LV_FP32_BF16SHADOW}[mode]
    A64 = synth.gaussian_matrix(n, seed=n + k, config=5)
    T0, B = synth.general_operands(n, p, seed=n, config=5)
    Us, Vs = synth.update_factors(n, r, 3, seed=n + r, config=5)
    A, Us, Vs = storage_inputs(A64, Us, Vs, nd)
    out = []
    for extra in (0, 1 << 24):
        buf, ws = _guarded(torch, lv.lv_view_footprint_general(n, k, r, code, p, strategy, s) + extra)
        h = lv.lv_view_create_general(dev(A, td), k, r, code, dev(np.asarray(T0, nd), td), dev(np.asarray(B, nd), td), ws,
                                      None, strategy, s)
        for t in range(3):
            lv.lv_view_update(h, dev(Us[t], td), dev(Vs[t], td), td)
        T = torch.empty(n, p, dtype=td, device="cuda")
        lv.lv_view_read_general(h, k, T, td)
        top = s or k
        S = torch.empty(n, n, dtype=td, device="cuda")
        lv._check(lv.load().lv_view_read_sum(h, top, S.data_ptr(), n, lv._stream(None, S.device)))
        out.append((host(T), host(S), host(_read(lv, h, top, n, td))))
        assert _intact(buf)
        lv.lv_view_destroy(h)
    tol = {"fp64": 1e-12, "fp32": 1e-5, "shadow": 1e-5}[mode]   # other slices: another order of the same sums
    for what, a, b in zip("TSP", *out):
        assert O.maxrel(a, b) < tol, what
    Af = A.copy()
    for t in range(3):
        Af = Af + Us[t] @ Vs[t].T
    x = np.asarray(T0, nd).astype(np.float64)
    for _ in range(k):
        x = Af @ x + np.asarray(B, nd).astype(np.float64)
    err = O.maxrel(out[0][0], x)
    note(f"general {mode} n={n} k={k} r={r} p={p} strategy={strategy} s={s}: T maxrel {err:.2e}")
    assert err < {"fp64": 1e-10, "fp32": 1e-4, "shadow": 5e-3}[mode]


@pytest.mark.parametrize("mode,specs,count,most", [
    (2, [(256, 2, 64)], 1, 132864), (2, [(256, 2, 64)], 40, 5262848), (2, [(300, 4, 32), (256, 16, 8)], 1, 155904),
    (2, [(256, 16, 8)], 64, 1136128), (2, [(300, 16, 32)], 8, 1073920), (1, [(256, 16, 1), (300, 8, 3)], 16, 263424),
    (0, [(256, 16, 2)], 32, 299776), (1, [(512, 16, 8)], 32, 1095424), (2, [(256, 8, 16)], 50, 1698816)])
def test_rounds(mode, specs, count, most):
    """The tables of a round are no larger than they were (bytes pinned as in
    test_workspace_sizes.py), and a round runs on a workspace of that size."""
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    td = torch.float64 if mode == 0 else torch.float32
    views = [lv.View(torch.zeros(n, n, dtype=td, device="cuda"), k, r_max=r, mode=mode)
             for _ in range(count) for n, k, r in specs]
    assert lv.lv_batch_footprint(views) <= most
    buf, ws = _guarded(torch, most // 256 * 256)
    batch = lv.lv_batch_create(views, ws)
    one = torch.ones(specs[0][0], 1, dtype=td, device="cuda")
    lv.lv_batch_stage(batch, 0, one, one, td, device=one.device)
    lv.lv_batch_update(batch, device=one.device)
    assert bool((views[0].read(1) == 1).all())
    assert all(float(v.read(1).abs().max()) == 0 for v in views[1:])
    assert _intact(buf)
    lv.lv_batch_destroy(batch)
    for v in views:
        v.close()


def _small(torch, lv, kind, A, T0, B, k, r, mode, model, s, strategy, td):
    """A chain or linear general form on the smallest workspace; returns (buffer, handle)."""
    lib, n, h = lv.load(), A.shape[0], ctypes.c_void_p()
    if kind == "chain":
        buf, ws = _guarded(torch, lib.lv_chain_footprint(n, k, r, mode, model, s))
        lv._check(lib.lv_chain_create(A.data_ptr(), n, n, k, r, mode, model, s, ws.data_ptr(), ws.numel(),
                                      lv._stream(None, A.device), ctypes.byref(h)))
    else:
        p = T0.shape[1]
        buf, ws = _guarded(torch, lib.lv_glin_footprint(n, k, r, mode, p, strategy))
        lv._check(lib.lv_glin_create(A.data_ptr(), n, n, k, r, mode, T0.data_ptr(), p, B.data_ptr(), p, p, strategy,
                                     ws.data_ptr(), ws.numel(), lv._stream(None, A.device), ctypes.byref(h)))
    return buf, h


@pytest.mark.parametrize("kind,n,k,r,model,s,strategy,p,dtype", [
    ("chain", 512, 2, 1, 1, 0, 0, 0, "f64"), ("chain", 300, 4, 8, 1, 0, 0, 0, "f64"), ("chain", 520, 8, 2, 2, 4, 0, 0, "f64"),
    ("chain", 700, 12, 1, 1, 0, 0, 0, "f32"), ("glin", 1000, 3, 1, 0, 0, 0, 130, "f64"), ("glin", 600, 4, 2, 0, 0, 1, 79, "f64"),
    ("glin", 512, 2, 8, 0, 0, 2, 3, "f64"), ("glin", 300, 5, 1, 0, 0, 1, 16, "f32")])
def test_models(kind, n, k, r, model, s, strategy, p, dtype):
    """Against the same handle on its full workspace: other slices, so another
    order of the same sums; the tolerances of the modes, a tenth of them."""
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    lib = lv.load()
    td, nd, mode = (torch.float64, np.float64, 0) if dtype == "f64" else (torch.float32, np.float32, 1)
    A = dev(np.asarray(synth.gaussian_matrix(n, seed=n, config=4), nd), td)
    Us, Vs = (np.asarray(x, nd) for x in synth.update_factors(n, r, 3, seed=n, config=4))
    T0 = B = None
    if kind == "glin":
        T0, B = (dev(np.asarray(x, nd), td) for x in synth.general_operands(n, p, seed=n, config=5))
    buf, h = _small(torch, lv, kind, A, T0, B, k, r, mode, model, s, strategy, td)
    full = lv.Chain(A, k, r_max=r, model=model, s=s) if kind == "chain" else lv.GLin(A, k, T0, B, r_max=r, strategy=strategy)
    update = lib.lv_chain_update if kind == "chain" else lib.lv_glin_update
    read = lib.lv_chain_read if kind == "chain" else lib.lv_glin_read
    st = lv._stream(None, A.device)
    for t in range(3):
        U, V = dev(Us[t], td), dev(Vs[t], td)
        lv._check(update(h, U.data_ptr(), V.data_ptr(), r, r, r, st))
        full.update(U, V)
        torch.cuda.synchronize()
    cols = n if kind == "chain" else p
    for i in (full.powers() if kind == "chain" else range(1, k + 1)):
        out = torch.empty(n, cols, dtype=td, device="cuda")
        lv._check(read(h, i, out.data_ptr(), cols, st))
        assert O.maxrel(host(out), host(full.read(i))) < (1e-11 if dtype == "f64" else 1e-5), i
    assert _intact(buf)
    (lib.lv_chain_destroy if kind == "chain" else lib.lv_glin_destroy)(h)
    full.close()

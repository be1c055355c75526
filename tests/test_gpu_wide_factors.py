"""Level passes from bfloat16 factors kept transposed (shadow mode, level
ranks 64 and up): every width of the pass, orders with one and with several
splits of the summation ranges, ragged orders, ranks below the view's largest,
and an order whose scratch is too small for the factors.  On integer matrices
whose values are exact in bfloat16 the powers must be exact; batches and
rounds must equal single updates bit for bit."""

from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import synth
from tests.gpu_util import dev, need_gpu, note, read_all, storage_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,r_max,r", [
    (256, 4, 128, 128), (400, 4, 128, 128), (257, 8, 32, 32), (1100, 8, 32, 20), (1024, 4, 64, 33), (2304, 16, 16, 16),
    (600, 8, 64, 5)])
def test_integer_powers_exact(n, k, r_max, r):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    g = synth.rng(11, 0, n, r)
    A = np.zeros((n, n))
    A[np.arange(n), g.permutation(n)] = 1.0
    view = lv.View(dev(A, torch.float32), k, r_max=r_max, mode=lv.LV_FP32_BF16SHADOW)
    P = O.reeval(A, k)
    cur = A.copy()
    for _ in range(2):
        U, V = np.zeros((n, r)), np.zeros((n, r))
        for c in range(r):
            a, b = g.integers(0, n, size=2)
            while a == b or cur[a, b]:
                a, b = g.integers(0, n, size=2)
            cur[a, b] = U[a, c] = V[b, c] = 1.0
        dU, dV = O.incr_factors(P, U, V)
        P = O.incr_update(P, U, V)
        big = max(np.abs(x).max() for x in [*dU.values(), *dV.values(), *P.values()])
        assert big < 256, "precondition: powers and factors exact in bfloat16"
        view.update(dev(U, torch.float32), dev(V, torch.float32))
        got = read_all(view)
        for i in P:
            np.testing.assert_array_equal(got[i], P[i], err_msg=f"P_{i}")
    note(f"exact: n={n} k={k} r={r}/{r_max}")
    view.close()


@pytest.mark.parametrize("n,k,r_max,r", [(300, 4, 32, 32), (1100, 4, 64, 40), (520, 8, 32, 32), (256, 4, 128, 128)])
def test_batches_and_rounds_equal_single_updates(n, k, r_max, r):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    A64 = synth.gaussian_matrix(n, seed=n + k, config=2)
    Us, Vs = synth.update_factors(n, r, 4, seed=n + r, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, np.float32)
    U, V = dev(Us, torch.float32), dev(Vs, torch.float32)
    one, batch, rounds = [lv.View(dev(A, torch.float32), k, r_max=r_max, mode=lv.LV_FP32_BF16SHADOW) for _ in range(3)]
    group = lv.Batch([rounds])   # a round's updates have rank r_max and the heights it tuned
    for v in (one, batch):
        v.set_tile_rows(rounds.tile_rows())
    for t in range(4):
        one.update(U[t], V[t])
        group.stage(0, U[t], V[t])
        group.update()
    batch.update_batch(U, V)
    for p in one.powers():
        assert torch.equal(one.read(p), batch.read(p)), f"P_{p}: batch"
        assert torch.equal(one.read(p), rounds.read(p)), f"P_{p}: round"
    group.close()
    for v in (one, batch, rounds):
        v.close()


@pytest.mark.parametrize("mode,n,k,r", [
    ("fp64", 100, 4, 32), ("fp64", 130, 4, 64), ("fp64", 700, 8, 32), ("fp64", 385, 2, 128), ("fp32", 257, 4, 32),
    ("fp32", 300, 8, 33), ("fp32", 1100, 4, 128)])
def test_integer_powers_exact_without_shadows(mode, n, k, r):
    """Gram and tail of ranks 32 to 256 on the double matrix cores: whole
    numbers stay whole (orders of one and of several row tiles, the last one
    cut short)."""
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    td = torch.float64 if mode == "fp64" else torch.float32
    g = synth.rng(12, 0, n, r)
    A = np.zeros((n, n))
    A[np.arange(n), g.permutation(n)] = 1.0
    view = lv.View(dev(A, td), k, r_max=r, mode=lv.LV_FP64 if mode == "fp64" else lv.LV_FP32)
    P = O.reeval(A, k)
    for _ in range(2):
        U = (g.random((n, r)) < 1.5 / n).astype(np.float64)
        V = (g.random((n, r)) < 1.5 / n).astype(np.float64)
        dU, dV = O.incr_factors(P, U, V)
        P = O.incr_update(P, U, V)
        assert max(np.abs(x).max() for x in [*dU.values(), *dV.values(), *P.values()]) < 2 ** 24
        view.update(dev(U, td), dev(V, td))
        got = read_all(view)
        for i in P:
            np.testing.assert_array_equal(got[i], P[i], err_msg=f"P_{i}")
    note(f"exact: {mode} n={n} k={k} r={r}")
    view.close()

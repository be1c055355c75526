"""Infinities and NaN in an update: they reach the entries that the update's
formulas give them, and no others, through the lane sums, the matrix-core
passes, Gram and tail; a batch leaves the values of single updates."""

from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import synth
from tests.gpu_util import dev, host, need_gpu, note, storage_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["inf", "nan"])
@pytest.mark.parametrize("mode,n,k,r", [("fp64", 300, 4, 1), ("fp64", 257, 8, 4), ("fp64", 256, 4, 32),
                                        ("fp32", 300, 8, 1), ("fp32", 513, 4, 4), ("fp32", 300, 4, 32),
                                        ("shadow", 300, 4, 1), ("shadow", 520, 8, 2)])
def test_nonfinite_entries(mode, n, k, r, what):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd, td = (np.float64, torch.float64) if mode == "fp64" else (np.float32, torch.float32)
    A64 = synth.gaussian_matrix(n, seed=n + k, config=2)
    Us, Vs = synth.update_factors(n, r, 2, seed=n + r, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, nd)
    Us[0][7, r - 1] = {"inf": np.inf, "nan": np.nan}[what]
    code = {"fp64": lv.LV_FP64, "fp32": lv.LV_FP32, "shadow": lv.LV_FP32_BF16SHADOW}[mode]
    one, batch = [lv.View(dev(A, td), k, r_max=r, mode=code) for _ in range(2)]
    with np.errstate(invalid="ignore"):
        P = O.incr_update(O.reeval(A, k), Us[0], Vs[0])
    one.update(dev(Us[0], td), dev(Vs[0], td))
    for i in P:
        got = host(one.read(i))
        assert np.array_equal(np.isfinite(got), np.isfinite(P[i])), f"P_{i}: finite"
        if mode == "shadow":   # rounded inputs: a sum near zero may take the other sign, and inf - inf is NaN
            continue
        assert np.array_equal(np.isnan(got), np.isnan(P[i])), f"P_{i}: NaN"
        assert np.array_equal(np.isposinf(got), np.isposinf(P[i])), f"P_{i}: +inf"
        assert np.array_equal(np.isneginf(got), np.isneginf(P[i])), f"P_{i}: -inf"
    one.update(dev(Us[1], td), dev(Vs[1], td))
    batch.update_batch(dev(Us, td), dev(Vs, td))
    for i in P:
        a, b = one.read(i), batch.read(i)
        assert bool(((a == b) | (a.isnan() & b.isnan())).all()), f"P_{i}: batch"
    note(f"{what} {mode} n={n} k={k} r={r}: {sum(int((~np.isfinite(x)).sum()) for x in P.values())} entries")
    one.close()
    batch.close()

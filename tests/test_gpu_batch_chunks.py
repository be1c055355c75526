"""Batches of updates whose levels take several updates per pass
(View.update_batch): every split of a batch into chunks and groups, ranks on
both sides of the widest shared pass, updates below the view's largest rank,
and chunks cut short by drift checks.  A batch must equal the same updates
applied one by one bit for bit."""

from __future__ import annotations

import numpy as np
import pytest

import synth
from tests.gpu_util import dev, need_gpu, note, storage_inputs

pytestmark = pytest.mark.gpu


def _pair(lv, A, td, mode, k, r_max, every):
    views = [lv.View(dev(A, td), k, r_max=r_max, mode=mode) for _ in range(2)]
    if every:
        for v in views:
            v.set_drift_check(every)
    return views


@pytest.mark.parametrize("mode,n,k,r_max,r,every", [
    ("fp32", 300, 4, 1, 1, 0), ("fp32", 513, 16, 1, 1, 0), ("fp32", 256, 16, 1, 1, 3), ("fp32", 700, 8, 2, 2, 0),
    ("fp32", 700, 8, 4, 3, 0), ("fp32", 520, 16, 8, 1, 0), ("fp32", 300, 4, 8, 8, 0), ("fp32", 300, 4, 16, 12, 0),
    ("fp64", 257, 16, 1, 1, 0), ("fp64", 400, 8, 3, 3, 5), ("fp64", 300, 4, 8, 2, 0), ("fp64", 256, 32, 2, 2, 0),
    ("shadow", 300, 8, 1, 1, 0), ("shadow", 300, 4, 4, 4, 3)])
def test_batches_equal_single_updates(mode, n, k, r_max, r, every):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd = np.float64 if mode == "fp64" else np.float32
    td = torch.float64 if mode == "fp64" else torch.float32
    counts = [2, 3, 8, 5, 1, 7, 17, 9]
    A64 = synth.gaussian_matrix(n, seed=n + k, config=2)
    Us, Vs = synth.update_factors(n, r, sum(counts), seed=n + r, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, nd)
    U, V = dev(Us, td), dev(Vs, td)
    a, b = _pair(lv, A, td, {"fp64": lv.LV_FP64, "fp32": lv.LV_FP32, "shadow": lv.LV_FP32_BF16SHADOW}[mode], k, r_max,
                 every)
    t = 0
    for c in counts:
        a.update_batch(U[t:t + c], V[t:t + c])
        for s in range(t, t + c):
            b.update(U[s], V[s])
        t += c
        for p in a.powers():
            same = torch.equal(a.read(p), b.read(p))
            assert same, f"P_{p} after a batch of {c} ({t} updates)"
    assert a.stats()["updates"] == t and a.stats()["drift_checks"] == b.stats()["drift_checks"]
    note(f"{mode} n={n} k={k} r={r}/{r_max} every={every}: {t} updates equal")
    a.close()
    b.close()

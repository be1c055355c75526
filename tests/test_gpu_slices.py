"""Row slices of the level passes at the default tile rows: orders around the
padding granule and the sizes where the slice count changes, with updates of
the view's largest rank and of a lower one (whose passes are cut into more
slices), against the FP64 oracle.  Tolerances as tests/test_gpu_parity.py:
1e-10 (FP64), 1e-4 (FP32), 5e-3 (bfloat16 shadows)."""

from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import synth
from tests.gpu_util import dev, need_gpu, note, read_all, storage_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,n,k,r_max", [("fp64", 1, 4, 1), ("fp64", 256, 16, 8), ("fp64", 257, 4, 4),
                                            ("fp32", 255, 16, 1), ("fp32", 512, 8, 8), ("fp32", 1281, 8, 4),
                                            ("fp32", 2303, 4, 16), ("shadow", 300, 8, 4), ("shadow", 1025, 4, 32)])
def test_default_slices(mode, n, k, r_max):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd = np.float64 if mode == "fp64" else np.float32
    td = torch.float64 if mode == "fp64" else torch.float32
    A64 = synth.gaussian_matrix(n, seed=n, config=2)
    Us, Vs = synth.update_factors(n, r_max, 4, seed=n, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, nd)
    view = lv.View(dev(A, td), k, r_max=r_max,
                   mode={"fp64": lv.LV_FP64, "fp32": lv.LV_FP32, "shadow": lv.LV_FP32_BF16SHADOW}[mode])
    P = O.reeval(A, k)
    for t in range(4):
        r = r_max if t % 2 == 0 else max(1, r_max // 4)
        view.update(dev(Us[t][:, :r], td), dev(Vs[t][:, :r], td))
        P = O.apply_updates(P, Us[t:t + 1, :, :r], Vs[t:t + 1, :, :r])
    got = read_all(view)
    tol = {"fp64": 1e-10, "fp32": 1e-4, "shadow": 5e-3}[mode]
    for i in P:
        err = O.maxrel(got[i], P[i])
        note(f"{mode} n={n} r_max={r_max} P_{i}: {err:.2e}")
        assert err < tol, f"P_{i}"
    view.close()

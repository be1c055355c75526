"""Wide products of the linear general form (p > 64), whose summation range is
split over several work-groups: the smallest order, one and several column
tiles, and a p wide enough for a single share.  Whole-number operands whose
sums stay below 2^24 must come out exact."""

from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import synth
from tests.gpu_util import dev, host, need_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strategy", [0, 1])
@pytest.mark.parametrize("n,p,dtype", [(70, 65, "f32"), (257, 128, "f64"), (700, 79, "f32"), (1300, 300, "f32"),
                                       (600, 4000, "f32")])
def test_wide_products_exact(n, p, dtype, strategy):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    td = torch.float64 if dtype == "f64" else torch.float32
    g = synth.rng(21, 0, n, p)
    k = 3
    A = (g.random((n, n)) < 2.0 / n).astype(np.float64)
    T0 = g.integers(-3, 4, size=(n, p)).astype(np.float64)
    B = g.integers(-3, 4, size=(n, p)).astype(np.float64)
    view = lv.GLin(dev(A, td), k, dev(T0, td), dev(B, td), r_max=2, strategy=strategy)
    for _ in range(2):
        U = (g.random((n, 2)) < 3.0 / n).astype(np.float64)
        V = (g.random((n, 2)) < 3.0 / n).astype(np.float64)
        view.update(dev(U, td), dev(V, td))
        A = A + U @ V.T
    ref = O.reeval_general_lin(A, T0, B, k)
    assert max(np.abs(x).max() for x in ref.values()) < 2 ** 20
    for i in ref:
        np.testing.assert_array_equal(host(view.read(i)), ref[i], err_msg=f"T_{i}")
    note(f"exact: n={n} p={p} {dtype} strategy {strategy}")
    view.close()

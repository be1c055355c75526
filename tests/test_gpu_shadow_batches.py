"""Batches of updates with bfloat16 shadows, whose levels up to rank 32 take
two or four updates per pass (View.update_batch): every level rank, chunks of
every remainder, ranks below the view's largest, ragged orders, other tile
heights, and orders whose scratch is too small for the shared pass.  A batch
must equal the same updates applied one by one bit for bit, and the shadows it
leaves must be those of its powers (a second batch reads them)."""

from __future__ import annotations

import numpy as np
import pytest

import synth
from tests.gpu_util import dev, need_gpu, note, storage_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,r_max,r,tiles", [
    (256, 16, 4, 4, 0), (300, 64, 1, 1, 0), (513, 32, 2, 2, 0), (700, 16, 4, 3, 320), (1030, 16, 4, 1, 0),
    (520, 8, 8, 8, 256), (768, 8, 16, 16, 0), (1300, 4, 32, 32, 448), (600, 4, 32, 17, 0), (256, 4, 128, 20, 0),
    (2050, 16, 8, 5, 1024)])
def test_batches_equal_single_updates(n, k, r_max, r, tiles):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    counts = [4, 1, 9, 2, 7]
    A64 = synth.gaussian_matrix(n, seed=n + k, config=2)
    Us, Vs = synth.update_factors(n, r, sum(counts), seed=n + r, config=2)
    A, Us, Vs = storage_inputs(A64, Us, Vs, np.float32)
    U, V = dev(Us, torch.float32), dev(Vs, torch.float32)
    a, b = [lv.View(dev(A, torch.float32), k, r_max=r_max, mode=lv.LV_FP32_BF16SHADOW) for _ in range(2)]
    if tiles:
        for v in (a, b):
            v.set_tile_rows([tiles] * len(v.tile_rows()))
    t = 0
    for c in counts:
        a.update_batch(U[t:t + c], V[t:t + c])
        for s in range(t, t + c):
            b.update(U[s], V[s])
        t += c
        for p in a.powers():
            assert torch.equal(a.read(p), b.read(p)), f"P_{p} after a batch of {c} ({t} updates)"
    note(f"n={n} k={k} r={r}/{r_max}: {t} updates equal")
    a.close()
    b.close()

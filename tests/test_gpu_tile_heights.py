"""512-row tiles beside the default's finer cut: they can be set, a tuning
file's 512 means them, and a view's heights can be copied to another one."""

from __future__ import annotations

import json

import pytest

import synth
from tests.gpu_util import dev, need_gpu, note, storage_inputs

import numpy as np

pytestmark = pytest.mark.gpu


def _inputs(n, r, nd):
    A64 = synth.gaussian_matrix(n, seed=n, config=2)
    Us, Vs = synth.update_factors(n, r, 3, seed=n, config=2)
    return storage_inputs(A64, Us, Vs, nd)


def _equal(a, b):
    import torch
    return all(torch.equal(a.read(p), b.read(p)) for p in a.powers())


@pytest.mark.parametrize("mode,n,r", [("fp32", 512, 1), ("fp64", 300, 2), ("fp64", 512, 1)])
def test_512_rows_are_one_tile_of_a_small_matrix(mode, n, r):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    nd, td = (np.float64, torch.float64) if mode == "fp64" else (np.float32, torch.float32)
    code = lv.LV_FP64 if mode == "fp64" else lv.LV_FP32
    A, Us, Vs = _inputs(n, r, nd)
    views = [lv.View(dev(A, td), 8, r_max=r, mode=code) for _ in range(4)]
    explicit, whole, default, copy = views
    assert default.tile_rows() == [512] * 3
    explicit.set_tile_rows([lv.LV_TILE_ROWS_512] * 3)
    whole.set_tile_rows([1024] * 3)           # up to 512 rows, a single tile too
    copy.set_tile_rows([256] * 3)
    copy.set_tile_rows(default.tile_rows())
    assert explicit.tile_rows() == [lv.LV_TILE_ROWS_512] * 3
    for t in range(3):
        for v in views:
            v.update(dev(Us[t], td), dev(Vs[t], td))
    assert _equal(explicit, whole)
    assert _equal(default, copy)
    note(f"{mode} n={n} r={r}: 512 rows equal one tile")
    for v in views:
        v.close()


def test_heights_of_a_tuning_file(tmp_path):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    n, td = 512, torch.float32
    A, Us, Vs = _inputs(n, 1, np.float32)
    lv.lv_tune_cache_clear()
    first = lv.View(dev(A, td), 8)
    lv.Batch([first]).close()
    path = tmp_path / "tiles.json"
    lv.lv_tune_cache_save(str(path))
    path.write_text(json.dumps({key: 512 for key in json.loads(path.read_text())}))
    lv.lv_tune_cache_clear()
    lv.lv_tune_cache_load(str(path))
    view, whole = [lv.View(dev(A, td), 8) for _ in range(2)]
    batch = lv.Batch([view])
    lv.lv_tune_cache_save(str(path))
    assert set(json.loads(path.read_text()).values()) == {512}
    lv.lv_tune_cache_clear()
    assert view.tile_rows() == [lv.LV_TILE_ROWS_512] * 3
    whole.set_tile_rows([1024] * 3)
    for t in range(3):
        batch.stage(0, dev(Us[t], td), dev(Vs[t], td))
        batch.update()
        whole.update(dev(Us[t], td), dev(Vs[t], td))
    assert _equal(view, whole)
    batch.close()
    for v in (first, view, whole):
        v.close()

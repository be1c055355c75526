"""Steps of the linear and skip models and of the linear general form at the
widths where their passes change: 8 columns (the widest vector step), 16 and
more (matrix cores for floats, 16-column chunks for doubles, operands whose
row stride is wider than they are), orders and powers whose workspace limits
the slices, and double products whose summation range is split.  Tolerances
and checks as in test_gpu_models.py and test_gpu_glin.py."""

from __future__ import annotations

import pytest

from tests import test_gpu_glin as glin
from tests import test_gpu_models as models

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,k,s,n,r,dtype", [
    ("skip", 16, 4, 520, 2, "f32"), ("lin", 6, 0, 300, 16, "f64"), ("skip", 16, 8, 300, 2, "f64"),
    ("lin", 4, 0, 300, 32, "f32"), ("lin", 2, 0, 257, 1, "f64"), ("lin", 3, 0, 512, 8, "f64"),
    ("exp", 8, 0, 300, 16, "f64"), ("exp", 8, 0, 700, 8, "f32"), ("skip", 6, 2, 1030, 7, "f32")])
def test_model_widths(model, k, s, n, r, dtype):
    models.test_models_track_oracle(model, k, s, n, r, dtype)


@pytest.mark.parametrize("strategy,n,k,r,p,dtype", [
    (2, 300, 8, 8, 3, "f32"), (2, 513, 5, 8, 1, "f64"), (2, 257, 5, 16, 5, "f64"), (2, 600, 8, 16, 40, "f32"),
    (2, 300, 4, 32, 130, "f32"), (2, 300, 2, 64, 2, "f64"), (2, 300, 1, 16, 7, "f32"),
    (0, 1000, 3, 2, 130, "f64"), (1, 1000, 3, 2, 130, "f64"), (0, 700, 4, 1, 32, "f64"), (1, 260, 3, 9, 200, "f64")])
def test_general_form_widths(strategy, n, k, r, p, dtype):
    glin.test_glin_tracks_oracle(strategy, n, k, r, p, dtype)

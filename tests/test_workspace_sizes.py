"""Workspace sizes do not grow: programs hold fixed workspaces, arenas and
memory budgets.  The sizes below are those of passes with 512-row slices and
one update at a time; what later passes need beyond them has to find room in
regions that lie idle during an update."""

from __future__ import annotations

import pytest

# (m, n, p, mode) -> bytes
OLS = [((256, 256, 1, 0), 3238400), ((600, 300, 4, 0), 13943552), ((1024, 1024, 1, 1), 42310400),
       ((8192, 4096, 16, 1), 746504960), ((1500, 700, 64, 0), 35882496)]


@pytest.fixture(scope="module")
def lib():
    from paper_1403_6968_amd import linview
    return linview.load()


@pytest.mark.parametrize("args,most", OLS)
def test_ols(lib, args, most):
    assert 0 < lib.lv_ols_footprint(*args) <= most

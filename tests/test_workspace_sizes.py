"""Workspace sizes do not grow: programs hold fixed workspaces, arenas and
memory budgets.  The sizes below are those of passes with 512-row slices and
one update at a time; what later passes need beyond them has to find room in
regions that lie idle during an update."""

from __future__ import annotations

import pytest

# (m, n, p, mode) -> bytes
OLS = [((256, 256, 1, 0), 3238400), ((600, 300, 4, 0), 13943552), ((1024, 1024, 1, 1), 42310400),
       ((8192, 4096, 16, 1), 746504960), ((1500, 700, 64, 0), 35882496)]

# (n, k, r_max, mode, model, s) -> bytes
CHAIN = [((300, 1, 8, 0, 1, 0), 2457856), ((300, 2, 4, 0, 2, 2), 4588544), ((300, 1, 8, 1, 1, 0), 1163520),
         ((512, 2, 1, 0, 1, 0), 4292864), ((512, 4, 1, 0, 1, 0), 8626432), ((1024, 12, 1, 0, 1, 0), 104777728),
         ((4096, 12, 1, 1, 1, 0), 1221959680), ((700, 16, 2, 0, 2, 4), 32243712), ((1500, 8, 16, 1, 2, 2), 120913920),
         ((65536, 3, 32, 0, 1, 0), 180640284672), ((600, 16, 8, 0, 0, 0), 38043648)]

# (n, k, r_max, mode, p, strategy) -> bytes
GLIN = [((2048, 1, 1, 0, 200, 0), 63340544), ((2048, 4, 1, 0, 200, 1), 84312064), ((1024, 1, 1, 1, 1000, 0), 54689792),
        ((1024, 16, 1, 1, 1, 0), 12714240), ((1024, 16, 1, 0, 16, 1), 12732416), ((65536, 1, 1, 0, 64, 2), 34898190848),
        ((1024, 1, 1, 1, 64, 2), 14983680), ((5000, 16, 1, 1, 16, 2), 337260544), ((700, 4, 2, 0, 7, 0), 5580288),
        ((500, 3, 4, 0, 1000, 2), 36802560), ((500, 9, 2, 1, 130, 1), 13678592), ((300, 2, 64, 0, 4096, 2), 148897792)]

# (n, k, r_max, mode, flags) -> bytes
VIEW = [((256, 16, 1, 0, 0), 3069440), ((512, 16, 1, 0, 0), 11565056), ((512, 2, 1, 0, 0), 4260608),
        ((512, 4, 8, 0, 0), 7750144), ((1024, 8, 3, 0, 0), 38554112), ((8192, 16, 1, 0, 0), 2790086144),
        ((512, 16, 1, 1, 0), 9940992), ((1024, 16, 1, 1, 0), 39001344), ((8192, 16, 1, 1, 0), 2453460480),
        ((1, 256, 2, 1, 0), 12532992), ((7157, 16, 32, 2, 0), 3257770496), ((1500, 16, 4, 2, 0), 112586240),
        ((300, 4, 8, 0, 1), 14389760), ((1024, 16, 3, 1, 1), 80933376), ((2000, 1, 5, 0, 0), 33997312)]
# (n, k, r_max, mode, p, strategy, s) -> bytes
GENERAL = [((300, 4, 8, 0, 7, 0, 0), 14963200), ((1024, 16, 3, 1, 7, 0, 0), 81818112),
           ((1024, 2, 16, 0, 1, 1, 0), 49111552), ((4096, 16, 1, 1, 1000, 1, 0), 1494935040),
           ((1024, 16, 1, 0, 64, 1, 4), 67992576), ((700, 16, 2, 2, 130, 1, 8), 55794176),
           ((2500, 16, 1, 0, 33, 0, 0), 601020416)]


@pytest.fixture(scope="module")
def lib():
    from paper_1403_6968_amd import linview
    return linview.load()


@pytest.mark.parametrize("args,most", OLS)
def test_ols(lib, args, most):
    assert 0 < lib.lv_ols_footprint(*args) <= most


@pytest.mark.parametrize("args,most", CHAIN)
def test_chain(lib, args, most):
    got = lib.lv_chain_footprint(*args)
    assert 0 < got <= most
    assert got <= lib.lv_chain_footprint_full(*args) <= 1.5 * got


@pytest.mark.parametrize("args,most", GLIN)
def test_linear_general_form(lib, args, most):
    got = lib.lv_glin_footprint(*args)
    assert 0 < got <= most
    assert got <= lib.lv_glin_footprint_full(*args) <= 2.1 * got


@pytest.mark.parametrize("args,most", VIEW)
def test_view(lib, args, most):
    got = lib.lv_view_footprint_ex(*args)
    assert 0 < got <= most
    assert got <= lib.lv_view_footprint_full(*args) <= 1.25 * got
    if args[3] != 0:   # the squaring scratch holds the finer cut
        assert lib.lv_view_footprint_full(*args) == got


@pytest.mark.parametrize("args,most", GENERAL)
def test_general_form(lib, args, most):
    got = lib.lv_view_footprint_general(*args)
    assert 0 < got <= most
    assert got <= lib.lv_view_footprint_general_full(*args) <= 1.25 * got
    if args[3] != 0:
        assert lib.lv_view_footprint_general_full(*args) == got

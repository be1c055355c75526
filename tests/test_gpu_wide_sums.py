"""Sums of the level passes from bfloat16 factors (shadow mode, level ranks 64
and up) over long ranges: a float chain may not run over thousands of terms,
however few work-groups the order asks for.

Whole-number operands whose first half of every sum is positive and whose
second half takes it back: 2048 terms stay below 2^24, so every product of the
update is exact as long as no float chain is longer, and a longer one loses
its lowest digits on the way up.  And Gaussian operands at an order with long
ranges against 64 bits, with the mode's bound."""

from __future__ import annotations

import pytest

from tests.gpu_util import need_gpu, note

pytestmark = pytest.mark.gpu


def _delta(A, U, V):
    """The change of A^2 under A += U V^T, in 64 bits."""
    A, U, V = A.double(), U.double(), V.double()
    W = V.T.contiguous()
    return U @ (A.T.contiguous() @ V).T.contiguous() + (A @ U + U @ (W @ U)) @ W


@pytest.mark.parametrize("side", ["X", "Y"])
@pytest.mark.parametrize("n,r", [(12288, 64), (12288, 128), (4000, 64)])
def test_long_sums_exact(n, r, side):
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    g = torch.Generator(device="cuda").manual_seed(n + r)
    whole = lambda *shape: torch.randint(86, 90, shape, generator=g, device="cuda").float()
    A = whole(n, n)
    A[(slice(n // 2, None) if side == "Y" else (slice(None), slice(n // 2, None)))] *= -1
    dense, unit = whole(n, r), torch.eye(n, r, device="cuda")
    dense[:r] = dense[-r:] = 0   # V^T U = 0: the factors are [U, A U] and [A^T V, V]; halves of one length
    U, V = (unit, dense) if side == "Y" else (dense, unit)
    assert 2048 * 89 * 89 < 2 ** 24 < 4096 * 86 * 86
    view = lv.View(A, 2, r_max=r, mode=lv.LV_FP32_BF16SHADOW)
    view.write(2, torch.zeros(n, n, device="cuda"))
    view.update(U, V)
    ref = _delta(A, U, V)
    assert ref.abs().max() < 2 ** 24
    # the split products of the top update carry 17 bits of a factor
    assert (A.double() @ U.double()).abs().max() < 2 ** 17
    assert (A.double().T.contiguous() @ V.double()).abs().max() < 2 ** 17
    bad = (view.read(2).double() - ref).abs().max().item()
    note(f"{side} n={n} r={r}: largest error {bad}")
    assert bad == 0
    view.close()


def test_long_sums_gaussian():
    torch = need_gpu()
    from paper_1403_6968_amd import linview as lv
    n, r = 8192, 64
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn(n, n, generator=g, device="cuda") * (0.45 / n ** 0.5)
    U, V = (torch.randn(n, r, generator=g, device="cuda") * (1e-2 / n ** 0.5) for _ in range(2))
    view = lv.View(A, 2, r_max=r, mode=lv.LV_FP32_BF16SHADOW)
    view.write(2, torch.zeros(n, n, device="cuda"))
    view.update(U, V)
    ref = _delta(A, U, V)
    err = ((view.read(2).double() - ref).abs().max() / ref.abs().max()).item()
    note(f"n={n} r={r}: max error {err:.2e} of the largest entry")
    assert err < 5e-3
    view.close()

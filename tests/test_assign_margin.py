"""The margin below which a(n) by matrix products leaves an item to the defined sums, against the worst case of
every rounding that is made (host arithmetic; no GPU)."""
import ctypes

import numpy as np
import pytest

from paper_1808_03969_amd import binding

U = 2.0 ** -24  # unit roundoff of fp32


def bf16(x):
    """fp32 -> bf16 -> fp32, to nearest, ties to even."""
    b = x.view(np.uint32)
    return ((b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


@pytest.fixture(scope="module")
def left_out():
    """Largest share of x c that hi hi' + lo hi' + hi lo' leaves out, over all significands of fp32."""
    x = (np.arange(1 << 23, dtype=np.uint32) | 0x3F800000).view(np.float32)
    hi = bf16(x)
    lo = bf16(x - hi)
    rest = np.abs((x - hi) - lo)  # exact: both differences are
    lo, rest = float(np.max(np.abs(lo) / x)), float(np.max(rest / x))
    return lo * lo + 2 * rest + rest * rest, lo + rest


@pytest.mark.parametrize("M,Ds", [(M, Ds) for M in range(4, 65, 4) for Ds in (1, 2, 3, 4, 5, 6, 8, 9, 12, 16, 20, 25, 32) if M * Ds <= 128])
def test_margin_covers_every_rounding(M, Ds, left_out):
    f = binding.load_library().rii_internal_assign_margin
    f.restype, f.argtypes = ctypes.c_float, [ctypes.c_int, ctypes.c_int]
    share, lo = left_out
    Dp = (M * Ds + 31) // 32 * 32
    # B = X^2 + C^2 = 1: X C <= 1/2; C^2 + 2 X C is largest at tan(2 phi) = 2
    partial = max(np.sin(t) ** 2 + 2 * (1 + 2 * lo) * np.sin(t) * np.cos(t) for t in np.linspace(0, np.pi / 2, 100001))
    score = 2 * share * 0.5 + 3 * Dp * 2 * U * partial + (Dp / 4 + 3) * U
    defined = 2 * (Ds + M + 2) * U
    moved = 4.01 * U  # both sides' coordinates, rounded once more when the origin is moved: 2 |x - c| u (X + C)
    assert f(M, Ds) * (1 - 1e-5) >= 2 * (score + defined + moved)

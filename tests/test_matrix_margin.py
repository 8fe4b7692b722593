"""The margin of the batched scan's filter by matrix products against the worst case of every rounding that is made (host
arithmetic; no GPU).  In units of u = 2^-24, per sub-space in terms of r (largest |residual|), n (|qh|^2) and b (largest |c|^2),
with |table entry| <= r + n + 2.01 b and 2 |qh . ch| <= n + 1.01 b, and the magnitude the margin is taken of being
2 r + 4.1 n + 7.1 b.  A row is lost only if the roundings below, all at their worst, exceed the margin."""
import ctypes

import numpy as np
import pytest

from paper_1808_03969_amd import binding

U = 2.0 ** -24


@pytest.mark.parametrize("M,Ds", [(M, Ds) for M in range(4, 65, 4) for Ds in range(1, 33) if M * Ds <= 128])
def test_margin_covers_every_rounding(M, Ds):
    f = binding.load_library().rii_internal_matrix_margin
    f.restype, f.argtypes = ctypes.c_float, [ctypes.c_int, ctypes.c_int]
    r, n, b = np.eye(3)
    entry, dot2 = r + n + 2.01 * b, n + 1.01 * b
    steps = (M * Ds + 31) // 32 * 32 + 1  # additions of the products and the start value, 2 u each (rounded or cut off), halved scale
    products = 2 * steps * (entry + r + dot2)        # twice (|tau - lo| / 2 + sum |qh ch|), 2 u
    residual = (2 * Ds + 2) * (entry + b + dot2)     # entry - b, then an addition per coordinate, 2 u (the products are exact)
    extremes = (M + 1) * r                           # lo and hi: M additions, and the margin's own
    distance = M * entry                             # the defined sum
    row = M * b                                      # B: M additions of the book's numbers, or
    row = np.maximum(row, 2 * steps * 1.01 * b + Ds * b)  # the squares of the row's coordinates added up, 2 u, against the book's sums of Ds
    start = 2 * (entry + r)                          # (tau - lo) / 2 and its factor
    worst = products + residual + extremes + distance + row + start
    share = float(np.max(worst / np.array([2, 4.1, 7.1]))) * U
    assert f(M, Ds) * (1 - 1e-5) >= share
    # the first bounds: twice (B / 2 + sum |qh ch|) in the products, and B
    first = 2 * steps * (b + dot2) + residual + extremes + distance + row + start
    assert f(M, Ds) * (1 - 1e-5) >= float(np.max(first / np.array([2, 4.1, 7.1]))) * U

"""Edges of the kernels' size ranges -- remainders, the smallest and largest sizes of a variant, the
lines of the dispatch rules -- against the CPU oracle.  The bar is that of the parity tests:
identifiers bit-exact, and distances bit-identical, because both sides perform the same fp32 operations
in the same order."""
import numpy as np
import pytest
import torch

from helpers import t2n

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rii():
    import paper_1808_03969_amd as r
    r.load_library()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return r


# every unrolled width, widths between them, and batches below, at and past a multiple of the queries per block
@pytest.mark.parametrize("Ds,M,Q", [(1, 8, 1), (2, 16, 257), (3, 32, 130), (4, 4, 700), (5, 12, 3), (6, 16, 1025), (8, 64, 97),
                                    (12, 8, 300), (16, 8, 2063), (20, 4, 9)])
def test_tables_over_widths_and_batches(Ds, M, Q, rii, oracle_lib):
    rng = np.random.default_rng(100 * Ds + M)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    q = rng.normal(size=(Q, M * Ds)).astype(np.float32)
    lut = rii.rii_build_lut(rii.Index(cb), torch.from_numpy(q).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(t2n(lut), oracle_lib.lut(cb, q))

"""The launches for queries that the scan by matrix products leaves: whatever their number turns out to be on the device,
their blocks are within the grid and their candidates within the scratch (host arithmetic; no GPU)."""
import ctypes

import pytest

from paper_1808_03969_amd import binding


@pytest.mark.parametrize("per", [1, 2, 4])
@pytest.mark.parametrize("rows", [262_144, 300_001, 1_000_000, 30_000_001, 1_000_000_000])
@pytest.mark.parametrize("Q,big", [(64, 1), (129, 1), (256, 1), (600, 1), (2044, 1), (2045, 3), (2499, 7), (10_000, 24)])
def test_blocks_and_lists_fit(per, rows, Q, big):
    lib = binding.load_library()
    chunks, blocks, lists = lib.rii_internal_left_chunks, lib.rii_internal_left_blocks, lib.rii_internal_left_lists
    for f, n in ((chunks, 4), (blocks, 3), (lists, 2)):
        f.restype = ctypes.c_int64
    chunks.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64, ctypes.c_int64]
    blocks.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int64]
    lists.argtypes = [ctypes.c_int64, ctypes.c_int64]
    # a batch's last piece has fewer queries and the same scratch and chunks (the grid is its own)
    for piece in (Q, max(1, Q // 2 + 1)):
        grid, places = blocks(per, piece, big), lists(Q, big)
        for n in range(1, piece + 1):
            groups = (n + per - 1) // per
            c = chunks(per, groups, rows, big)
            tile = 4096
            step = -(-(-(-rows // c)) // tile) * tile
            c = -(-rows // step)
            assert 1 <= c and groups * c <= grid
            assert n * c <= places or (c == 1 and n <= places)


def test_parts_of_left_list_queries_fit():
    """Blocks that queries left by the lists' products get: within the grid (one a query of the batch, 256 at least; 256 where k_few
    takes more than 64 of them), which is also what their candidates have room for."""
    parts = binding.load_library().rii_internal_ivf_left_parts
    parts.restype, parts.argtypes = ctypes.c_int64, [ctypes.c_int64]
    for n in list(range(1, 600)) + [4095, 4096, 65_535]:
        assert 1 <= parts(n) and n * parts(n) <= max(n, 256)
        assert n <= 256 or parts(n) == 1
    assert parts(1) >= 16 and parts(64) == 4

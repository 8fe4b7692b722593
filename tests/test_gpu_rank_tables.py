"""Queries through the lists, the tables made by the ranking, against the steps one by one (rii_build_lut's tables, which other tests compare
with the oracle): widths with a kernel of their own, batches on both sides of the chip's size, more lists than a block has threads."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,Ds,N,K,Q,topk,L", [(64, 2, 20_001, 300, 33, 10, 400), (64, 2, 20_001, 1_100, 300, 100, 999), (32, 3, 20_000, 70, 1, 100, 3_000),
                                               (32, 4, 5_000, 2_049, 257, 7, 50), (16, 4, 30_000, 40, 700, 129, 5_000), (8, 1, 4_000, 9, 260, 1, 1),
                                               (12, 2, 9_000, 33, 5, 20, 2_000)])
def test_query_equals_its_steps(M, Ds, N, K, Q, topk, L):
    import paper_1808_03969_amd as rii
    rng = np.random.default_rng(M * K)
    index = rii.Index(rng.standard_normal((M, 256, Ds)).astype(np.float32))
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    index.add(codes)
    index.build_lists(codes[rng.permutation(N)[:K]].copy())
    q = torch.from_numpy(rng.standard_normal((Q, M * Ds)).astype(np.float32)).cuda()
    ids, dist = rii.rii_query(index, q, topk, L=L)
    lut = rii.rii_build_lut(index, q)
    probe, _ = rii.rii_coarse_assign(index, lut, min(K, -(-K * L // N)))
    ref = rii.rii_adc_scan_ivf(index, lut, probe, topk, L=L)
    assert torch.equal(ids, ref[0]) and torch.equal(dist, ref[1])

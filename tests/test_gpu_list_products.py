"""The inverted index in batches, lists by matrix products, against the kernels of one query a block (the same call in small
batches, which are theirs) and the CPU oracle: identifiers and distances bit for bit."""
import ctypes

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


def make(rii, M, Ds, N, lengths, kind, seed):
    """An index of N random codes in lists of the given lengths (members spread over the identifiers)."""
    rng = np.random.default_rng(seed)
    cb = rng.standard_normal((M, 256, Ds)).astype(np.float32)
    if kind == "far":
        cb += 30.0
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    if kind == "clustered":  # a few dozen different codes
        codes = codes[rng.integers(0, 48, N)]
    if kind == "one":        # more members within the bound than a query's list has places
        codes[:] = codes[0]
    K = len(lengths)
    a = rng.permutation(np.repeat(np.arange(K), lengths))
    assert len(a) == N
    order = np.argsort(a, kind="stable").astype(np.int32)
    off = np.zeros(K + 1, np.int64)
    off[1:] = np.cumsum(lengths)
    index = rii.Index(cb)
    index.add(codes)
    coarse = rng.integers(0, 256, (K, M), dtype=np.uint8)
    index.set_lists(coarse, off, order)
    return index, codes, off, order, rng


def bytes_held(index):
    return index.info()["device_bytes"]


def both(rii, index, lut, probe, topk, L):
    """The batch in one call, which has to take the products' scratch, and a hundred queries at a time, which must not."""
    parts = [rii.rii_adc_scan_ivf(index, lut[i:i + 100].contiguous(), probe[i:i + 100].contiguous(), topk, L=L) for i in range(0, lut.shape[0], 100)]
    ref = torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
    before = bytes_held(index)
    ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, topk, L=L)
    torch.cuda.synchronize()
    assert bytes_held(index) > before + lut.shape[0] * 8192  # (list and groups of a query)
    assert torch.equal(ids, ref[0]) and torch.equal(dist, ref[1])
    return t2n(ids), t2n(dist)


# every kernel there is; batches that leave the last query tile and stage short, lists of less than a wave, of whole and of ragged
# tiles, an empty one and one of most members; one result to the most; caps inside a list, inside a block of 32 and at its edge;
# codes shared by hundreds of members; code words far from the origin
CASES = [
    (16, 8, 20_000, 20, 2107, 8, 100, "normal", 0), (16, 8, 20_000, 20, 2200, 8, 128, "normal", 7777),
    (16, 4, 40_011, 40, 2100, 9, 1, "normal", 0), (16, 6, 20_003, 7, 1500, 4, 10, "clustered", 0),
    (32, 2, 30_000, 15, 2050, 5, 100, "far", 0), (32, 3, 20_001, 20, 2305, 8, 37, "normal", 7200),
    (32, 4, 33_000, 33, 2111, 8, 100, "clustered", 0), (64, 2, 20_000, 16, 1433, 6, 100, "normal", 7008),
    (64, 2, 20_032, 16, 1400, 6, 1, "normal", 0), (12, 8, 20_000, 20, 1111, 8, 100, "normal", 0),
    (8, 8, 20_000, 20, 3300, 8, 20, "normal", 0), (8, 12, 20_000, 20, 3111, 8, 60, "clustered", 0),
    (8, 16, 20_000, 9, 3200, 4, 100, "normal", 8191), (16, 8, 60_000, 6, 700, 3, 100, "one", 0),
]


@pytest.mark.parametrize("M,Ds,N,K,Q,nprobe,topk,kind,L", CASES)
def test_whole_batches(rii, oracle_lib, M, Ds, N, K, Q, nprobe, topk, kind, L):
    rng = np.random.default_rng(Q)
    lengths = np.full(K, N // K)
    lengths[0] += N - lengths.sum()
    lengths[1] -= 31
    lengths[2] += 31                       # ragged ones
    if K > 10:
        lengths[3] += lengths[4] + lengths[5] - 1
        lengths[4], lengths[5] = 0, 1      # an empty one, one of a single member
    index, codes, off, order, rng = make(rii, M, Ds, N, lengths, kind, Q)
    q = torch.from_numpy(rng.standard_normal((Q, M * Ds)).astype(np.float32) + (30.0 if kind == "far" else 0.0)).cuda()
    lut = rii.rii_build_lut(index, q)
    # the first three lists are probed by most queries, so that they fill several stages
    probe = np.stack([rng.permutation(K)[:nprobe] for _ in range(Q)]).astype(np.int32)
    for i in range(0, Q, 2):
        probe[i] = np.concatenate([np.arange(3), 3 + rng.permutation(K - 3)])[:nprobe][rng.permutation(nprobe)]
    ids, dist = both(rii, index, lut, torch.from_numpy(probe).cuda(), topk, L)
    A = t2n(lut[:2])
    for i in range(2):  # the definition, in numpy
        rows = np.concatenate([order[off[l]:off[l + 1]] for l in probe[i]])[:L or None]
        d = np.zeros(len(rows), np.float32)
        for m in range(M):
            d += A[i, m][codes[rows, m]]
        best = np.lexsort((rows, d))[:topk]
        assert np.array_equal(ids[i], rows[best]) and np.array_equal(dist[i], d[best])


def test_lists_named_twice_and_queries_left_over(rii):
    """Lists that a query names twice count twice; numbers that are no list count as empty ones in the products only, so they are not
    tested; tables that no query made, not finite ones among them, go query by query."""
    index, codes, off, order, rng = make(rii, 16, 8, 20_000, np.full(20, 1000), "normal", 3)
    q = torch.from_numpy(rng.standard_normal((2200, 128)).astype(np.float32)).cuda()
    lut = rii.rii_build_lut(index, q)
    lut[5] = torch.rand_like(lut[5])
    lut[77] = -lut[77]
    lut[2199] = 0.0
    lut[100, 3, 7] = float("nan")
    lut[101, 15, 255] = float("inf")
    probe = torch.from_numpy(rng.integers(0, 20, (2200, 9)).astype(np.int32)).cuda()
    probe[9] = 4
    both(rii, index, lut, probe, 100, 0)


def test_no_room_and_most_tables_left(rii):
    """A device without room for the scratch: query by query.  More than three eighths of the tables made by no query: nothing is
    multiplied, all of them go query by query."""
    index, codes, off, order, rng = make(rii, 32, 3, 20_000, np.full(20, 1000), "normal", 4)
    q = torch.from_numpy(rng.standard_normal((2300, 96)).astype(np.float32)).cuda()
    lut = rii.rii_build_lut(index, q)
    probe = torch.from_numpy(np.stack([rng.permutation(20)[:8] for _ in range(2300)]).astype(np.int32)).cuda()
    room = rii.load_library().rii_internal_matrix_room
    room.restype, room.argtypes = None, [ctypes.c_void_p, ctypes.c_size_t]
    room(index.handle, 1 << 16)
    before = bytes_held(index)
    rii.rii_adc_scan_ivf(index, lut[:100].contiguous(), probe[:100].contiguous(), 100)
    small = rii.rii_adc_scan_ivf(index, lut, probe, 100)
    held = bytes_held(index)
    assert held < before + (8 << 20)
    room(index.handle, (1 << 64) - 1)
    both(rii, index, lut, probe, 100, 0)
    again = rii.rii_adc_scan_ivf(index, lut, probe, 100)
    assert torch.equal(again[0], small[0]) and torch.equal(again[1], small[1])
    lut[::2] = torch.rand_like(lut[::2])
    parts = [rii.rii_adc_scan_ivf(index, lut[i:i + 100].contiguous(), probe[i:i + 100].contiguous(), 100) for i in range(0, 2300, 100)]
    out = rii.rii_adc_scan_ivf(index, lut, probe, 100)
    assert torch.equal(out[0], torch.cat([p[0] for p in parts])) and torch.equal(out[1], torch.cat([p[1] for p in parts]))


def test_query_and_graph(rii):
    """rii_query by the lists, with its cap, against small batches; a captured call, replayed on other queries."""
    rng = np.random.default_rng(8)
    cb = rng.standard_normal((16, 256, 8)).astype(np.float32)
    index = rii.Index(cb)
    index.add(rng.integers(0, 256, (50_001, 16), dtype=np.uint8))
    index.reconfigure(50, iters=1, seed=1)
    q = torch.from_numpy(rng.standard_normal((2500, 128)).astype(np.float32)).cuda()
    whole = rii.rii_query(index, q, 100, L=7_500)
    parts = [rii.rii_query(index, q[i:i + 100].contiguous(), 100, L=7_500) for i in range(0, 2500, 100)]
    assert torch.equal(whole[0], torch.cat([p[0] for p in parts])) and torch.equal(whole[1], torch.cat([p[1] for p in parts]))
    none = rii.rii_query_noalloc(index, q[:1000].contiguous(), 100, L=7_500)
    assert torch.equal(none[0], whole[0][:1000])
    lut = rii.rii_build_lut(index, q)
    probe, _ = rii.rii_coarse_assign(index, lut, 8)
    out = rii.rii_adc_scan_ivf(index, lut, probe, 100)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        held = rii.rii_adc_scan_ivf(index, lut, probe, 100)
    for turn in range(3):
        lut.copy_(lut.roll(1, 0))
        probe.copy_(probe.roll(1, 0))
        out = out[0].roll(1, 0), out[1].roll(1, 0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(held[0], out[0]) and torch.equal(held[1], out[1]), turn
        eager = rii.rii_adc_scan_ivf(index, lut, probe, 100)
        torch.cuda.synchronize()
        assert torch.equal(eager[0], out[0])


# Queries that the products leave share the chip: none, one, some, as many as k_few does not take, more, all of them; lists of so many members that
# the streaming kernel would have the batch, and fewer of them (k_few's); a cap inside a list
@pytest.mark.parametrize("M,Ds,N,K,Q,nprobe,topk,L", [(16, 4, 1_200_003, 8, 300, 2, 10, 0), (8, 8, 1_200_000, 8, 420, 2, 128, 290_001), (32, 3, 900_000, 6, 300, 2, 10, 0),
                                                      (64, 2, 600_000, 5, 150, 2, 10, 0), (12, 8, 600_001, 5, 200, 2, 20, 0),
                                                      (16, 8, 400_000, 16, 800, 2, 100, 0), (32, 4, 320_000, 16, 700, 2, 100, 39_990),
                                                      (12, 8, 400_000, 16, 500, 2, 64, 0)])
def test_left_queries_share_the_chip(rii, M, Ds, N, K, Q, nprobe, topk, L):
    from paper_1808_03969_amd import binding
    lengths = np.full(K, N // K)
    lengths[0] += N - lengths.sum()
    index, codes, off, order, rng = make(rii, M, Ds, N, lengths, "normal", Q)
    lut = rii.rii_build_lut(index, torch.from_numpy(rng.standard_normal((Q, M * Ds)).astype(np.float32)).cuda())
    foreign = torch.from_numpy(rng.random((Q, M, 256)).astype(np.float32)).cuda() * lut.mean() * 2
    probe = torch.from_numpy(np.stack([rng.permutation(K)[:nprobe] for _ in range(Q)]).astype(np.int32)).cuda()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    binding.rii_index_set_scan_events(index, ev[0].cuda_event, ev[1].cuda_event)
    for left in (0, 1, 3, 33, 64, 65, Q * 3 // 8, Q):
        mixed = lut.clone()
        at = torch.from_numpy(np.sort(rng.permutation(Q)[:left])).cuda()
        mixed[at] = foreign[at]
        parts = [rii.rii_adc_scan_ivf(index, mixed[i:i + 10].contiguous(), probe[i:i + 10].contiguous(), topk, L=L) for i in range(0, Q, 10)]
        binding.rii_index_read_scan_counters(index)
        ids, dist = rii.rii_adc_scan_ivf(index, mixed, probe, topk, L=L)
        torch.cuda.synchronize()
        # (with more than three eighths of the tables foreign nothing is multiplied)
        assert binding.rii_index_read_scan_counters(index)[5] == (left if left <= Q * 3 // 8 else Q)
        assert torch.equal(ids, torch.cat([p[0] for p in parts])) and torch.equal(dist, torch.cat([p[1] for p in parts])), left
    binding.rii_index_set_scan_events(index, None, None)


# Queries whose bound thousands of members share (copies of one code): more listed than are scored one a thread, up to what a list of candidates
# holds and past it, in batches of few queries (several blocks for such a list) and of many
@pytest.mark.parametrize("M,Ds,N,K,Q,topk,copies", [(16, 4, 200_000, 5, 420, 10, 250), (16, 4, 200_000, 5, 420, 10, 12_000), (16, 8, 200_000, 5, 430, 100, 16_000),
                                                    (16, 8, 200_000, 5, 430, 100, 17_000), (8, 8, 200_000, 5, 700, 10, 5_000), (32, 3, 200_000, 5, 300, 128, 9_000),
                                                    (64, 2, 200_000, 5, 200, 1, 15_000), (12, 8, 200_000, 5, 200, 100, 8_000), (16, 4, 200_000, 5, 2_600, 10, 7_000)])
def test_long_lists_of_candidates(rii, M, Ds, N, K, Q, topk, copies):
    from paper_1808_03969_amd import binding
    rng = np.random.default_rng(M + copies)
    cb = rng.standard_normal((M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 256, (N, M), dtype=np.uint8)
    a = rng.permutation(np.repeat(np.arange(K), N // K))
    codes[rng.permutation(np.nonzero(a == 0)[0])[:copies]] = codes[0]
    off = np.arange(K + 1, dtype=np.int64) * (N // K)
    index = rii.Index(cb)
    index.add(codes)
    index.set_lists(codes[:K].copy(), off, np.argsort(a, kind="stable").astype(np.int32))
    q = rng.standard_normal((Q, M * Ds)).astype(np.float32)
    q[::7] = np.concatenate([cb[m][codes[0][m]] for m in range(M)]) + 0.01 * q[::7]
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    probe = torch.from_numpy(np.stack([np.append(0, 1 + rng.permutation(K - 1)[:1]) for _ in range(Q)]).astype(np.int32)).cuda()
    parts = [rii.rii_adc_scan_ivf(index, lut[i:i + 10].contiguous(), probe[i:i + 10].contiguous(), topk) for i in range(0, Q, 10)]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    binding.rii_index_set_scan_events(index, ev[0].cuda_event, ev[1].cuda_event)
    before = bytes_held(index)
    for _ in range(2):
        binding.rii_index_read_scan_counters(index)
        ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, topk)
        torch.cuda.synchronize()
        left = binding.rii_index_read_scan_counters(index)[5]
        assert 0 <= left - (len(q[::7]) if copies > 16_384 else 0) <= 8  # (others that happen to be near the copies)
        assert bytes_held(index) > before
        assert torch.equal(ids, torch.cat([p[0] for p in parts])) and torch.equal(dist, torch.cat([p[1] for p in parts]))
    binding.rii_index_set_scan_events(index, None, None)


# both sides of the line from which a batch goes by products: long lists (M = 8 and 16 take more queries there), many short ones (M = 16, M = 64)
@pytest.mark.parametrize("M,Ds,N,K,nprobe,below,above", [(8, 8, 260_000, 20, 4, 1000, 1070), (16, 4, 260_000, 20, 4, 630, 670),
                                                         (64, 2, 100_000, 1000, 50, 3600, 3850), (16, 4, 100_000, 1000, 50, 4300, 4600)])
def test_line_of_the_rule(rii, M, Ds, N, K, nprobe, below, above):
    index, codes, off, order, rng = make(rii, M, Ds, N, np.full(K, N // K), "normal", K)
    lut = rii.rii_build_lut(index, torch.from_numpy(rng.standard_normal((above, M * Ds)).astype(np.float32)).cuda())
    probe = torch.from_numpy(np.stack([rng.permutation(K)[:nprobe] for _ in range(above)]).astype(np.int32)).cuda()
    small = rii.rii_adc_scan_ivf(index, lut[:below].contiguous(), probe[:below].contiguous(), 10)
    torch.cuda.synchronize()
    before = bytes_held(index)
    ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, 10)
    torch.cuda.synchronize()
    assert bytes_held(index) > before + above * 8192
    assert torch.equal(ids[:below], small[0]) and torch.equal(dist[:below], small[1])
    index.close()
    index, *_ = make(rii, M, Ds, N, np.full(K, N // K), "normal", K)
    before = bytes_held(index)
    rii.rii_adc_scan_ivf(index, lut[:below].contiguous(), probe[:below].contiguous(), 10)
    torch.cuda.synchronize()
    assert bytes_held(index) < before + below * 8192  # (scratch of the look-ups)


# Probes so long that the members the bound is taken of are a small part: without places for what it lists all queries would be left
@pytest.mark.parametrize("M,Ds,K,nprobe,Q,topk,L", [(16, 4, 20, 20, 60, 128, 0), (8, 8, 16, 16, 120, 100, 0), (32, 2, 40, 40, 50, 128, 3_900_001)])
def test_bound_of_a_small_part(rii, M, Ds, K, nprobe, Q, topk, L):
    from paper_1808_03969_amd import binding
    index, codes, off, order, rng = make(rii, M, Ds, 4_000_000, np.full(K, 4_000_000 // K), "normal", K)
    lut = rii.rii_build_lut(index, torch.from_numpy(rng.standard_normal((Q, M * Ds)).astype(np.float32)).cuda())
    probe = torch.from_numpy(np.stack([rng.permutation(K)[:nprobe] for _ in range(Q)]).astype(np.int32)).cuda()
    parts = [rii.rii_adc_scan_ivf(index, lut[i:i + 10].contiguous(), probe[i:i + 10].contiguous(), topk, L=L) for i in range(0, Q, 10)]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    binding.rii_index_set_scan_events(index, ev[0].cuda_event, ev[1].cuda_event)
    before = bytes_held(index)
    binding.rii_index_read_scan_counters(index)
    ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, topk, L=L)
    torch.cuda.synchronize()
    assert binding.rii_index_read_scan_counters(index)[5] <= Q // 10
    binding.rii_index_set_scan_events(index, None, None)
    assert bytes_held(index) > before + Q * 65_536
    assert torch.equal(ids, torch.cat([p[0] for p in parts])) and torch.equal(dist, torch.cat([p[1] for p in parts]))


# Lists of candidates of as many rounds of a block as one does by itself, one more, and none more than the first
@pytest.mark.parametrize("M,Ds,copies", [(16, 4, 5_900), (16, 4, 6_400), (16, 4, 900), (32, 3, 6_000), (32, 3, 6_400), (12, 8, 2_900), (12, 8, 3_300)])
def test_lists_of_candidates_for_one_block(rii, M, Ds, copies):
    test_long_lists_of_candidates(rii, M, Ds, 200_000, 5, 420, 10, copies)

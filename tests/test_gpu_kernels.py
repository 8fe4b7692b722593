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


def plain_index(rii, oracle, rng, N, M, K, Ds=2, repeat=None):
    """Random code books and codes with K coarse centres; `repeat`: that many copies of one centre."""
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    if repeat:
        coarse[rng.permutation(K)[:repeat]] = coarse[0]
    a = rng.integers(0, K, size=N).astype(np.int32)
    off, lids = oracle.build_lists(a, K)
    index = rii.Index(cb)
    index.add(codes)
    index.set_lists(coarse, off, lids)
    return dict(cb=cb, codes=codes, coarse=coarse, off=off, lids=lids, index=index)


# few / many queries (one large block or several small ones to a CU), few queries over many centres
# (distances computed by a kernel of their own), all centres asked for, equal distances at the cut --
# fewer and more of them than the block can sort
@pytest.mark.parametrize("M,K,Q,n,repeat", [(8, 1, 3, 1, 0), (16, 97, 300, 97, 0), (12, 1000, 5, 64, 0), (32, 8192, 32, 100, 0),
                                            (32, 8192, 33, 256, 0), (64, 9000, 2, 1024, 0), (64, 16384, 257, 1000, 0),
                                            (16, 3000, 300, 10, 200), (8, 4096, 270, 8, 4000), (16, 4096, 7, 300, 4096)])
def test_ranking_of_lists(M, K, Q, n, repeat, rii, oracle_lib):
    rng = np.random.default_rng(K + Q)
    d = plain_index(rii, oracle_lib, rng, 2000, M, K, repeat=repeat)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    ids, d0 = rii.rii_coarse_assign(d["index"], rii.rii_build_lut(d["index"], torch.from_numpy(q).cuda()), n)
    torch.cuda.synchronize()
    A = oracle_lib.lut(d["cb"], q)
    for i in range(0, Q, max(1, Q // 9)):
        ref = oracle_lib.coarse_rank(A[i], d["coarse"], n)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(d0)[i], ref[1]), i


# every number of matrix steps with and without a coordinate to spare, the width past them; batches below, at
# and past a wave's 64 vectors and a grid's worth of them; code words that coincide or differ by a
# rounding (decided by the defined sums), vectors that are code words, that are huge, tiny or infinite
@pytest.mark.parametrize("Ds,M,n", [(1, 8, 65), (2, 64, 1000), (3, 32, 63), (4, 5, 64), (5, 12, 1), (6, 16, 20011), (8, 16, 50003),
                                    (12, 8, 129), (13, 3, 700), (16, 8, 40000), (20, 4, 300)])
def test_encode_over_widths_and_ties(Ds, M, n, rii, oracle_lib):
    rng = np.random.default_rng(Ds * 1000 + M)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    cb[:, 200] = cb[:, 17]
    cb[:, 90] = np.nextafter(cb[:, 91], np.float32(np.inf))
    cb[0] = np.round(cb[0] * 4)  # a grid: exact ties
    x = rng.normal(size=(n, M * Ds)).astype(np.float32)
    x[::7] = np.round(x[::7] * 2) / 2
    x[::5] = cb[np.arange(M), rng.integers(0, 256, size=((n + 4) // 5, M))].reshape(-1, M * Ds)
    if n > 40:
        x[3] *= np.float32(1e18)
        x[11] *= np.float32(1e-25)
        x[12] = 0
        x[22, Ds // 2] = np.inf
        x[31, :] = -np.inf
    ref = oracle_lib.encode(cb, x)
    buf = torch.empty(n * M * Ds + 1, dtype=torch.float32, device="cuda")
    for shift in (0, 1):  # vectors at an address that is a multiple of 16, and of 4 only
        xd = buf[shift:shift + n * M * Ds].view(n, M * Ds)
        xd.copy_(torch.from_numpy(x))
        got = rii.rii_encode_device(rii.Index(cb), xd)
        torch.cuda.synchronize()
        assert np.array_equal(t2n(got), ref), shift


# few rows (below, at and past a block) and many, every number of outputs per thread, inner tiles with and
# without a remainder, several blocks of outputs
@pytest.mark.parametrize("D,n", [(1, 5), (16, 32), (17, 33), (64, 1), (128, 1000), (300, 77), (32, 65536), (33, 65500), (90, 66001),
                                 (128, 65409), (129, 32770), (200, 33000)])
def test_rotation_over_dimensions(D, n, rii, oracle_lib):
    rng = np.random.default_rng(D)
    R = rng.normal(size=(D, D)).astype(np.float32)
    x = rng.normal(size=(n, D)).astype(np.float32)
    x[n // 2] = -0.0
    y = rii.rii_rotate(torch.from_numpy(R).cuda(), torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    ref = oracle_lib.rotate(R, x)
    assert np.array_equal(t2n(y).view(np.uint32), ref.view(np.uint32))


# rounds of 1024 rows: below, at and past one and several; one block a query and several (few queries, and
# many rounds); all lists of keys the block sorts or ranks; `copies`: that many rows share a code, so that
# whole keys and not only distances decide what the buffer keeps
@pytest.mark.parametrize("M,N,Q,topk,copies", [(4, 1, 3, 5, 1), (8, 1023, 300, 10, 1), (16, 1024, 2, 100, 1), (16, 1025, 257, 100, 1),
                                               (16, 5000, 1, 128, 1), (32, 8193, 5, 1000, 1), (64, 20000, 300, 1, 1),
                                               (12, 30011, 20, 100, 1), (16, 60000, 130, 300, 1), (8, 9000, 40, 100, 3000),
                                               (16, 9000, 260, 100, 9000), (32, 7000, 2, 600, 3500)])
def test_small_scans(M, N, Q, topk, copies, rii, oracle_lib):
    rng = np.random.default_rng(N + Q)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    if copies > 1:
        codes = codes[rng.integers(0, max(1, N // copies), size=N)]
    K = max(1, min(40, N // 50))
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    # lists of very different lengths, the second one empty
    off, lids = oracle_lib.build_lists(np.where(rng.random(N) < .3, 0, rng.integers(min(2, K - 1), K, size=N)).astype(np.int32), K)
    index = rii.Index(cb)
    index.add(codes)
    index.set_lists(coarse, off, lids)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    qd = torch.from_numpy(q).cuda()
    lut = rii.rii_build_lut(index, qd)
    A = oracle_lib.lut(cb, q)
    # target sets: none, one identifier, all, a few, many; sorted
    sizes = [[0, 1, N, N // 50, N // 3][i % 5] for i in range(Q)]
    sets = [np.sort(rng.permutation(N)[:s]).astype(np.int32) for s in sizes]
    toff = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)])).cuda()
    tids = torch.from_numpy(np.concatenate(sets + [np.zeros(1, np.int32)])).cuda()
    nprobe = (K + 1) // 2
    probe, _ = rii.rii_coarse_assign(index, lut, nprobe)
    got = dict(linear=rii.rii_adc_scan_linear(index, lut, topk),
               subset=rii.rii_adc_scan_subset(index, lut, tids, toff, N, topk),
               lists=rii.rii_adc_scan_ivf(index, lut, probe, topk),
               first=rii.rii_adc_scan_ivf(index, lut, probe, topk, L=N // 3 + 1),
               members=rii.rii_adc_scan_ivf(index, lut, probe, topk, tids, toff),
               capped=rii.rii_adc_scan_ivf(index, lut, probe, topk, tids, toff, L=N // 9 + 1))
    index.set_threshold(N // 10)
    got["query"] = rii.rii_query(index, qd, topk, tids, toff, N, L=max(1, N // K))
    torch.cuda.synchronize()
    got = {n: (t2n(i), t2n(d)) for n, (i, d) in got.items()}
    for i in sorted(set(range(0, Q, max(1, Q // 10))) | {Q - 1}):
        S = sets[i]
        iv = lambda L, S: oracle_lib.inverted_index(A[i], codes, coarse, off, lids, topk, nprobe, Lcap=L, S=S)[:2]
        ref = dict(linear=oracle_lib.linear_scan(A[i], codes, topk), subset=oracle_lib.linear_scan(A[i], codes, topk, S=S),
                   lists=iv(0, None), first=iv(N // 3 + 1, None), members=iv(0, S), capped=iv(N // 9 + 1, S),
                   query=oracle_lib.query(cb, q[i], codes, coarse, off, lids, topk, max(1, N // K), N // 10, S=S)[:2])
        for name, (ids, dist) in ref.items():
            assert np.array_equal(got[name][0][i], ids) and np.array_equal(got[name][1][i], dist), (name, i)


# a(n) by matrix products: every number of steps over the dimension (and a dimension past them), centres below,
# at and past a tile of 16, items at and past a block's; repeated centres and items that lie on a
# centre (ties go to the list of undecided items), code books far from the origin (nearly all do)
@pytest.mark.parametrize("M,Ds,N,K,shift", [(4, 2, 256, 1, 0), (8, 4, 1000, 16, 0), (8, 5, 257, 17, 0), (12, 8, 5001, 33, 0),
                                            (16, 6, 20000, 1000, 0), (32, 4, 3001, 1500, 0), (64, 2, 1025, 40, 0), (16, 9, 900, 30, 0),
                                            (16, 6, 4000, 100, 50)])
def test_assignment_by_matrix_products(M, Ds, N, K, shift, rii, oracle_lib):
    rng = np.random.default_rng(N + K)
    cb = (rng.normal(size=(M, 256, Ds)) + shift).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    coarse[K // 2] = coarse[0]
    codes[::9] = coarse[rng.integers(0, K, size=len(codes[::9]))]
    index = rii.Index(cb)
    index.add(codes[:N - N // 4])
    index.build_lists(coarse)
    index.add(codes[N - N // 4:])  # pushed into the lists: rows of a stored array from a row on
    a = index.get_lists()[3]
    T = oracle_lib.sym_table(cb)
    i = np.unique(np.concatenate([np.arange(0, N, max(1, N * K // 4_000_000)), np.arange(N - 70, N)]))
    assert np.array_equal(a[i], oracle_lib.assign(T, codes[i], coarse))


# posting lists by a counting sort on the device: items below, at and past a wave's 64 and a chunk's 4096, one
# list, as many lists as the block counts, more than that (host path), everything in one list
@pytest.mark.parametrize("N,K,same", [(1, 1, False), (64, 3, False), (4096, 257, False), (4097, 1000, True), (30011, 1024, False),
                                      (70000, 38400, False), (50000, 38401, False)])
def test_lists_from_assignment(N, K, same, rii, oracle_lib):
    rng = np.random.default_rng(N)
    cb = rng.normal(size=(4, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, 4), dtype=np.uint8)
    if same:
        codes[:] = codes[0]
    index = rii.Index(cb)
    index.add(codes[:(N + 1) // 2])
    index.build_lists(rng.integers(0, 256, size=(K, 4), dtype=np.uint8))
    if N > 1:
        index.add(codes[(N + 1) // 2:])
    _, off, ids, a = index.get_lists()
    ref_off, ref_ids = oracle_lib.build_lists(a, K)
    assert np.array_equal(off, ref_off) and np.array_equal(ids, ref_ids)


def test_reconfigure_centres_are_the_best_codes(rii, oracle_lib):
    """One round of the clustering (the sample is the whole database): the new centre of a cell is, per
    sub-space, the code with the smallest sum of table entries over the members, lowest on ties."""
    rng = np.random.default_rng(6)
    N, M, K = 3000, 8, 30
    cb = rng.normal(size=(M, 256, 3)).astype(np.float32)
    cb[:, 200] = cb[:, 10]
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    codes[:40] = codes[0]
    T = oracle_lib.sym_table(cb)
    index = rii.Index(cb)
    index.add(codes)
    index.reconfigure(K, iters=0, seed=3)
    start, _, _, a = index.get_lists()
    assert np.array_equal(a, oracle_lib.assign(T, codes, start))
    index.reconfigure(K, iters=1, seed=3)
    want = start.copy()
    for k in range(K):
        for m in range(M):
            h = np.bincount(codes[a == k, m], minlength=256)
            if h.sum():
                want[k, m] = np.argmin(np.cumsum(np.concatenate([[np.zeros(256)], h[:, None] * T[m].astype(np.float64)]), axis=0)[-1])
    assert np.array_equal(index.get_lists()[0], want)


# the query procedure without target sets takes one branch for the whole batch: the batched scan, two queries a
# block, one query; the lists; and the threshold above the database size
@pytest.mark.parametrize("M,N,Q,topk,K,theta", [(16, 150_003, 301, 10, 0, 0), (8, 120_001, 2100, 110, 0, 0), (32, 110_000, 3, 100, 0, 0),
                                                (16, 3000, 9, 20, 12, 0), (16, 3000, 9, 20, 12, 4000)])
def test_query_without_target_sets(M, N, Q, topk, K, theta, rii, oracle_lib):
    rng = np.random.default_rng(N)
    d = plain_index(rii, oracle_lib, rng, N, M, max(K, 1))
    index = d["index"]
    if not K:  # an index that has no lists
        index = rii.Index(d["cb"])
        index.add(d["codes"])
    index.set_threshold(theta)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    qd = torch.from_numpy(q).cuda()
    L = max(1, N // max(K, 1))
    ids, dist = rii.rii_query(index, qd, topk, L=L)
    torch.cuda.synchronize()
    A = oracle_lib.lut(d["cb"], q)
    for i in range(0, Q, max(1, Q // 8)):
        if K:
            ref = oracle_lib.query(d["cb"], q[i], d["codes"], d["coarse"], d["off"], d["lids"], topk, L, theta)
        else:
            ref = oracle_lib.linear_scan(A[i], d["codes"], topk)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), i


# tables that a caller made: entries of either sign where the scans take any (the sums of 64 and of other numbers of
# sub-spaces are formed row by row), in every form of the small scan, topk small enough for a bound early on
@pytest.mark.parametrize("M,N,Q", [(64, 5000, 3), (64, 20000, 2), (12, 5000, 3)])
def test_small_scans_with_signed_tables(M, N, Q, rii, oracle_lib):
    rng = np.random.default_rng(N + M)
    d = plain_index(rii, oracle_lib, rng, N, M, 6)
    A = rng.normal(size=(Q, M, 256)).astype(np.float32)
    lut = torch.from_numpy(A).cuda()
    sets = [np.sort(rng.permutation(N)[:N // 2]).astype(np.int32) for _ in range(Q)]
    tids = torch.from_numpy(np.concatenate(sets)).cuda()
    toff = torch.arange(Q + 1).cuda() * (N // 2)
    probe, _ = rii.rii_coarse_assign(d["index"], lut, 6)
    got = dict(linear=rii.rii_adc_scan_linear(d["index"], lut, 5),
               subset=rii.rii_adc_scan_subset(d["index"], lut, tids, toff, N // 2, 5),
               lists=rii.rii_adc_scan_ivf(d["index"], lut, probe, 5),
               capped=rii.rii_adc_scan_ivf(d["index"], lut, probe, 5, tids, toff, L=N // 3))
    torch.cuda.synchronize()
    for i in range(Q):
        iv = lambda L, S: oracle_lib.inverted_index(A[i], d["codes"], d["coarse"], d["off"], d["lids"], 5, 6, Lcap=L, S=S)[:2]
        ref = dict(linear=oracle_lib.linear_scan(A[i], d["codes"], 5), subset=oracle_lib.linear_scan(A[i], d["codes"], 5, S=sets[i]),
                   lists=iv(0, None), capped=iv(N // 3, sets[i]))
        for name, (ids, dist) in ref.items():
            assert np.array_equal(t2n(got[name][0])[i], ids) and np.array_equal(t2n(got[name][1])[i], dist), (name, i)


# a query that is not a number in one coordinate, beside ordinary ones: at 8, 16 and 32 sub-spaces such distances are no
# candidates (as in the streaming kernels), else they come after all others with their identifiers in order; one block a
# query over several rounds (300 queries) and several blocks, the coordinate in the first and in the last sub-space,
# either sign
@pytest.mark.parametrize("M,N,Q,topk", [(8, 3000, 4, 10), (16, 9000, 4, 100), (32, 2500, 4, 20), (64, 9000, 4, 100), (64, 5000, 300, 100),
                                        (12, 9000, 4, 100)])
def test_small_scans_of_a_query_that_is_not_a_number(M, N, Q, topk, rii, oracle_lib):
    rng = np.random.default_rng(M)
    d = plain_index(rii, oracle_lib, rng, N, M, 6)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    q[1, 2 * M - 1], q[2, 0], q[3, M] = np.nan, np.nan, np.inf
    q[1, 2 * M - 1] = np.copysign(q[1, 2 * M - 1], np.float32(-1 if M in (8, 16, 32) else 1))
    lut = rii.rii_build_lut(d["index"], torch.from_numpy(q).cuda())
    got = rii.rii_adc_scan_linear(d["index"], lut, topk)
    probe = torch.arange(6, dtype=torch.int32).repeat(Q, 1).cuda()
    lists = rii.rii_adc_scan_ivf(d["index"], lut, probe, topk)
    torch.cuda.synchronize()
    A = oracle_lib.lut(d["cb"], q)
    ref = oracle_lib.linear_scan(A[0], d["codes"], topk)
    for ids, dist in (got, lists):
        ids, dist = t2n(ids), t2n(dist)
        assert np.array_equal(ids[0], ref[0]) and np.array_equal(dist[0], ref[1])
        for i in (1, 2):
            if M in (8, 16, 32):
                assert np.all(ids[i] == -1) and np.all(np.isinf(dist[i])), i
            else:
                assert np.array_equal(ids[i], np.arange(topk)) and np.all(np.isnan(dist[i])), i
        assert np.array_equal(ids[3], np.arange(topk)) and np.all(np.isposinf(dist[3]))


# a table that starts at any float of a larger array
@pytest.mark.parametrize("M", [8, 12, 16, 32, 64])
def test_small_scans_of_a_table_at_any_float(M, rii, oracle_lib):
    rng = np.random.default_rng(M)
    d = plain_index(rii, oracle_lib, rng, 3000, M, 50)
    A = oracle_lib.lut(d["cb"], rng.normal(size=(2, 2 * M)).astype(np.float32))
    for shift in (1, 2, 3):
        buf = torch.empty(A.size + shift, dtype=torch.float32, device="cuda")
        lut = buf[shift:].view(A.shape)
        lut.copy_(torch.from_numpy(A))
        ids, dist = rii.rii_adc_scan_linear(d["index"], lut, 10)
        lists, d0 = rii.rii_coarse_assign(d["index"], lut, 7)
        torch.cuda.synchronize()
        for i in range(2):
            ref = oracle_lib.linear_scan(A[i], d["codes"], 10)
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (shift, i)
            ref = oracle_lib.coarse_rank(A[i], d["coarse"], 7)
            assert np.array_equal(t2n(lists)[i], ref[0]) and np.array_equal(t2n(d0)[i], ref[1]), (shift, i)


# centres in pairs whose distances to every item differ by some 10^-4 of them and less, on both sides of what the
# matrix products may decide; code books of 8, 32 and 128 coordinates
@pytest.mark.parametrize("M,Ds,N,K", [(4, 2, 3000, 40), (8, 4, 3000, 300), (16, 8, 3000, 600)])
def test_assignment_between_centres_that_nearly_coincide(M, Ds, N, K, rii, oracle_lib):
    rng = np.random.default_rng(N + M)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    cb[:, 1::2] = cb[:, ::2] * (1 + rng.choice([1e-6, 1e-5, 1e-4, 1e-3], size=(M, 128, 1)) * rng.normal(size=(M, 128, Ds)))
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    coarse[1::2] = coarse[::2]
    coarse[np.arange(1, K, 2), rng.integers(0, M, size=K // 2)] ^= 1
    index = rii.Index(cb)
    index.add(codes)
    index.build_lists(coarse)
    assert np.array_equal(index.get_lists()[3], oracle_lib.assign(oracle_lib.sym_table(cb), codes, coarse))


# enough items and centres for the undecided ones to be counted, and centres of which none, some or all occur twice: few
# items undecided (by the defined sums one by one), many (by the pruned search), most (which takes all items then); the
# same with too few centres to be counted.  Code books away from the origin.
@pytest.mark.parametrize("N,K,twice", [(530_000, 2050, 0.0), (1_700_000, 2050, 0.4), (530_000, 2050, 1.0), (530_000, 560, 1.0)])
def test_assignment_with_many_undecided_items(N, K, twice, rii, oracle_lib):
    rng = np.random.default_rng(K)
    M = 16
    cb = (rng.normal(size=(M, 256, 2)) + 30).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    n2 = int(twice * K) // 2
    coarse[K - n2:] = coarse[:n2]
    index = rii.Index(cb)
    index.add(codes)
    index.build_lists(coarse)
    a = index.get_lists()[3]
    brute = rii.rii_assign(index, torch.from_numpy(codes).cuda(), torch.from_numpy(coarse).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(a, t2n(brute))
    some = rng.integers(0, N, size=500)
    assert np.array_equal(a[some], oracle_lib.assign(oracle_lib.sym_table(cb), codes[some], coarse))


# the pruned search on its own: dimensions past the matrix products', and a few items added to many lists
@pytest.mark.parametrize("M,Ds,K,few", [(16, 9, 1100, 0), (32, 6, 1500, 3), (12, 12, 1024, 0), (16, 6, 1024, 200), (64, 2, 2000, 255)])
def test_pruned_assignment(M, Ds, K, few, rii, oracle_lib):
    rng = np.random.default_rng(K)
    N = 3000
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 16, size=(N, M), dtype=np.uint8) + np.repeat(rng.integers(0, 15, size=(N // 50, M), dtype=np.uint8) * 16, 50, axis=0)
    coarse = codes[rng.permutation(N)[:K]].copy()
    coarse[7] = coarse[3]
    index = rii.Index(cb)
    index.add(codes[:N - few])
    index.build_lists(coarse)
    if few:
        index.add(codes[N - few:])
    assert np.array_equal(index.get_lists()[3], oracle_lib.assign(oracle_lib.sym_table(cb), codes, coarse))


# many results from few rows: the blocks of a query hand over as many keys as the batch's scratch has room for, also
# where the scratch has a fixed size; one query in many blocks, many queries in few, every way to the rows
@pytest.mark.parametrize("M,N,Q,topk", [(16, 60000, 1, 1000), (64, 60000, 3, 700), (12, 65536, 70, 300), (32, 50001, 16, 1024), (8, 65000, 200, 500)])
def test_small_scans_with_many_results(M, N, Q, topk, rii, oracle_lib):
    from paper_1808_03969_amd import binding
    rng = np.random.default_rng(N + M)
    d = plain_index(rii, oracle_lib, rng, N, M, 4)
    index = d["index"]
    assert Q > 64 or binding.rii_scan_linear_plan(index, Q, topk)[1] >= 4  # (one block a query leaves the chip idle)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    qd = torch.from_numpy(q).cuda()
    lut = rii.rii_build_lut(index, qd)
    sets = [np.sort(rng.permutation(N)[:N - 7 * i]).astype(np.int32) for i in range(Q)]
    tids = torch.from_numpy(np.concatenate(sets)).cuda()
    toff = torch.from_numpy(np.concatenate([[0], np.cumsum([len(s) for s in sets])])).cuda()
    probe, _ = rii.rii_coarse_assign(index, lut, 4)
    index.reserve_workspace(Q, topk, N, 4)
    held = index.info()["device_bytes"]
    got = dict(linear=rii.rii_adc_scan_linear(index, lut, topk), subset=rii.rii_adc_scan_subset(index, lut, tids, toff, N, topk),
               lists=rii.rii_adc_scan_ivf(index, lut, probe, topk), query=rii.rii_query(index, qd, topk, L=N),
               fixed=rii.rii_query_noalloc(index, qd, topk, L=N))
    torch.cuda.synchronize()
    assert index.info()["device_bytes"] == held
    A = oracle_lib.lut(d["cb"], q)
    for i in sorted({0, Q // 2, Q - 1}):
        whole = oracle_lib.linear_scan(A[i], d["codes"], topk)
        for name, (ids, dist) in got.items():
            ref = oracle_lib.linear_scan(A[i], d["codes"], topk, S=sets[i]) if name == "subset" else whole
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (name, i)


# a batch whose small scans' room would exceed the scratch of a fixed size: they get less of it
def test_small_scans_in_a_scratch_of_a_fixed_size(rii, oracle_lib):
    rng = np.random.default_rng(77)
    M, N, Q, topk = 64, 30000, 760, 100  # 50 MB of tables, 62 MB with the hand-over area of its size
    d = plain_index(rii, oracle_lib, rng, N, M, 3)
    index = rii.Index(d["cb"])
    index.add(d["codes"])
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    ids, dist = rii.rii_query_noalloc(index, torch.from_numpy(q).cuda(), topk)
    torch.cuda.synchronize()
    for i in (0, 400, Q - 1):
        ref = oracle_lib.linear_scan(oracle_lib.lut(d["cb"], q[i:i + 1])[0], d["codes"], topk)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), i


# lists of very different lengths: half of all members in one, a quarter in another, the rest short or empty; queries
# that probe none, one or both of the long ones, in one block a query and in several, on both sides of the lines
@pytest.mark.parametrize("M,N,Q,topk", [(16, 60000, 200, 10), (16, 200000, 300, 100), (64, 30000, 5, 1), (32, 30000, 260, 10), (12, 50000, 3, 300)])
def test_scans_of_uneven_lists(M, N, Q, topk, rii, oracle_lib):
    rng = np.random.default_rng(N)
    K = 60
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    u = rng.random(N)
    off, lids = oracle_lib.build_lists(np.where(u < .5, 7, np.where(u < .75, 31, rng.integers(10, K, size=N))).astype(np.int32), K)
    index = rii.Index(cb)
    index.add(codes)
    index.set_lists(coarse, off, lids)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    q[::3] = np.concatenate([cb[m][coarse[7, m]] for m in range(M)]) + 0.1 * q[::3]  # the longest list is the nearest
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    A = oracle_lib.lut(cb, q)
    for P in (1, 2, 20):
        probe, _ = rii.rii_coarse_assign(index, lut, P)
        ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, topk)
        torch.cuda.synchronize()
        for i in range(0, Q, max(1, Q // 7)):
            ref = oracle_lib.inverted_index(A[i], codes, coarse, off, lids, topk, P)[:2]
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (P, i)


# a small scan in several blocks with the scan events set: they are recorded around its kernel, which keeps no tallies,
# and the results are the usual ones
def test_scan_events_of_a_small_scan(rii, oracle_lib):
    from paper_1808_03969_amd import binding
    rng = np.random.default_rng(2)
    d = plain_index(rii, oracle_lib, rng, 60000, 16, 4)
    q = rng.normal(size=(1, 32)).astype(np.float32)
    lut = rii.rii_build_lut(d["index"], torch.from_numpy(q).cuda())
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()  # (makes the handles)
    binding.rii_index_set_scan_events(d["index"], ev[0].cuda_event, ev[1].cuda_event)
    ids, dist = rii.rii_adc_scan_linear(d["index"], lut, 10)
    torch.cuda.synchronize()
    binding.rii_index_set_scan_events(d["index"], None, None)
    assert 0 < ev[0].elapsed_time(ev[1]) < 5
    assert binding.rii_index_read_scan_counters(d["index"]) == [0] * 8
    ref = oracle_lib.linear_scan(oracle_lib.lut(d["cb"], q)[0], d["codes"], 10)
    assert np.array_equal(t2n(ids)[0], ref[0]) and np.array_equal(t2n(dist)[0], ref[1])


# ---- the streaming kernels past the small scans' lines
# every code some 3,200 times: buffers full of equal distances in the kernels for four, two and one query a block,
# whose common bound counts them (four) or that fall back to sorting, and in the block's buffer for many results
@pytest.mark.parametrize("Q,topk,per_block", [(300, 100, 4), (1027, 17, 4), (521, 128, 2), (6, 100, 1), (3, 128, 1), (5, 700, 1)])
def test_streaming_scans_of_repeated_codes(Q, topk, per_block, rii, oracle_lib):
    from paper_1808_03969_amd import binding
    rng = np.random.default_rng(topk)
    M, N = 8, 120_003
    cb = rng.normal(size=(M, 256, 4)).astype(np.float32)
    codes = rng.integers(0, 256, size=(37, M), dtype=np.uint8)[rng.integers(0, 37, size=N)]
    index = rii.Index(cb)
    index.add(codes)
    assert binding.rii_scan_linear_plan(index, Q, topk)[0] == per_block
    q = rng.normal(size=(Q, 4 * M)).astype(np.float32)
    ids, dist = rii.rii_adc_scan_linear(index, rii.rii_build_lut(index, torch.from_numpy(q).cuda()), topk)
    torch.cuda.synchronize()
    A = oracle_lib.lut(cb, q)
    for i in sorted(set(range(0, Q, max(1, Q // 9))) | {Q - 1}):
        ref = oracle_lib.linear_scan(A[i], codes, topk)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), i


# numbers of sub-spaces without a rotated form, and a block's buffer over short shares (16,500 rows, top-1024)
@pytest.mark.parametrize("M,N,Q,topk", [(12, 150_001, 3, 20), (12, 150_001, 40, 128), (12, 100_000, 5, 300), (64, 150_001, 3, 50),
                                        (64, 100_003, 20, 128), (64, 100_003, 5, 400), (16, 66_000, 64, 1024), (32, 66_000, 64, 129)])
def test_streaming_scans_past_the_lines(M, N, Q, topk, rii, oracle_lib):
    rng = np.random.default_rng(N + topk)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    index = rii.Index(cb)
    index.add(codes)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    S = np.sort(rng.permutation(N)[:N - 9]).astype(np.int32)
    tids = torch.from_numpy(np.tile(S, 2)).cuda()
    lin = rii.rii_adc_scan_linear(index, lut, topk)
    sub = rii.rii_adc_scan_subset(index, lut[:2].contiguous(), tids, torch.arange(3).cuda() * len(S), len(S), topk)
    torch.cuda.synchronize()
    A = oracle_lib.lut(cb, q)
    for i in sorted({0, 1, Q // 2, Q - 1}):
        ref = oracle_lib.linear_scan(A[i], codes, topk)
        assert np.array_equal(t2n(lin[0])[i], ref[0]) and np.array_equal(t2n(lin[1])[i], ref[1]), i
        if i < 2:
            ref = oracle_lib.linear_scan(A[i], codes, topk, S=S)
            assert np.array_equal(t2n(sub[0])[i], ref[0]) and np.array_equal(t2n(sub[1])[i], ref[1]), ("subset", i)


# many short lists and empty ones, more members than the small scans take (the streaming kernel for lists) and more lists
# than either keeps prefix sums for (the kernel that walks them one by one); with a target set, with a cap, with both
@pytest.mark.parametrize("M,N,K,P,L,topk", [(8, 400_000, 900, 500, 150_000, 20), (12, 300_000, 900, 700, 150_000, 128),
                                            (64, 300_000, 900, 700, 150_000, 5), (16, 300_000, 900, 600, 130_001, 100),
                                            (8, 40_000, 4_700, 4_300, 9_000, 20), (12, 40_000, 4_700, 4_097, 20_000, 300),
                                            (32, 40_000, 4_700, 4_700, 1_000, 1_000), (64, 30_000, 4_400, 4_200, 9_000, 10)])
def test_scans_of_many_lists(M, N, K, P, L, topk, rii, oracle_lib):
    rng = np.random.default_rng(K + M)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    coarse = rng.integers(0, 256, size=(K, M), dtype=np.uint8)
    off, lids = oracle_lib.build_lists((rng.integers(0, K // 2, size=N) * 2).astype(np.int32), K)  # every other one is empty
    index = rii.Index(cb)
    index.add(codes)
    index.set_lists(coarse, off, lids)
    Q = 4
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    S = np.sort(rng.permutation(N)[:N // 2]).astype(np.int32)
    tids, toff = torch.from_numpy(np.tile(S, Q)).cuda(), torch.arange(Q + 1).cuda() * len(S)
    probe, _ = rii.rii_coarse_assign(index, lut, P)
    A = oracle_lib.lut(cb, q)
    for use_S, cap in ((False, 0), (True, 0), (False, L), (True, L // 3)):
        ids, dist = rii.rii_adc_scan_ivf(index, lut, probe, topk, tids if use_S else None, toff if use_S else None, L=cap)
        torch.cuda.synchronize()
        for i in range(Q):
            ref = oracle_lib.inverted_index(A[i], codes, coarse, off, lids, topk, P, S=S if use_S else None, Lcap=cap)[:2]
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (use_S, cap, i)

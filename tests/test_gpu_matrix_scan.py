"""The batched linear scan by matrix products against the CPU oracle.  The products only decide which rows are scored;
what is returned comes from the defined sums, so identifiers and distances must be the oracle's bit for bit."""
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


def check(rii, oracle, index, lut, codes, topk, at):
    ids, dist = rii.rii_adc_scan_linear(index, lut, topk)
    torch.cuda.synchronize()
    A, ids, dist = t2n(lut), t2n(ids), t2n(dist)
    for i in at:
        ref = oracle.linear_scan(A[i], codes, topk)
        assert np.array_equal(ids[i], ref[0]) and np.array_equal(dist[i], ref[1]), i


def counted(rii, index, call):
    """The call's results and the scan counters it leaves."""
    from paper_1808_03969_amd import binding
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    binding.rii_index_set_scan_events(index, ev[0].cuda_event, ev[1].cuda_event)
    binding.rii_index_read_scan_counters(index)
    out = call()
    torch.cuda.synchronize()
    counters = binding.rii_index_read_scan_counters(index)
    binding.rii_index_set_scan_events(index, None, None)
    return out, counters


def by_look_ups(rii, index, lut, topk):
    """The same queries by the look-up kernels: batches that are too small for the matrix products."""
    from paper_1808_03969_amd import binding
    assert binding.rii_scan_linear_plan(index, 32, topk)[0] != 32
    parts = [rii.rii_adc_scan_linear(index, lut[i:i + 32], topk) for i in range(0, lut.shape[0], 32)]
    return torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])


# every number of matrix steps and every width of the fit, sub-spaces with and without a rotated stored form, two planes,
# the fewest rows and rows that leave the last tile of 512 nearly empty or full, query tiles short and full, one result
# to the most; code words far from the origin, of one value, clustered codes
MATRIX_CASES = [
    (16, 8, 262144, 128, 100, "normal"), (16, 8, 262145, 257, 1, "far"), (32, 3, 300_000, 129, 128, "normal"),
    (32, 3, 400_127, 280, 10, "clustered"), (64, 2, 263_000, 129, 100, "normal"), (12, 8, 524_288, 64, 1000, "normal"),
    (8, 16, 262_655, 261, 50, "flat"), (8, 4, 524_289, 159, 300, "normal"), (4, 32, 524_800, 70, 1024, "normal"),
    (8, 1, 262_200, 130, 100, "normal"), (16, 6, 1_400_003, 256, 100, "clustered"), (12, 5, 262_500, 64, 20, "far"),
    (16, 2, 270_000, 513, 200, "tiny"), (32, 4, 262_200, 160, 64, "huge")]


def matrix_case(rii, M, Ds, N, Q, topk, kind):
    from paper_1808_03969_amd import binding
    rng = np.random.default_rng(N + M)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    q = rng.normal(size=(Q, M * Ds)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    if kind == "far":
        cb += 300.0
        q += 300.0
    size = {"tiny": 1e-12, "huge": 1e9, "small": 1e-8}.get(kind)
    if size:                       # magnitudes at the ends of what the scaling reaches and past it
        cb *= size
        q *= size
        q[1] *= 50.0
    if kind == "flat":
        cb[1] = cb[1, :1]          # a sub-space whose code words are all the same
        cb[2, :, 1:] = 0.5         # one that varies in one coordinate only
    if kind == "clustered":        # rows in the order of their clusters
        proto = rng.integers(0, 256, size=(500, M), dtype=np.uint8)
        codes = np.where(rng.random((N, M)) < 0.2, codes, proto[np.sort(rng.integers(0, 500, size=N))])
    index = rii.Index(cb)
    index.add(codes)
    assert binding.rii_scan_linear_plan(index, Q, topk)[0] == 32
    return index, codes, rii.rii_build_lut(index, torch.from_numpy(q).cuda())


@pytest.mark.parametrize("M,Ds,N,Q,topk,kind", MATRIX_CASES)
def test_matrix_scan(M, Ds, N, Q, topk, kind, rii, oracle_lib):
    index, codes, lut = matrix_case(rii, M, Ds, N, Q, topk, kind)
    check(rii, oracle_lib, index, lut, codes, topk, sorted(set(range(0, Q, max(1, Q // 6))) | {Q - 1}))


# the products decide for every query of these batches (a query that the fit or an empty list handed to the look-up kernels
# would have the right results whatever the products say), and no query's results are another's
@pytest.mark.parametrize("M,Ds,N,Q,topk,kind", MATRIX_CASES + [(16, 2, 270_000, 513, 200, "small")])
def test_products_do_the_work(M, Ds, N, Q, topk, kind, rii):
    index, _, lut = matrix_case(rii, M, Ds, N, Q, topk, kind)
    (ids, dist), counters = counted(rii, index, lambda: rii.rii_adc_scan_linear(index, lut, topk))
    # (1e-12: below what the scaling reaches, nothing is left of the code words in fp16)
    assert (counters[5], counters[6] > 0) == ((Q, False) if kind == "tiny" else (0, True))
    want = by_look_ups(rii, index, lut, topk)
    assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])


# tables that no query made, in a batch with others: random entries, of both signs, all equal, not finite, infinite,
# huge and tiny; and queries far from every code word
@pytest.mark.parametrize("M,topk", [(16, 100), (16, 120), (32, 10), (12, 50), (64, 100)])
def test_tables_that_no_query_made(M, topk, rii, oracle_lib):
    rng = np.random.default_rng(M)
    N, Q = 262_777, 300
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    index = rii.Index(cb)
    index.add(codes)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    q[3] *= 1e4
    q[4] *= 1e-4
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    lut[7] = torch.rand_like(lut[7])
    lut[9] = 3.0
    lut[11] *= 1e20
    lut[12] *= 1e-20
    lut[14] = torch.rand_like(lut[14]) * 100
    lut[15, 0, 7:9] = float("inf")
    lut[16, 1] += 50.0
    check(rii, oracle_lib, index, lut, codes, topk, [0, 3, 4, 6, 7, 8, 9, 10, 11, 12, 14, 15, 16, 17, Q - 1])


# one row over and over: more rows within every query's bound than its list holds
@pytest.mark.parametrize("M,topk", [(8, 100), (32, 128), (64, 10)])
def test_lists_that_overflow(M, topk, rii, oracle_lib):
    rng = np.random.default_rng(M)
    N, Q = 262_144 + 700, 270
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(5, M), dtype=np.uint8)[rng.integers(0, 5, size=N)]
    index = rii.Index(cb)
    index.add(codes)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    check(rii, oracle_lib, index, lut, codes, topk, [0, 1, 33, Q - 1])


# the query procedure takes the same way, within scratch that was reserved (in pieces where it is short: 700 queries' tables
# leave room for half of them), and in a captured graph that is replayed
@pytest.mark.parametrize("Q,topk,reserve", [(270, 20, (300, 200)), (700, 100, (700, 100))])
def test_query_reserved_and_captured(Q, topk, reserve, rii, oracle_lib):
    rng = np.random.default_rng(5)
    M, N = 16, 262_999
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    index = rii.Index(cb)
    index.add(codes)
    index.reserve_workspace(*reserve)
    before = index.info()["device_bytes"]
    q = torch.from_numpy(rng.normal(size=(Q, 2 * M)).astype(np.float32)).cuda()
    want = rii.rii_query(index, q, topk)
    torch.cuda.synchronize()
    assert index.info()["device_bytes"] == before
    for i in (0, 33, Q // 2 + 40, Q - 1):
        ref = oracle_lib.linear_scan(oracle_lib.lut(cb, t2n(q[i:i + 1]))[0], codes, topk)
        assert np.array_equal(t2n(want[0])[i], ref[0]) and np.array_equal(t2n(want[1])[i], ref[1])
    out = (torch.empty_like(want[0]), torch.empty_like(want[1]))
    if reserve[0] != Q:  # an index whose first call of this kind is the captured one
        index = rii.Index(cb)
        index.add(codes)
        index.reserve_workspace(*reserve)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rii.rii_query(index, q, topk, out=out)
    first = rii.rii_query(index, q, topk)  # before any replay
    torch.cuda.synchronize()
    assert torch.equal(first[0], want[0]) and torch.equal(first[1], want[1])
    for _ in range(3):
        out[0].zero_()
        out[1].zero_()
        rii.rii_query(index, q[:3], topk)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], want[0]) and torch.equal(out[1], want[1])


# queries that are left to the look-up kernels: none, one, a part of a group of four, some, more than a round of blocks,
# half, all; every kernel that takes them (four, two and one a block, in row chunks and whole, with and without k_select)
@pytest.mark.parametrize("M,Ds,topk,N", [(16, 2, 100, 262_777), (8, 4, 10, 900_001), (32, 3, 100, 1_200_000), (8, 2, 120, 262_777), (32, 3, 128, 300_000),
                                         (32, 2, 300, 270_001), (64, 2, 100, 262_777), (64, 1, 200, 400_000), (12, 5, 100, 262_777),
                                         (12, 3, 500, 900_001)])
def test_left_over_queries(M, Ds, topk, N, rii):
    rng = np.random.default_rng(M + topk)
    Q = 600
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    index = rii.Index(cb)
    index.add(rng.integers(0, 256, size=(N, M), dtype=np.uint8))
    lut = rii.rii_build_lut(index, torch.from_numpy(rng.normal(size=(Q, M * Ds)).astype(np.float32)).cuda())
    foreign = torch.from_numpy(rng.random((Q, M, 256)).astype(np.float32)).cuda() * lut.mean() * 2
    for left in (0, 1, 3, 70, 290, 600):
        mixed = lut.clone()
        at = torch.from_numpy(np.sort(rng.permutation(Q)[:left])).cuda()
        mixed[at] = foreign[at]
        (ids, dist), counters = counted(rii, index, lambda: rii.rii_adc_scan_linear(index, mixed, topk))
        # (with more than 3/8 or 3/4 of the tables foreign, the others are left with them and nothing is multiplied)
        given_up = left > Q * (3 if topk <= 100 and M in (8, 16, 32) else 6) // 8
        assert counters[5] == (Q if given_up else left) and (counters[6] == 0) == given_up
        want = by_look_ups(rii, index, mixed, topk)
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1]), left


def device_room(index, most):
    """The products' scratch: the device is taken to have room for `most` bytes."""
    from paper_1808_03969_amd import binding
    f = binding.load_library().rii_internal_matrix_room
    f.restype, f.argtypes = None, [ctypes.c_void_p, ctypes.c_size_t]
    f(index.handle, most)


def scratch_case(rii, Q, topk, N=300_000, M=16, Ds=2, seed=3):
    rng = np.random.default_rng(seed)
    index = rii.Index(rng.normal(size=(M, 256, Ds)).astype(np.float32))
    index.add(rng.integers(0, 256, size=(N, M), dtype=np.uint8))
    lut = rii.rii_build_lut(index, torch.from_numpy(rng.normal(size=(Q, M * Ds)).astype(np.float32)).cuda())
    return index, lut, by_look_ups(rii, index, lut, topk)


# a device without room for the products' scratch (pieces within what the look-ups have), with room for a part of it, with room
# for all: larger pieces each time, over all rows; what the look-ups have is kept, and further calls ask for nothing
def test_device_without_room(rii):
    Q, topk = 1100, 100
    index, lut, want = scratch_case(rii, Q, topk)

    def scan():
        (ids, dist), counters = counted(rii, index, lambda: rii.rii_adc_scan_linear(index, lut, topk))
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
        return index.info()["device_bytes"], counters[6]

    start, before = None, 1 << 62
    for most in (0, 24 << 20, 1 << 62):
        device_room(index, most)
        held, blocks = scan()
        start = held if start is None else start
        assert held - start <= min(most, 1 << 30) and (most == 0 or held > start)
        assert 0 < blocks < before
        assert scan() == (held, blocks)
        before = blocks


# a graph of a call by look-ups reads the handle's scratch: the next call with the same arguments, which gets the products'
# scratch, leaves that alone.  A graph of a call by products holds theirs: a larger call does not move it.
def test_graphs_keep_their_scratch(rii):
    Q, topk = 300, 50
    index, lut, want = scratch_case(rii, 1500, topk)
    part, first = lut[:Q].contiguous(), (want[0][:Q], want[1][:Q])
    device_room(index, 0)
    assert counted(rii, index, lambda: rii.rii_adc_scan_linear(index, part, topk))[1][6] == 0
    held = index.info()["device_bytes"]

    def capture():
        out = (torch.empty_like(first[0]), torch.empty_like(first[1]))
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            rii.rii_adc_scan_linear(index, part, topk, out=out)
        return graph, out

    def replay(graph, out):
        for _ in range(3):
            out[0].zero_()
            out[1].zero_()
            got, counters = counted(rii, index, lambda: rii.rii_adc_scan_linear(index, part, topk))
            assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1]) and counters[6] > 0
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out[0], first[0]) and torch.equal(out[1], first[1])

    graphs = [capture()]
    device_room(index, 1 << 62)
    assert index.info()["device_bytes"] == held
    replay(*graphs[0])
    held = index.info()["device_bytes"]
    graphs.append(capture())
    got = rii.rii_adc_scan_linear(index, lut, topk)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    small = 8 * 1500 * (topk + 64 * 128)  # (the look-ups' scratch grew, as it always did, and with it the first graph's went)
    assert index.info()["device_bytes"] <= held + 2 * small
    replay(*graphs[1])


# Rows that collapsed onto few codes: as many as an eighth of the rows share the distance of the bound, and the lists hold them;
# a quarter of them do, and the lists of the queries there run over in a round that is not the first.
@pytest.mark.parametrize("share,left", [(0.02, 0), (0.25, 60)])
def test_collapsed_clusters(share, left, rii):
    M, N, Q, topk, copies = 16, 1_400_003, 260, 10, 2
    rng = np.random.default_rng(8)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    place = rng.random(N)
    for c in range(copies):
        codes[(place >= c * share) & (place < (c + 1) * share)] = codes[c]
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    for i in range(60):  # queries at the two rows
        q[4 * i] = np.concatenate([cb[m][codes[i % copies][m]] for m in range(M)]) + 0.01 * q[4 * i]
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    (ids, dist), counters = counted(rii, index, lambda: rii.rii_adc_scan_linear(index, lut, topk))
    assert counters[5] == left and counters[6] > 0
    want = by_look_ups(rii, index, lut, topk)
    assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])


# reserved scratch: the plan names what the call does, in scratch for a few queries (look-ups), for the batch and for a larger one
@pytest.mark.parametrize("reserve,products", [((130, 50), False), ((40, 1024), True), ((600, 1024), True)])
def test_plan_within_reserved_scratch(reserve, products, rii):
    from paper_1808_03969_amd import binding
    Q, topk = 600, 300
    index, lut, want = scratch_case(rii, Q, topk)
    again = rii.Index(np.zeros((16, 256, 2), dtype=np.float32))  # (nothing has sized its scratch)
    again.add(index.get_codes())
    again.reserve_workspace(*reserve)
    held = again.info()["device_bytes"]
    assert (binding.rii_scan_linear_plan(again, Q, topk)[0] == 32) == products
    # (an index of another code book: tables that no query made, all left to the look-up kernels)
    (ids, dist), counters = counted(rii, again, lambda: rii.rii_adc_scan_linear(again, lut, topk))
    assert counters[5] == (Q if products else 0) and again.info()["device_bytes"] == held
    assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])

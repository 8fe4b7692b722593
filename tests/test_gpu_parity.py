"""Parity of the HIP library with the CPU oracle, element by element, through the C ABI.

Bar (written out): identifiers, codes, list numbers bit-exact; fp32 distances within 1e-5
relative (they are expected to be bit-identical, because both sides add the same fp32 table
entries in the same order).  Sizes are small enough for the oracle to finish in seconds but
span several blocks, several tiles per block and a ragged tail.
"""
import os

import numpy as np
import pytest
import torch

import synth
from helpers import RTOL, check_topk, t2n

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rii():
    import paper_1808_03969_amd as r
    r.load_library()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return r


def make_index(rii, oracle, N, D, M, K, kind="gaussian", seed=1, iters=4, Q=24):
    """Data, codebooks (product trainer), codes, coarse codes, oracle-built lists, product handle."""
    gen = {"gaussian": synth.gaussian, "sift": synth.sift_like, "mixture": synth.mixture}[kind]
    x = t2n(gen(1000 + seed, 0, N, D))
    q = t2n(gen(2000 + seed, 0, Q, D))
    train = x[t2n(synth.sample_rows(3000 + seed, N, min(N, 4000)))]
    cb = rii.rii_train_codebooks(train, M, iters=iters, seed=4000 + seed)
    codes = rii.rii_encode(cb, x)
    coarse = codes[t2n(synth.sample_rows(5000 + seed, N, K))].copy() if K else None
    d = dict(N=N, D=D, M=M, K=K, x=x, q=q, cb=cb, codes=codes, coarse=coarse)
    index = rii.Index(cb)
    index.add(codes)
    if K:
        T = oracle.sym_table(cb)
        a = oracle.assign(T, codes, coarse)
        off, lids = oracle.build_lists(a, K)
        index.set_lists(coarse, off, lids)
        d.update(T=T, a=a, off=off, lids=lids)
    d["index"] = index
    d["q_dev"] = torch.from_numpy(q).cuda()
    d["lut_ref"] = oracle.lut(cb, q)
    return d


@pytest.fixture(scope="module")
def idx32(rii, oracle_lib):
    # 70,001 rows: 18 tiles of 4096 rows with a ragged tail, M = 32 (the largest configuration's M)
    return make_index(rii, oracle_lib, N=70001, D=96, M=32, K=50, kind="mixture", seed=1)


@pytest.fixture(scope="module")
def idx16(rii, oracle_lib):
    return make_index(rii, oracle_lib, N=150000, D=128, M=16, K=97, kind="sift", seed=2)


@pytest.fixture(scope="module")
def idx8(rii, oracle_lib):
    # the tiny configuration: N = 10,000, D = 128, M = 8, linear scan, top-10
    return make_index(rii, oracle_lib, N=10000, D=128, M=8, K=16, kind="gaussian", seed=3, Q=100)


def lut_dev(rii, d):
    return rii.rii_build_lut(d["index"], d["q_dev"])


# ---------------------------------------------------------------- encode / tables
@pytest.mark.parametrize("name", ["idx8", "idx16", "idx32"])
def test_host_and_device_encode_bit_exact(name, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    ref = oracle_lib.encode(d["cb"], d["x"][:20000])
    assert np.array_equal(d["codes"][:20000], ref)
    dev = rii.rii_encode_device(d["index"], torch.from_numpy(d["x"][:20000]).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(t2n(dev), ref)
    assert np.array_equal(d["index"].get_codes(5, 100), d["codes"][5:105])


@pytest.mark.parametrize("name", ["idx8", "idx16", "idx32"])
def test_lut_bit_exact(name, rii, request):
    d = request.getfixturevalue(name)
    lut = lut_dev(rii, d)
    torch.cuda.synchronize()
    assert np.array_equal(t2n(lut), d["lut_ref"])


# ---------------------------------------------------------------- Alg. 1, whole database
@pytest.mark.parametrize("name,topk", [("idx8", 10), ("idx16", 100), ("idx32", 100), ("idx32", 1), ("idx16", 1024), ("idx32", 128), ("idx32", 129), ("idx16", 2), ("idx16", 65),
                                       ("idx8", 128)])  # (one chunk, 100 < topk <= 128: the two-queries-per-block kernel)
def test_linear_scan(name, topk, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    ids, dist = rii.rii_adc_scan_linear(d["index"], lut_dev(rii, d), topk)
    torch.cuda.synchronize()
    ids, dist = t2n(ids), t2n(dist)
    for i in range(len(d["q"])):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], topk)
        check_topk(ids[i], dist[i], ref[0], ref[1], rtol=RTOL)
        assert np.array_equal(dist[i], ref[1])  # same additions in the same order


@pytest.mark.parametrize("M", [8, 32])
def test_linear_scan_one_to_three_queries(M, rii, oracle_lib):
    """Fewer than four queries take the one-query-per-block kernel with the rows split over
    blocks (18 per query here).  With topk <= 18 the kernel seeds the shared bound itself, above
    that the separate seeding pass runs; both sides of that switch and every batch size 1..3."""
    N = 300001
    rng = np.random.default_rng(21 + M)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    q = rng.normal(size=(3, 2 * M)).astype(np.float32)
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    A = oracle_lib.lut(cb, q)
    for Q in (1, 2, 3):
        for topk in (1, 5, 18, 19, 100, 128):
            ids, dist = rii.rii_adc_scan_linear(index, lut[:Q].contiguous(), topk)
            torch.cuda.synchronize()
            for i in range(Q):
                ref = oracle_lib.linear_scan(A[i], codes, topk)
                assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (Q, topk, i)
    # target lists much shorter than the stated upper bound: most blocks of the launch have no
    # rows, fewer than topk of them can contribute to the seeded bound
    tids, toff = synth.subset_batch(83, N, [5000, 3])
    sub = rii.rii_adc_scan_subset(index, lut[:2].contiguous(), tids.cuda(), toff.cuda(), N, 10)
    torch.cuda.synchronize()
    tids, toff = t2n(tids), t2n(toff)
    for i in range(2):
        ref = oracle_lib.linear_scan(A[i], codes, 10, S=tids[toff[i]:toff[i + 1]])
        assert np.array_equal(t2n(sub[0])[i], ref[0]) and np.array_equal(t2n(sub[1])[i], ref[1])


def test_scans_over_random_shapes(rii, oracle_lib):
    """Forty seeded shape draws (rows, M, batch size, topk, whole database or target lists): every
    dispatch path of the scan entry points is hit somewhere, each result is compared with the
    oracle element by element, and every call is made twice (the second must repeat the first)."""
    rng = np.random.default_rng(int(os.environ.get("RII_TEST_SEED", "2024")))  # other seeds: more draws of the same kind
    for case in range(40):
        M = int(rng.choice([8, 16, 32, 32, 12, 64]))
        N = int(rng.choice([1, 63, 4097, 20000, 70001, 140000, 600000]))
        N = max(1, N + int(rng.integers(-40, 40)))
        Q = int(rng.choice([1, 2, 3, 4, 5, 17, 64, 130, 270]))
        topk = int(rng.choice([1, 7, 100, 101, 128, 129, 300]))
        Ds = 2
        cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
        codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
        if N > 300:
            codes[N // 2:N // 2 + 150] = codes[0]  # a run of exact ties
        q = rng.normal(size=(Q, M * Ds)).astype(np.float32)
        index = rii.Index(cb)
        index.add(codes)
        lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
        A = oracle_lib.lut(cb, q)
        subset = bool(rng.integers(0, 2))
        if subset:
            sizes = [int(rng.integers(0, N + 1)) for _ in range(Q)]
            tids, toff = synth.subset_batch(300 + case, N, sizes)
            args = (index, lut, tids.cuda(), toff.cuda(), max(sizes), topk)
            call = rii.rii_adc_scan_subset
            tids, toff = t2n(tids), t2n(toff)
        else:
            args = (index, lut, topk)
            call = rii.rii_adc_scan_linear
        first = call(*args)
        torch.cuda.synchronize()
        again = call(*args)
        torch.cuda.synchronize()
        assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1]), f"case {case}: not repeatable"
        ids, dist = t2n(first[0]), t2n(first[1])
        for i in range(0, Q, max(1, Q // 12)):
            S = tids[toff[i]:toff[i + 1]] if subset else None
            ref = oracle_lib.linear_scan(A[i], codes, topk, S=S)
            assert np.array_equal(ids[i], ref[0]) and np.array_equal(dist[i], ref[1]), \
                f"case {case}: N={N} M={M} Q={Q} topk={topk} subset={subset} query {i}"


def test_linear_scan_ties_and_padding(rii, oracle_lib):
    """Many identical codes (exact distance ties) and fewer rows than topk, in the kernel for small scans (the
    streaming kernels meet such codes in test_gpu_kernels.py)."""
    rng = np.random.default_rng(5)
    cb = rng.normal(size=(8, 256, 4)).astype(np.float32)
    base = rng.integers(0, 256, size=(37, 8)).astype(np.uint8)
    codes = np.tile(base, (300, 1))  # 11,100 rows, every code 300 times
    q = rng.normal(size=(6, 32)).astype(np.float32)
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    ids, dist = rii.rii_adc_scan_linear(index, lut, 700)
    torch.cuda.synchronize()
    A = oracle_lib.lut(cb, q)
    for i in range(6):
        ref = oracle_lib.linear_scan(A[i], codes, 700)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])
    # a full buffer of equal distances cannot make room by a distance bound alone and falls back to whole keys ...
    for topk in (100, 128):
        ids, dist = rii.rii_adc_scan_linear(index, lut, topk)
        torch.cuda.synchronize()
        for i in range(6):
            ref = oracle_lib.linear_scan(A[i], codes, topk)
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (topk, i)
    # ... also with one block a query (a larger batch)
    qb = rng.normal(size=(300, 32)).astype(np.float32)
    lutb = rii.rii_build_lut(index, torch.from_numpy(qb).cuda())
    Ab = oracle_lib.lut(cb, qb)
    ids, dist = rii.rii_adc_scan_linear(index, lutb, 100)
    torch.cuda.synchronize()
    for i in range(0, 300, 7):
        ref = oracle_lib.linear_scan(Ab[i], codes, 100)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), ("batched", i)
    small = rii.Index(cb)
    small.add(codes[:5])
    ids, dist = rii.rii_adc_scan_linear(small, lut, 8)
    torch.cuda.synchronize()
    for i in range(6):
        ref = oracle_lib.linear_scan(A[i], codes[:5], 8)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])


@pytest.mark.parametrize("kind", ["uniform", "clustered"])
def test_linear_scan_two_planes_pool_and_seeding(kind, rii, oracle_lib):
    """M = 32 codes are stored as two 16-byte planes and the one-query scan fetches second halves
    on demand: on codes where nearly every slice stays open half-way (uniform bytes) and on codes
    where most slices abandon (clustered data).  N is large enough for the blocks' fixed shares
    plus the shared pool of row units (18 blocks per query), with a ragged last tile; topk on both
    sides of the switch between bound seeding inside the kernel and the separate pass."""
    N, M = 300001, 32
    if kind == "uniform":
        rng = np.random.default_rng(5)
        cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
        codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
        q = rng.normal(size=(3, 2 * M)).astype(np.float32)
    else:
        x = t2n(synth.mixture(1031, 0, N, 96))
        q = t2n(synth.mixture(2031, 0, 3, 96))
        cb = rii.rii_train_codebooks(x[:4000], M, iters=3, seed=9)
        codes = rii.rii_encode(cb, x)
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    A = oracle_lib.lut(cb, q)
    for topk in (1, 18, 19, 100):
        refs = [oracle_lib.linear_scan(A[i], codes, topk) for i in range(3)]
        for Q in (1, 2, 3):
            for rep in range(2):
                ids, dist = rii.rii_adc_scan_linear(index, lut[:Q].contiguous(), topk)
                torch.cuda.synchronize()
                for i in range(Q):
                    assert np.array_equal(t2n(ids)[i], refs[i][0]) and np.array_equal(t2n(dist)[i], refs[i][1]), (Q, topk, i, rep)


def test_subset_scan_without_gather_copy(rii, oracle_lib, idx32):
    """RII_OPT_GATHER_COPY = 0 drops the whole-row copy of M = 32 codes: scans over target
    identifiers then gather the two halves of a row from the two planes.  Same results, N * M
    bytes less; the option cannot change once codes are stored."""
    from paper_1808_03969_amd import binding
    d = idx32
    lean = rii.Index(d["cb"])
    lean.set_option(binding.RII_OPT_GATHER_COPY, 0)
    lean.add(d["codes"][:40000])
    lean.add(d["codes"][40000:])                       # grows the array: both planes move
    with pytest.raises(rii.RiiError):
        lean.set_option(binding.RII_OPT_GATHER_COPY, 1)
    full = rii.Index(d["cb"])
    full.add(d["codes"][:40000])
    full.add(d["codes"][40000:])
    assert full.info()["device_bytes"] - lean.info()["device_bytes"] >= d["N"] * 32
    full.close()
    assert np.array_equal(lean.get_codes(), d["codes"])
    lut = rii.rii_build_lut(lean, d["q_dev"])
    Q = len(d["q"])
    for sizes, topk in (([5000] * Q, 100), ([d["N"]] * Q, 10), ([1 + 37 * i for i in range(Q)], 129)):
        tids, toff = synth.subset_batch(91, d["N"], sizes)
        ids, dist = rii.rii_adc_scan_subset(lean, lut, tids.cuda(), toff.cuda(), max(sizes), topk)
        torch.cuda.synchronize()
        for i in range(Q):
            S = t2n(tids)[t2n(toff)[i]:t2n(toff)[i + 1]]
            ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], topk, S=S)
            check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    lean.set_lists(d["coarse"], d["off"], d["lids"])
    lean.set_threshold(3000)
    tids, toff = synth.subset_batch(92, d["N"], [2000, 4000] * (Q // 2))
    qi, qd = rii.rii_query(lean, d["q_dev"], 50, tids.cuda(), toff.cuda(), 4000, L=2000)
    torch.cuda.synchronize()
    for i in range(Q):
        S = t2n(tids)[t2n(toff)[i]:t2n(toff)[i + 1]]
        ref = oracle_lib.query(d["cb"], d["q"][i], d["codes"], d["coarse"], d["off"], d["lids"], 50, 2000, 3000, S=S)
        check_topk(t2n(qi)[i], t2n(qd)[i], ref[0], ref[1])


def test_reserve_workspace_then_no_growth(rii, oracle_lib, idx16):
    """After rii_index_reserve_workspace(Q, topk, ., nprobe) no online call within those limits
    changes the bytes the handle holds (its scratch is never re-allocated), whatever the batch
    size; results are the usual ones."""
    d = idx16
    index = rii.Index(d["cb"])
    index.add(d["codes"])
    index.set_lists(d["coarse"], d["off"], d["lids"])
    Q, R, K = len(d["q"]), 100, d["K"]
    index.reserve_workspace(Q, R, max_targets=d["N"], nprobe=K)
    held = index.info()["device_bytes"]
    lut = rii.rii_build_lut(index, d["q_dev"])
    tids, toff = synth.subset_batch(93, d["N"], [7000] * Q)
    tids, toff = tids.cuda(), toff.cuda()
    for nq in (1, 2, 3, 4, 5, 8, 17, Q):
        for topk in (1, 10, R):
            rii.rii_adc_scan_linear(index, lut[:nq].contiguous(), topk)
            rii.rii_adc_scan_subset(index, lut[:nq].contiguous(), tids, toff[:nq + 1].contiguous(), 7000, topk)
            for P in (1, 7, K):
                probe, _ = rii.rii_coarse_assign(index, lut[:nq].contiguous(), P)
                rii.rii_adc_scan_ivf(index, lut[:nq].contiguous(), probe, topk)
            index.set_threshold(5000)
            rii.rii_query(index, d["q_dev"][:nq].contiguous(), topk, L=d["N"])          # all K lists
            rii.rii_query(index, d["q_dev"][:nq].contiguous(), topk, tids, toff[:nq + 1].contiguous(), 7000, L=d["N"])
            index.set_threshold(10 ** 9)
            rii.rii_query(index, d["q_dev"][:nq].contiguous(), topk)                    # linear branch
            torch.cuda.synchronize()
            assert index.info()["device_bytes"] == held, (nq, topk)
    ids, dist = rii.rii_adc_scan_linear(index, lut, R)
    torch.cuda.synchronize()
    for i in range(0, Q, 5):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], R)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])


def test_reserved_scratch_of_many_results_over_a_large_array(rii, oracle_lib):
    """Row chunks of a large batch are made for up to 100 results only: reserving for 1024 results holds room for
    their candidates once, not once a chunk; no call within the reservation grows it.  (The batch goes by matrix products.)"""
    reserved_scratch_over_a_large_array(52_000_000, 1, 32, 1024, rii, oracle_lib)


def test_reserved_scratch_over_a_large_array_by_look_ups(rii, oracle_lib):
    """The same with more than 128 coordinates and enough rows: the row chunks themselves (eleven at most, of 100 candidates)."""
    reserved_scratch_over_a_large_array(101_000_000, 17, 4, 1100, rii, oracle_lib)


def reserved_scratch_over_a_large_array(N, Ds, group, lists, rii, oracle_lib):
    from paper_1808_03969_amd import binding
    M, Q = 8, 8000
    rng = np.random.default_rng(3)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    index = rii.Index(cb)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    codes = torch.randint(0, 256, (N, M), generator=g, device="cuda", dtype=torch.uint8)
    index.add(codes)
    before = index.info()["device_bytes"]
    index.reserve_workspace(Q, 1024)
    held = index.info()["device_bytes"]
    # tables, candidates once, the bound-seeding pass' minima, room for the blocks of smaller batches; a quarter to spare
    assert held - before <= 1.25 * (Q * M * 1024 + Q * lists * 8 + 2048 * 8192 + 4400 * 1024 * 8) + (1 << 20)
    q = torch.randn((2100, M * Ds), generator=g, device="cuda")
    plan = binding.rii_scan_linear_plan(index, 2100, 100)
    assert plan[0] == group and plan[1] > 1
    lut = rii.rii_build_lut(index, q)
    ids, dist = rii.rii_adc_scan_linear(index, lut, 100)
    torch.cuda.synchronize()
    assert index.info()["device_bytes"] == held
    A = oracle_lib.lut(cb, t2n(q[:1]))
    ref = oracle_lib.linear_scan(A[0], t2n(codes), 100)
    assert np.array_equal(t2n(ids)[0], ref[0]) and np.array_equal(t2n(dist)[0], ref[1])


@pytest.mark.parametrize("M", [16, 32])
def test_linear_scan_large_topk_block_buffer(M, rii, oracle_lib):
    """topk above the per-wave buffers' reach: the waves of a block share one candidate buffer and
    compact it together whenever it fills.  Rows stored in order of DEcreasing distance to query 0
    make every row a candidate when it is met, so the buffer fills again and again and waves join
    compactions from every point of their loop (and after their rows have run out); query 1 meets
    the same rows in random order; target lists of uneven length take the same path."""
    N, Q = 1_300_000 + 77, 16  # 16 blocks per query, ~80k rows (20 tiles) each
    rng = np.random.default_rng(640 + M)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    q[1] = q[0] * 1.01  # nearly the same order of rows for query 1
    A = oracle_lib.lut(cb, q)
    full = oracle_lib.linear_scan(A[0], codes, N)       # all rows in (distance, id) order
    codes = np.ascontiguousarray(codes[full[0][::-1]])  # farthest first
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    for topk in (129, 1000, 1024):
        ids, dist = rii.rii_adc_scan_linear(index, lut, topk)
        torch.cuda.synchronize()
        for i in range(Q):
            ref = oracle_lib.linear_scan(A[i], codes, topk)
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1]), (M, topk, i)
    lut = lut[:2].contiguous()
    tids, toff = synth.subset_batch(91, N, [N - 5, 1500])
    sub = rii.rii_adc_scan_subset(index, lut, tids.cuda(), toff.cuda(), N, 700)
    torch.cuda.synchronize()
    tids, toff = t2n(tids), t2n(toff)
    for i in range(2):
        ref = oracle_lib.linear_scan(A[i], codes, 700, S=tids[toff[i]:toff[i + 1]])
        assert np.array_equal(t2n(sub[0])[i], ref[0]) and np.array_equal(t2n(sub[1])[i], ref[1]), (M, "subset", i)
    # one block per query (a short array), fewer rows than topk in one of them
    small = rii.Index(cb)
    small.add(codes[:5000])
    ids, dist = rii.rii_adc_scan_linear(small, lut, 1024)
    torch.cuda.synchronize()
    for i in range(2):
        ref = oracle_lib.linear_scan(A[i], codes[:5000], 1024)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])
    tiny = rii.Index(cb)
    tiny.add(codes[:300])
    ids, dist = rii.rii_adc_scan_linear(tiny, lut, 512)
    torch.cuda.synchronize()
    for i in range(2):
        ref = oracle_lib.linear_scan(A[i], codes[:300], 512)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])


@pytest.mark.parametrize("M,kind", [(8, "uniform"), (16, "clustered"), (32, "uniform"), (32, "clustered")])
def test_half_precision_table_variant(M, kind, rii, oracle_lib):
    """The separately evaluated variant of the batched kernel whose filter table holds fp16 entries
    (packed fp16 sums) instead of 15-bit integers: rows that pass are re-scored in fp32 as in the
    library's kernel, so the result must equal the oracle's bit for bit -- the filter may only let
    too many rows through, never too few.  Large-magnitude and tiny tables included (the scale of
    the fp16 table is a power of two chosen per group of four queries)."""
    from paper_1808_03969_amd import binding
    N, Q, topk = 150_003, 270, 50  # 68 groups of four: enough blocks for the batched kernel, last group short
    rng = np.random.default_rng(900 + M)
    cb = rng.normal(size=(M, 256, 2)).astype(np.float32)
    if kind == "uniform":
        codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    else:  # a few hundred distinct prototypes with some bytes changed: near-ties and long equal prefixes
        proto = rng.integers(0, 256, size=(300, M), dtype=np.uint8)
        codes = proto[rng.integers(0, 300, size=N)]
        flip = rng.random(size=(N, M)) < 0.1
        codes[flip] = rng.integers(0, 256, size=int(flip.sum()), dtype=np.uint8)
    q = rng.normal(size=(Q, 2 * M)).astype(np.float32)
    q[4:8] *= 1000.0   # one group of four with large distances,
    q[8:12] *= 1e-3    # one with the queries near the origin,
    q[13] *= 300.0     # one group of mixed magnitudes
    index = rii.Index(cb)
    index.add(codes)
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    A = oracle_lib.lut(cb, q)
    assert binding.rii_scan_linear_plan(index, Q, topk)[0] == 4
    ids, dist = binding.rii_bench_scan_linear_half(index, lut, topk)
    torch.cuda.synchronize()
    ids, dist = t2n(ids), t2n(dist)
    for i in range(Q):
        ref = oracle_lib.linear_scan(A[i], codes, topk)
        assert np.array_equal(ids[i], ref[0]) and np.array_equal(dist[i], ref[1]), (M, kind, i)
    # the library's own kernel on the same call (the flag does not stick)
    ids2, dist2 = rii.rii_adc_scan_linear(index, lut, topk)
    torch.cuda.synchronize()
    assert np.array_equal(t2n(ids2), ids) and np.array_equal(t2n(dist2), dist)
    with pytest.raises(rii.RiiError):
        binding.rii_bench_scan_linear_half(index, lut[:2].contiguous(), topk)  # not a four-queries-per-block launch


@pytest.mark.parametrize("M,Q,topk", [(8, 263, 100), (16, 258, 10)])
def test_linear_scan_large_batch_in_row_chunks(M, Q, topk, rii, oracle_lib):
    """As the next test, with so few coordinates that the batch goes by matrix products."""
    large_batch_in_row_chunks(M, Q, topk, 2, 32, rii, oracle_lib)


@pytest.mark.parametrize("M,Q,topk,Ds", [(8, 263, 100, 17), (16, 258, 10, 9)])
def test_linear_scan_large_batch_in_row_chunks_by_look_ups(M, Q, topk, Ds, rii, oracle_lib):
    """A batch that takes the several-queries-per-block kernel (more than 128 coordinates), over a code array long enough to
    be cut into row chunks; Q is not a multiple of four (short last group).  Codes are uniform
    bytes; copies of row 5 sit on both sides of every fifth tile boundary (the chunks here come
    out 65 tiles long, so every chunk boundary has them) and query 0 is row 5's own
    reconstruction, so its top-100 is a run of exact ties that crosses several chunks."""
    large_batch_in_row_chunks(M, Q, topk, Ds, 4, rii, oracle_lib)


def large_batch_in_row_chunks(M, Q, topk, Ds, group, rii, oracle_lib):
    from paper_1808_03969_amd import binding
    N = 2 * 2097152 + 3 * 4096 + 77
    rng = np.random.default_rng(11 + M)
    cb = rng.normal(size=(M, 256, Ds)).astype(np.float32)
    codes = rng.integers(0, 256, size=(N, M), dtype=np.uint8)
    for b in range(4096, N, 4096 * 5):
        codes[b - 1:b + 1] = codes[5]
    q = rng.normal(size=(Q, Ds * M)).astype(np.float32)
    q[0] = np.concatenate([cb[m][codes[5][m]] for m in range(M)])
    index = rii.Index(cb)
    index.add(codes)
    plan = binding.rii_scan_linear_plan(index, Q, topk)
    assert plan[0] == group and plan[1] > 1
    lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
    ids, dist = rii.rii_adc_scan_linear(index, lut, topk)
    torch.cuda.synchronize()
    ids, dist = t2n(ids), t2n(dist)
    A = oracle_lib.lut(cb, q)
    for i in range(Q):
        ref = oracle_lib.linear_scan(A[i], codes, topk)
        assert np.array_equal(ids[i], ref[0]) and np.array_equal(dist[i], ref[1]), f"query {i}"


def test_generic_m(rii, oracle_lib):
    """M = 12 takes the run-time-M code path (of the kernel for small scans)."""
    d = make_index(rii, oracle_lib, N=9000, D=48, M=12, K=0, seed=7, Q=5)
    ids, dist = rii.rii_adc_scan_linear(d["index"], lut_dev(rii, d), 20)
    torch.cuda.synchronize()
    for i in range(5):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], 20)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])


def test_m64(rii, oracle_lib):
    d = make_index(rii, oracle_lib, N=30000, D=128, M=64, K=0, kind="sift", seed=8, Q=4)
    ids, dist = rii.rii_adc_scan_linear(d["index"], lut_dev(rii, d), 50)
    torch.cuda.synchronize()
    for i in range(4):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], 50)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])


# ---------------------------------------------------------------- Alg. 1, target identifiers
@pytest.mark.parametrize("name", ["idx16", "idx32"])
def test_subset_scan(name, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    N, Q = d["N"], len(d["q"])
    sizes = [0, 1, 5, 99, 100, 101, 4096, 4097, 30000, N] + [1000 + 37 * i for i in range(Q - 10)]
    tids, toff = synth.subset_batch(77, N, sizes)
    ids, dist = rii.rii_adc_scan_subset(d["index"], lut_dev(rii, d), tids.cuda(), toff.cuda(), max(sizes), 100)
    torch.cuda.synchronize()
    ids, dist = t2n(ids), t2n(dist)
    tids, toff = t2n(tids), t2n(toff)
    for i in range(Q):
        S = tids[toff[i]:toff[i + 1]]
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], 100, S=S)
        check_topk(ids[i], dist[i], ref[0], ref[1])
        assert np.all(np.isin(ids[i][ids[i] >= 0], S))  # results are members of S (Sec. 5.3)
    # S = everything is the plain scan
    full = rii.rii_adc_scan_linear(d["index"], lut_dev(rii, d), 100)
    torch.cuda.synchronize()
    assert np.array_equal(ids[9], t2n(full[0])[9])


# ---------------------------------------------------------------- Alg. 2
@pytest.mark.parametrize("name", ["idx8", "idx16", "idx32"])
def test_coarse_assign(name, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    for P in (1, 7, d["K"]):
        ks, d0 = rii.rii_coarse_assign(d["index"], lut_dev(rii, d), P)
        torch.cuda.synchronize()
        for i in range(len(d["q"])):
            ref = oracle_lib.coarse_rank(d["lut_ref"][i], d["coarse"], P)
            assert np.array_equal(t2n(ks)[i], ref[0]) and np.array_equal(t2n(d0)[i], ref[1])


def test_coarse_assign_full_sort_path(rii, oracle_lib):
    """nprobe above the fused-selection limit ranks all K lists with the in-LDS sort."""
    d = make_index(rii, oracle_lib, N=6000, D=32, M=8, K=1500, seed=9, Q=3)
    ks, d0 = rii.rii_coarse_assign(d["index"], lut_dev(rii, d), 1500)
    torch.cuda.synchronize()
    for i in range(3):
        ref = oracle_lib.coarse_rank(d["lut_ref"][i], d["coarse"], 1500)
        assert np.array_equal(t2n(ks)[i], ref[0]) and np.array_equal(t2n(d0)[i], ref[1])


@pytest.mark.parametrize("name", ["idx16", "idx32"])
def test_ivf_scan(name, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    Q, K, N = len(d["q"]), d["K"], d["N"]
    lut = lut_dev(rii, d)
    sizes = [N // 3] * Q
    tids, toff = synth.subset_batch(78, N, sizes)
    tids_d, toff_d = tids.cuda(), toff.cuda()
    tids, toff = t2n(tids), t2n(toff)
    for P in (1, 8, K):
        probe, _ = rii.rii_coarse_assign(d["index"], lut, P)
        for use_S, L in ((False, 0), (True, 0), (False, 777), (True, 501)):
            ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, 100,
                                             target_ids=tids_d if use_S else None,
                                             target_offsets=toff_d if use_S else None, L=L)
            torch.cuda.synchronize()
            for i in range(Q):
                S = tids[toff[i]:toff[i + 1]] if use_S else None
                ref = oracle_lib.inverted_index(d["lut_ref"][i], d["codes"], d["coarse"], d["off"], d["lids"],
                                                R=100, P=P, S=S, Lcap=L)
                check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    # all lists, no cap, no filter == the plain scan (Sec. 4.2)
    probe, _ = rii.rii_coarse_assign(d["index"], lut, K)
    a = rii.rii_adc_scan_ivf(d["index"], lut, probe, 100)
    b = rii.rii_adc_scan_linear(d["index"], lut, 100)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("M", [12, 8])
def test_ivf_scan_short_and_empty_lists(M, rii, oracle_lib):
    """Many short posting lists, some of them empty (more coarse centres than distinct nearest
    ones), probed in every combination of target set and candidate cap by the kernel for small scans; M = 12
    takes the run-time-M code path.  The cap cuts inside a list, lies beyond all members, or is 1."""
    d = make_index(rii, oracle_lib, N=5000, D=48, M=M, K=700, seed=9, Q=7)
    N, K, Q = d["N"], d["K"], len(d["q"])
    # every seventh centre becomes a copy of centre 0: ties go to the smaller index, so the copies' lists are empty
    d["coarse"][1::7] = d["coarse"][0]
    d["a"] = oracle_lib.assign(d["T"], d["codes"], d["coarse"])
    d["off"], d["lids"] = oracle_lib.build_lists(d["a"], K)
    d["index"].set_lists(d["coarse"], d["off"], d["lids"])
    assert (np.diff(d["off"]) == 0).sum() >= 90
    lut = lut_dev(rii, d)
    tids, toff = synth.subset_batch(81, N, [N // 2] * Q)
    tids_d, toff_d = tids.cuda(), toff.cuda()
    tids, toff = t2n(tids), t2n(toff)
    for P in (1, 40, K):
        probe, _ = rii.rii_coarse_assign(d["index"], lut, P)
        for use_S, L in ((False, 0), (True, 0), (False, 1), (False, 333), (False, 10 * N), (True, 57)):
            ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, 20,
                                             target_ids=tids_d if use_S else None,
                                             target_offsets=toff_d if use_S else None, L=L)
            torch.cuda.synchronize()
            for i in range(Q):
                S = tids[toff[i]:toff[i + 1]] if use_S else None
                ref = oracle_lib.inverted_index(d["lut_ref"][i], d["codes"], d["coarse"], d["off"], d["lids"],
                                                R=20, P=P, S=S, Lcap=L)
                check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])


@pytest.mark.parametrize("M", [16, 32])
def test_ivf_scan_nearest_list_empty_and_last(M, rii, oracle_lib):
    """The nearest probed list of every query is empty and is the last list of the arrays, so its
    start is one row past the list-ordered codes (N * M a whole number of 2 MB pages here): waves
    without a next tile must prefetch a real member's row, not that start."""
    N, K, Q = (1 << 17) if M == 16 else (1 << 16), 33, 5
    d = make_index(rii, oracle_lib, N=N, D=2 * M, M=M, K=K - 1, seed=12, iters=2, Q=Q)
    # an extra centre equal to each query's own code would be nearest; one centre serves all
    # queries here because they are made equal up to a tiny perturbation of the first
    q = np.repeat(d["q"][:1], Q, axis=0) + np.arange(Q, dtype=np.float32)[:, None] * 1e-3
    qcode = oracle_lib.encode(d["cb"], q[:1])
    coarse = np.concatenate([d["coarse"], qcode], axis=0)
    off = np.concatenate([d["off"], d["off"][-1:]])           # list K-1 empty, start == N
    d["index"].set_lists(coarse, off, d["lids"])
    A = oracle_lib.lut(d["cb"], q)
    lut = rii.rii_build_lut(d["index"], torch.from_numpy(q).cuda())
    tids, toff = synth.subset_batch(82, N, [N // 3] * Q)
    for P in (1, 2, 9, K):
        probe, _ = rii.rii_coarse_assign(d["index"], lut, P)
        assert np.all(t2n(probe)[:, 0] == K - 1)
        for use_S, L in ((False, 0), (True, 0), (False, 700), (True, 50)):
            ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, 10,
                                             target_ids=tids.cuda() if use_S else None,
                                             target_offsets=toff.cuda() if use_S else None, L=L)
            torch.cuda.synchronize()
            for i in range(Q):
                S = t2n(tids)[t2n(toff)[i]:t2n(toff)[i + 1]] if use_S else None
                ref = oracle_lib.inverted_index(A[i], d["codes"], coarse, off, d["lids"], R=10, P=P, S=S, Lcap=L)
                check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])


def test_ivf_and_query_over_random_shapes(rii, oracle_lib):
    """Sixteen seeded draws of (rows, M, lists, batch size, lists probed, cap, target lists, topk)
    for the inverted-index scan and the query procedure, each compared with the oracle."""
    rng = np.random.default_rng(int(os.environ.get("RII_TEST_SEED", "4242")))
    for case in range(16):
        M = int(rng.choice([8, 16, 32, 12]))
        N = int(rng.choice([700, 5000, 20011]))
        K = int(rng.choice([1, 9, 64, 257]))
        K = min(K, N)
        Q = int(rng.choice([1, 3, 8, 40]))
        topk = int(rng.choice([1, 10, 100, 130]))
        d = make_index(rii, oracle_lib, N=N, D=2 * M, M=M, K=K, seed=50 + case, iters=2, Q=Q)
        lut = lut_dev(rii, d)
        P = int(rng.integers(1, K + 1))
        L = int(rng.choice([0, 1, 50, N]))
        use_S = bool(rng.integers(0, 2))
        sizes = [int(rng.integers(0, N + 1)) for _ in range(Q)]
        tids, toff = synth.subset_batch(900 + case, N, sizes)
        tids_d, toff_d = tids.cuda(), toff.cuda()
        tids, toff = t2n(tids), t2n(toff)
        probe, _ = rii.rii_coarse_assign(d["index"], lut, P)
        ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, topk, target_ids=tids_d if use_S else None,
                                         target_offsets=toff_d if use_S else None, L=L)
        torch.cuda.synchronize()
        for i in range(Q):
            S = tids[toff[i]:toff[i + 1]] if use_S else None
            ref = oracle_lib.inverted_index(d["lut_ref"][i], d["codes"], d["coarse"], d["off"], d["lids"],
                                            R=topk, P=P, S=S, Lcap=L)
            check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
        theta = int(rng.choice([0, N // 3, N + 1]))
        Lq = max(1, L)
        d["index"].set_threshold(theta)
        ids, dist = rii.rii_query(d["index"], d["q_dev"], topk, tids_d if use_S else None, toff_d if use_S else None,
                                  max(sizes) if use_S else 0, Lq)
        torch.cuda.synchronize()
        for i in range(Q):
            S = tids[toff[i]:toff[i + 1]] if use_S else None
            ref = oracle_lib.query(d["cb"], d["q"][i], d["codes"], d["coarse"], d["off"], d["lids"], topk, Lq, theta, S=S)
            check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
        d["index"].set_threshold(0)


# ---------------------------------------------------------------- PartialSort + Take
def test_topk_on_explicit_candidates(rii):
    g = torch.Generator().manual_seed(3)
    lens = [0, 1, 50, 1024, 1025, 5000, 16384, 40000]
    off = torch.zeros(len(lens) + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.tensor(lens), 0)
    dist = torch.randn(int(off[-1]), generator=g)  # negative values too
    dist[off[5]:off[5] + 2500] = dist[off[5]]      # a long run of exact ties
    cid = torch.randperm(int(off[-1]), generator=g).to(torch.int32)
    for topk in (1, 100, 1024):
        ids, out = rii.rii_topk(dist.cuda(), cid.cuda(), off.cuda(), topk)
        torch.cuda.synchronize()
        for s, n in enumerate(lens):
            dd, ii = dist[off[s]:off[s + 1]].numpy(), cid[off[s]:off[s + 1]].numpy()
            order = np.lexsort((ii, dd))[:topk]
            k = len(order)
            assert np.array_equal(t2n(ids)[s][:k], ii[order]) and np.array_equal(t2n(out)[s][:k], dd[order])
            assert np.all(t2n(ids)[s][k:] == -1) and np.all(np.isinf(t2n(out)[s][k:]))
    # positions as identifiers, and the full-sort path for topk > 1024
    lens2 = [3000, 16384, 1]
    off2 = torch.tensor([0, 3000, 19384, 19385], dtype=torch.int64)
    dist2 = torch.randn(19385, generator=g)
    ids, out = rii.rii_topk(dist2.cuda(), None, off2.cuda(), 4000, max_segment=16384)
    torch.cuda.synchronize()
    for s, n in enumerate(lens2):
        dd = dist2[off2[s]:off2[s + 1]].numpy()
        order = np.lexsort((np.arange(n), dd))[:4000]
        assert np.array_equal(t2n(ids)[s][:len(order)], order)
        assert np.all(t2n(ids)[s][len(order):] == -1)


# ---------------------------------------------------------------- Alg. 3
@pytest.mark.parametrize("name", ["idx16", "idx32"])
def test_query_switch(name, rii, oracle_lib, request):
    d = request.getfixturevalue(name)
    N, K, Q = d["N"], d["K"], len(d["q"])
    theta, L, R = 3000, 2 * (N // K), 100
    d["index"].set_threshold(theta)
    sizes = [theta - 1, theta, theta + 1, 0, 10, N, N // 2, 200] + [500 * (i + 1) for i in range(Q - 8)]
    tids, toff = synth.subset_batch(79, N, sizes)
    ids, dist = rii.rii_query(d["index"], d["q_dev"], R, tids.cuda(), toff.cuda(), max(sizes), L)
    torch.cuda.synchronize()
    tids, toff = t2n(tids), t2n(toff)
    modes = []
    for i in range(Q):
        S = tids[toff[i]:toff[i + 1]]
        ref = oracle_lib.query(d["cb"], d["q"][i], d["codes"], d["coarse"], d["off"], d["lids"], R, L, theta, S=S)
        modes.append(ref[2])
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    assert modes[:3] == [0, 1, 1] and 0 in modes[3:] and 1 in modes[3:]
    # whole database
    ids, dist = rii.rii_query(d["index"], d["q_dev"], R, L=L)
    torch.cuda.synchronize()
    for i in range(Q):
        ref = oracle_lib.query(d["cb"], d["q"][i], d["codes"], d["coarse"], d["off"], d["lids"], R, L, theta)
        assert ref[2] == 1
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    # theta above N: everything is a linear scan
    d["index"].set_threshold(N + 1)
    ids, dist = rii.rii_query(d["index"], d["q_dev"], R, L=L)
    torch.cuda.synchronize()
    for i in range(0, Q, 5):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], d["codes"], R)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    d["index"].set_threshold(0)


# ---------------------------------------------------------------- lists, addition, reconfigure
def test_assign_and_build_lists(rii, oracle_lib, idx16):
    d = idx16
    a = rii.rii_assign(d["index"], torch.from_numpy(d["codes"][:30000]).cuda(), torch.from_numpy(d["coarse"]).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(t2n(a), d["a"][:30000])
    other = rii.Index(d["cb"])
    other.add(d["codes"][:40000])
    other.build_lists(d["coarse"])
    coarse, off, lids, assign = other.get_lists()
    a_ref = oracle_lib.assign(d["T"], d["codes"][:40000], d["coarse"])
    off_ref, lids_ref = oracle_lib.build_lists(a_ref, d["K"])
    assert np.array_equal(assign, a_ref) and np.array_equal(off, off_ref) and np.array_equal(lids, lids_ref)
    inf = other.info()
    assert inf["paper_bytes"] == oracle_lib.index_bytes(40000, d["K"], d["M"])


@pytest.mark.parametrize("M", [16, 32])
def test_add_then_search_then_reconfigure(M, rii, oracle_lib):
    """Data addition keeps the lists of the old centres (Sec. 4.3); reconfigure rebuilds them.
    (M = 32 keeps its codes in two planes plus a whole-row copy: all three must follow.)"""
    d = make_index(rii, oracle_lib, N=20000, D=96, M=M, K=20, kind="mixture", seed=11, Q=8)
    extra_x = t2n(synth.mixture(6011, 0, 4000, 96, shift=0.5, means_seed=1011))
    extra = rii.rii_encode(d["cb"], extra_x)
    d["index"].add(extra)
    codes = np.concatenate([d["codes"], extra])
    a = oracle_lib.assign(d["T"], codes, d["coarse"])
    off, lids = oracle_lib.build_lists(a, 20)
    _, off_g, lids_g, a_g = d["index"].get_lists()
    assert np.array_equal(a_g, a) and np.array_equal(off_g, off) and np.array_equal(lids_g, lids)
    lut = lut_dev(rii, d)
    probe, _ = rii.rii_coarse_assign(d["index"], lut, 4)
    ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, 50)
    torch.cuda.synchronize()
    for i in range(8):
        ref = oracle_lib.inverted_index(d["lut_ref"][i], codes, d["coarse"], off, lids, R=50, P=4)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    # reconfigure: deterministic, lists are the oracle's lists for the new centres
    d["index"].reconfigure(40, iters=3, seed=5)
    coarse1, off1, lids1, a1 = d["index"].get_lists()
    d["index"].reconfigure(40, iters=3, seed=5)
    coarse2, off2, lids2, a2 = d["index"].get_lists()
    assert np.array_equal(coarse1, coarse2) and np.array_equal(lids1, lids2)
    a_ref = oracle_lib.assign(d["T"], codes, coarse1)
    off_ref, lids_ref = oracle_lib.build_lists(a_ref, 40)
    assert np.array_equal(a1, a_ref) and np.array_equal(off1, off_ref) and np.array_equal(lids1, lids_ref)
    probe, _ = rii.rii_coarse_assign(d["index"], lut, 6)
    ids, dist = rii.rii_adc_scan_ivf(d["index"], lut, probe, 50)
    torch.cuda.synchronize()
    for i in range(8):
        ref = oracle_lib.inverted_index(d["lut_ref"][i], codes, coarse1, off1, lids1, R=50, P=6)
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    # the other views of the grown code array: linear scan, gathered scan, read-back
    lin = rii.rii_adc_scan_linear(d["index"], lut, 50)
    tids = torch.arange(1, codes.shape[0], 5, dtype=torch.int32).cuda()
    toff = torch.tensor([0, tids.numel()], dtype=torch.int64).cuda()
    sub = rii.rii_adc_scan_subset(d["index"], lut[:1].contiguous(), tids, toff, tids.numel(), 50)
    torch.cuda.synchronize()
    assert np.array_equal(d["index"].get_codes(), codes)
    for i in range(8):
        ref = oracle_lib.linear_scan(d["lut_ref"][i], codes, 50)
        assert np.array_equal(t2n(lin[0])[i], ref[0]) and np.array_equal(t2n(lin[1])[i], ref[1])
    ref = oracle_lib.linear_scan(d["lut_ref"][0], codes, 50, S=t2n(tids))
    assert np.array_equal(t2n(sub[0])[0], ref[0]) and np.array_equal(t2n(sub[1])[0], ref[1])


def test_determinism(rii, idx32):
    d = idx32
    lut = lut_dev(rii, d)
    a = rii.rii_adc_scan_linear(d["index"], lut, 100)
    b = rii.rii_adc_scan_linear(d["index"], lut, 100)
    torch.cuda.synchronize()
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_pruned_assignment_equals_brute_force(rii, oracle_lib):
    """a(n) among many centres; the lists must be the ones brute force gives, on clustered and on unclustered data.
    (At 96 dimensions the matrix products decide most of it; test_gpu_kernels.py has the pruned search by itself.)"""
    for kind, seed in (("mixture", 21), ("gaussian", 22)):
        d = make_index(rii, oracle_lib, N=30000, D=96, M=16, K=0, kind=kind, seed=seed, Q=2)
        coarse = d["codes"][t2n(synth.sample_rows(9, 30000, 1500))].copy()
        coarse[7] = coarse[3]  # a duplicated centre: ties must go to the lower number
        d["index"].build_lists(coarse)
        _, off, lids, a = d["index"].get_lists()
        T = oracle_lib.sym_table(d["cb"])
        a_ref = oracle_lib.assign(T, d["codes"], coarse)
        assert np.array_equal(a, a_ref)
        brute = rii.rii_assign(d["index"], torch.from_numpy(d["codes"]).cuda(), torch.from_numpy(coarse).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(t2n(brute), a_ref)
        off_ref, lids_ref = oracle_lib.build_lists(a_ref, 1500)
        assert np.array_equal(off, off_ref) and np.array_equal(lids, lids_ref)


def test_add_in_odd_pieces_and_read_back(rii, oracle_lib):
    """Codes appended in pieces of odd length read back unchanged and score like one array
    (the stored form of a row depends on its row number)."""
    for M, D in ((8, 32), (16, 64), (32, 96), (12, 48)):
        rng = np.random.default_rng(M)
        cb = rng.normal(size=(M, 256, D // M)).astype(np.float32)
        codes = rng.integers(0, 256, size=(9001, M)).astype(np.uint8)
        index = rii.Index(cb)
        cut = [0, 1, 38, 1000, 1003, 5000, 9001]
        for a, b in zip(cut[:-1], cut[1:]):
            if (a // 7) % 2:
                index.add(torch.from_numpy(codes[a:b]).cuda())
            else:
                index.add(codes[a:b])
        assert np.array_equal(index.get_codes(), codes)
        assert np.array_equal(index.get_codes(37, 1970), codes[37:2007])
        q = rng.normal(size=(3, D)).astype(np.float32)
        lut = rii.rii_build_lut(index, torch.from_numpy(q).cuda())
        ids, dist = rii.rii_adc_scan_linear(index, lut, 50)
        tids = torch.arange(3, 9001, 7, dtype=torch.int32).cuda()
        toff = torch.tensor([0, 0, 500, tids.numel()], dtype=torch.int64).cuda()
        sub = rii.rii_adc_scan_subset(index, lut, tids, toff, tids.numel(), 50)
        torch.cuda.synchronize()
        A = oracle_lib.lut(cb, q)
        for i in range(3):
            ref = oracle_lib.linear_scan(A[i], codes, 50)
            assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])
            S = t2n(tids)[t2n(toff)[i]:t2n(toff)[i + 1]]
            ref = oracle_lib.linear_scan(A[i], codes, 50, S=S)
            assert np.array_equal(t2n(sub[0])[i], ref[0]) and np.array_equal(t2n(sub[1])[i], ref[1])


def test_check_target_ids(rii, idx8):
    """The optional precondition check on target identifiers (sorted, in range; Sec. 4.2)."""
    index, N = idx8["index"], idx8["N"]
    dev = lambda a, t: torch.tensor(a, dtype=t).cuda()
    off = dev([0, 3, 3, 6], torch.int64)
    assert rii.rii_check_target_ids(index, dev([0, 5, N - 1, 2, 3, 4], torch.int32), off) == 0
    assert rii.rii_check_target_ids(index, None, dev([0, 0, 0], torch.int64)) == 0
    # a descent is fine across two queries' ranges, not inside one
    assert rii.rii_check_target_ids(index, dev([0, 5, 4, 2, 3, 4], torch.int32), off) == -4
    assert rii.rii_check_target_ids(index, dev([0, 5, 5, 2, 3, 4], torch.int32), off) == -4   # repeated
    assert rii.rii_check_target_ids(index, dev([0, 5, N, 2, 3, 4], torch.int32), off) == -4   # out of range
    assert rii.rii_check_target_ids(index, dev([-1, 5, 6, 2, 3, 4], torch.int32), off) == -4
    assert rii.rii_check_target_ids(index, dev([0, 5, 6, 2, 3, 4], torch.int32), dev([0, 4, 3, 6], torch.int64)) == -1
    big = torch.arange(0, N, 3, dtype=torch.int32).cuda()
    assert rii.rii_check_target_ids(index, big, dev([0, big.numel()], torch.int64)) == 0
    big[big.numel() // 2] = 0
    assert rii.rii_check_target_ids(index, big, dev([0, big.numel()], torch.int64)) == -4


def test_error_codes(rii, idx8):
    """Argument errors come back as status codes and leave the outputs untouched."""
    d = idx8
    lut = lut_dev(rii, d)
    E = rii.RiiError
    for bad, status in ((0, -1), (2000, -7)):
        with pytest.raises(E) as e:
            rii.rii_adc_scan_linear(d["index"], lut, bad)
        assert e.value.status == status
    with pytest.raises(E) as e:
        rii.rii_coarse_assign(d["index"], lut, d["K"] + 1)
    assert e.value.status == -1
    bare = rii.Index(d["cb"])
    bare.add(d["codes"][:100])
    with pytest.raises(E) as e:
        rii.rii_coarse_assign(bare, lut, 1)
    assert e.value.status == -3                      # no coarse centres / lists
    probe = torch.zeros((len(d["q"]), 1), dtype=torch.int32, device="cuda")
    with pytest.raises(E) as e:
        rii.rii_adc_scan_ivf(bare, lut, probe, 5)
    assert e.value.status == -3
    coarse = d["codes"][:4].copy()
    off = np.array([0, 25, 50, 75, 100], dtype=np.int64)
    ids = np.arange(100, dtype=np.int32)
    bare.set_lists(coarse, off, ids)                 # valid
    with pytest.raises(E) as e:
        bare.set_lists(coarse, off, ids[::-1].copy())  # lists not ascending
    assert e.value.status == -4
    dup = ids.copy(); dup[3] = 2
    with pytest.raises(E) as e:
        bare.set_lists(coarse, off, dup)             # not a permutation
    assert e.value.status == -4
    with pytest.raises(E) as e:
        bare.set_lists(coarse, np.array([0, 25, 50, 75, 99], dtype=np.int64), ids)
    assert e.value.status == -1
    # M = 2 is outside what the scan kernels are built for
    cb2 = np.zeros((2, 256, 2), dtype=np.float32)
    tiny = rii.Index(cb2)
    with pytest.raises(E) as e:
        tiny.add(np.zeros((4, 2), dtype=np.uint8))
    assert e.value.status == -7
    out_i = torch.full((len(d["q"]), 5), 123, dtype=torch.int32, device="cuda")
    out_d = torch.full((len(d["q"]), 5), 7.0, device="cuda")
    with pytest.raises(E):
        rii.rii_adc_scan_linear(d["index"], lut, 0, out=(out_i, out_d))
    torch.cuda.synchronize()
    assert int(out_i.min()) == 123 and float(out_d.max()) == 7.0


def test_threshold_calibration(rii, oracle_lib, idx16):
    """theta is measured on the GPU; whatever value comes out, Alg. 3 with it equals the oracle's."""
    d = idx16
    N, K, R = d["N"], d["K"], 50
    L = N // K
    theta = d["index"].calibrate_threshold(L, topk=R, nq=16, seed=3)
    assert 0 <= theta <= N + 1 and d["index"].info()["theta"] == theta
    assert d["index"].calibrate_threshold(L, topk=R, nq=16, max_targets=4096, seed=3) <= 4097
    d["index"].set_threshold(theta)
    Q = len(d["q"])
    sizes = [max(1, min(N, int(theta * f))) for f in (0.25, 0.5, 0.9, 1.0, 1.1, 2.0, 4.0)] + [N // 3] * (Q - 7)
    tids, toff = synth.subset_batch(80, N, sizes)
    ids, dist = rii.rii_query(d["index"], d["q_dev"], R, tids.cuda(), toff.cuda(), max(sizes), L)
    torch.cuda.synchronize()
    tids, toff = t2n(tids), t2n(toff)
    for i in range(Q):
        ref = oracle_lib.query(d["cb"], d["q"][i], d["codes"], d["coarse"], d["off"], d["lids"], R, L, theta,
                               S=tids[toff[i]:toff[i + 1]])
        check_topk(t2n(ids)[i], t2n(dist)[i], ref[0], ref[1])
    d["index"].set_threshold(0)


def test_rotation_opq_variant(rii, oracle_lib):
    """Sec. 4.5: rotate, then plain PQ.  The rotation is bit-identical to the oracle's, and the
    whole rotated pipeline (encode, table, scan) matches the oracle run on the rotated inputs."""
    rng = np.random.default_rng(4)
    for D in (24, 96, 130):
        Rm, _ = np.linalg.qr(rng.normal(size=(D, D)))
        Rm = Rm.astype(np.float32)
        x = rng.normal(size=(1003, D)).astype(np.float32)
        y = rii.rii_rotate(torch.from_numpy(Rm).cuda(), torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(t2n(y), oracle_lib.rotate(Rm, x))
    D, M, N = 96, 16, 20000
    Rm, _ = np.linalg.qr(rng.normal(size=(D, D)))
    Rm = Rm.astype(np.float32)
    x = t2n(synth.mixture(31, 0, N, D))
    q = t2n(synth.mixture(32, 0, 6, D, means_seed=31))
    Rd = torch.from_numpy(Rm).cuda()
    xr = rii.rii_rotate(Rd, torch.from_numpy(x).cuda())
    qr = rii.rii_rotate(Rd, torch.from_numpy(q).cuda())
    cb = rii.rii_train_codebooks(t2n(xr)[:4000], M, iters=3, seed=1)
    index = rii.Index(cb)
    codes = rii.rii_encode_device(index, xr)
    index.add(codes)
    ids, dist = rii.rii_adc_scan_linear(index, rii.rii_build_lut(index, qr), 30)
    torch.cuda.synchronize()
    xr_ref, qr_ref = oracle_lib.rotate(Rm, x), oracle_lib.rotate(Rm, q)
    codes_ref = oracle_lib.encode(cb, xr_ref)
    assert np.array_equal(t2n(codes), codes_ref)
    A = oracle_lib.lut(cb, qr_ref)
    for i in range(6):
        ref = oracle_lib.linear_scan(A[i], codes_ref, 30)
        assert np.array_equal(t2n(ids)[i], ref[0]) and np.array_equal(t2n(dist)[i], ref[1])

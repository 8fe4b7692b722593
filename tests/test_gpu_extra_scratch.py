"""The scratch that batches by matrix products and filter calls can do without: what one kind of call is refused, or a captured graph of
it holds, changes nothing for the others or for larger calls of its own."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rii():
    import paper_1808_03969_amd as r
    r.load_library()
    assert torch.cuda.is_available(), "these tests need the GPU"
    return r


def make(rii, N=300_000, K=20, M=16, Ds=2):
    rng = np.random.default_rng(N + K)
    index = rii.Index(rng.standard_normal((M, 256, Ds)).astype(np.float32))
    index.add(rng.integers(0, 256, (N, M), dtype=np.uint8))
    a = rng.permutation(np.arange(N) % K)
    off = np.arange(K + 1, dtype=np.int64) * (N // K)
    index.set_lists(rng.integers(0, 256, (K, M), dtype=np.uint8), off, np.argsort(a, kind="stable").astype(np.int32))
    return index, rng


def tables(rii, index, rng, Q):
    return rii.rii_build_lut(index, torch.from_numpy(rng.standard_normal((Q, 32)).astype(np.float32)).cuda())


def filters(rng, N, K, Q, nprobe, size):
    """Lists and a target set a query."""
    sets = np.concatenate([np.sort(rng.permutation(N)[:size]) for _ in range(Q)]).astype(np.int32)
    probe = np.stack([rng.permutation(K)[:nprobe] for _ in range(Q)]).astype(np.int32)
    return torch.from_numpy(probe).cuda(), torch.from_numpy(sets).cuda(), torch.arange(Q + 1, dtype=torch.int64).cuda() * size


def multiplied(rii, index, call):
    """The call's result and the blocks that multiplied in it."""
    from paper_1808_03969_amd import binding
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    binding.rii_index_set_scan_events(index, ev[0].cuda_event, ev[1].cuda_event)
    binding.rii_index_read_scan_counters(index)
    out = call()
    torch.cuda.synchronize()
    blocks = binding.rii_index_read_scan_counters(index)[6]
    binding.rii_index_set_scan_events(index, None, None)
    return out, blocks


def device_room(rii, index, most):
    room = rii.load_library().rii_internal_matrix_room
    room.restype, room.argtypes = None, [ctypes.c_void_p, ctypes.c_size_t]
    room(index.handle, most)


def test_captured_filter_call(rii):
    """A graph of one small filter call: a large scan goes by products all the same, larger filter calls get their lists of picked
    members, and the graph's replays stay right."""
    index, rng = make(rii)
    N, K = 300_000, 20
    lut = tables(rii, index, rng, 1500)
    probe, tids, toff = filters(rng, N, K, 200, 6, 30_000)
    small = lut[:1].contiguous(), probe[:1].contiguous(), tids[:30_000].contiguous(), toff[:2].contiguous()

    def one(out=None):
        return rii.rii_adc_scan_ivf(index, small[0], small[1], 50, small[2], small[3], L=700, out=out)

    first = one()
    torch.cuda.synchronize()
    out = torch.empty_like(first[0]), torch.empty_like(first[1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one(out)
    parts = [rii.rii_adc_scan_ivf(index, lut[i:i + 1].contiguous(), probe[i:i + 1].contiguous(), 50, tids[i * 30_000:(i + 1) * 30_000].contiguous(),
                                  toff[:2].contiguous(), L=700) for i in range(200)]
    torch.cuda.synchronize()
    for L in (700, 2000):
        before = index.info()["device_bytes"]
        many = rii.rii_adc_scan_ivf(index, lut[:200].contiguous(), probe, 50, tids, toff, L=L)
        torch.cuda.synchronize()
        assert index.info()["device_bytes"] >= before + 200 * 700 * 4  # (lists of L members a query)
        if L == 700:
            assert torch.equal(many[0], torch.cat([p[0] for p in parts])) and torch.equal(many[1], torch.cat([p[1] for p in parts]))
        for _ in range(3):
            out[0].zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out[0], first[0]) and torch.equal(out[1], first[1])
            one()
    want = [rii.rii_adc_scan_linear(index, lut[i:i + 50].contiguous(), 50) for i in range(0, 1500, 50)]
    got, blocks = multiplied(rii, index, lambda: rii.rii_adc_scan_linear(index, lut, 50))
    assert blocks > 0
    assert torch.equal(got[0], torch.cat([w[0] for w in want])) and torch.equal(got[1], torch.cat([w[1] for w in want]))


def test_refusals_are_apart(rii):
    """A device that has room for the linear scan's pieces and a filter call's lists, and none for the batch through the lists."""
    index, rng = make(rii)
    lut = tables(rii, index, rng, 2500)
    probe = torch.from_numpy(np.stack([rng.permutation(20)[:6] for _ in range(2500)]).astype(np.int32)).cuda()
    part = lut[:1100].contiguous()
    want = [rii.rii_adc_scan_linear(index, part[i:i + 50].contiguous(), 100) for i in range(0, 1100, 50)]
    rii.rii_adc_scan_ivf(index, lut[:1100].contiguous(), probe[:1100].contiguous(), 1000)  # (look-ups' scratch)
    device_room(rii, index, 24 << 20)
    before = index.info()["device_bytes"]
    rii.rii_adc_scan_ivf(index, lut, probe, 100)
    torch.cuda.synchronize()
    refused = index.info()["device_bytes"]
    assert refused < before + (20 << 20)  # (no room for 2500 queries' groups and candidates)
    got, blocks = multiplied(rii, index, lambda: rii.rii_adc_scan_linear(index, part, 100))
    assert blocks > 0 and index.info()["device_bytes"] > refused
    assert torch.equal(got[0], torch.cat([w[0] for w in want])) and torch.equal(got[1], torch.cat([w[1] for w in want]))


def test_calls_that_vary_a_little(rii):
    """Filter calls of slowly growing caps ask the device for scratch now and then, not each time."""
    index, rng = make(rii)
    lut = tables(rii, index, rng, 300)
    probe, tids, toff = filters(rng, 300_000, 20, 300, 6, 10_000)
    held = set()
    for L in range(1000, 1500, 10):
        rii.rii_adc_scan_ivf(index, lut, probe, 20, tids, toff, L=L)
        held.add(index.info()["device_bytes"])
    assert len(held) <= 6


def test_no_set_reaches_the_lists(rii):
    """No target set is as large as the threshold: nothing is asked for that only lists with target sets need (400 MB for 4000 queries
    with a cap of 25,000), and the result is that of smaller batches."""
    index, rng = make(rii)
    index.set_threshold(30_000)
    Q, size = 4000, 20
    q = torch.from_numpy(rng.standard_normal((Q, 32)).astype(np.float32)).cuda()
    _, tids, toff = filters(rng, 300_000, 20, Q, 1, size)
    parts = [rii.rii_query(index, q[i:i + 50].contiguous(), 10, tids[i * size:(i + 50) * size].contiguous(), toff[:51].contiguous(), size, L=25_000)
             for i in range(0, Q, 50)]
    before = index.info()["device_bytes"]
    out = rii.rii_query(index, q, 10, tids, toff, size, L=25_000)
    torch.cuda.synchronize()
    # (tables, plan, probed lists and the scan's own scratch, a quarter more)
    assert index.info()["device_bytes"] < before + 1.25 * Q * (16 * 1024 + 8 + 20 * 4) + (64 << 20)
    assert torch.equal(out[0], torch.cat([p[0] for p in parts])) and torch.equal(out[1], torch.cat([p[1] for p in parts]))

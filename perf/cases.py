"""Performance cases: the work a user of this library has it do, through its public entry points.

A search service holds an index (codes of one database, usually with posting lists) and calls it
with one query at a time or with a batch; a loader encodes vectors and builds or extends the
index.  Six kinds of calls cover that:

  query   rii_query on a batch: tables, then the inverted index, or the linear scan where the index
          has no lists (the paper's Alg. 3 without a target set)
  scan    rii_build_lut + rii_adc_scan_linear: exhaustive search (Alg. 1 over the whole database)
  lists   rii_build_lut + rii_coarse_assign + rii_adc_scan_ivf: the inverted index with a fixed
          number of lists and no candidate cap (Alg. 2)
  subset  rii_build_lut + rii_adc_scan_subset: exhaustive search in each query's target set
  filter  rii_query with a target set per query, of very different sizes, so that both branches of
          Alg. 3 are taken inside one batch: the search in a subset that the method is about
  encode  rii_encode_device, after rii_rotate where the index belongs to the OPQ variant (Sec. 4.5)
  build   a new index from codes: add, reconfigure (Alg. 4), a second add that pushes into the lists

The data are those of the library's own configurations: SIFT-shaped, the Deep-shaped mixture, and
i.i.d. normal vectors for the tiny one.  Distances are defined to the last bit (fp32, sub-spaces
ascending, ties by identifier), so every output is compared exactly.
"""
import math
from dataclasses import replace

import torch

import paper_1808_03969_amd as rii
from paper_1808_03969_amd import workloads

# sub-spaces and dimensions that go together in the configurations and tests; 64 is what the paper
# uses on SIFT1M, 12 stands for the sizes without a kernel of their own
SHAPES = {8: 128, 12: 96, 16: 128, 32: 96, 64: 128}
TRAIN_ROWS, TRAIN_ITERS = 5_000, 3  # code books good enough for real code statistics, quick to make


def listed():
    return [
        # one request against a small collection: ten thousand vectors, no lists; latency and launches
        dict(name="one_small", kind="query", data="gaussian", M=8, D=128, N=10_000, K=0, Q=1, topk=10, L=1),
        # one request against a million vectors with lists: what an interactive service sends most
        dict(name="one_lists", kind="query", data="sift", M=16, D=128, N=1_000_003, K=1_000, Q=1, topk=100, L=8_000),
        # one exact request over a hundred million codes: the memory stream itself
        dict(name="one_scan_large", kind="scan", data="mixture", M=32, D=96, N=100_000_000, K=0, Q=1, topk=100, L=1),
        # the SIFT-shaped batch, exhaustive
        dict(name="batch_scan", kind="scan", data="sift", M=16, D=128, N=1_000_000, K=0, Q=10_000, topk=100, L=1),
        # an exhaustive batch over an array larger than the caches, ragged in rows and queries
        dict(name="batch_scan_large", kind="scan", data="mixture", M=32, D=96, N=30_000_001, K=0, Q=2_499, topk=100, L=1),
        # the SIFT-shaped batch through the lists
        dict(name="batch_lists", kind="lists", data="sift", M=16, D=128, N=1_000_000, K=1_000, Q=10_000, topk=100, nprobe=8),
        # a clustered batch through the lists of a large index
        dict(name="batch_lists_large", kind="lists", data="mixture", M=32, D=96, N=16_000_000, K=4_096, Q=4_001, topk=100,
             nprobe=64),
        # the paper's setting on SIFT1M: 64 sub-spaces, nearest neighbour, 5000 candidates
        dict(name="lists_m64", kind="query", data="sift", M=64, D=128, N=1_000_000, K=1_000, Q=777, topk=1, L=5_000),
        # target sets of one per cent of the database, exhaustive
        dict(name="subset_scan", kind="subset", data="sift", M=16, D=128, N=1_000_000, K=0, Q=1_000, topk=100, s_min=10_000,
             s_max=10_000),
        # target sets from a hundred identifiers to the whole database, the switch at the paper's crossover
        dict(name="filter_mixed", kind="filter", data="sift", M=16, D=128, N=1_000_000, K=1_000, Q=500, topk=100, L=1_000,
             s_min=100, s_max=1_000_000, theta=25_000),
        # the database side of the OPQ variant: rotate and encode a load of new vectors
        dict(name="encode_rotated", kind="encode", data="sift", M=16, D=128, N=500_000, rotate=True),
        # a new index with lists, then a fifth more vectors pushed into them
        dict(name="build_and_add", kind="build", data="mixture", M=16, D=96, N=1_000_000, K=1_000, iters=2),
    ]


def _log_int(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm; nearly always an odd size."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    """Table look-ups (or code-word distances) of a pass, dearer where one query is scanned at a time."""
    per_query = case["M"] not in (8, 16, 32) or case.get("topk", 1) > 100
    return work(case)["flops"] * (16 if per_query else 1)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["query", "scan", "lists", "subset", "filter", "query", "scan", "lists", "encode", "build"])
        M = rng.choice([8, 16, 16, 32, 32, 64, 12])
        D = SHAPES[M]
        # (the SIFT-shaped recipe has 128 coordinates, the mixture any number)
        data = rng.choice(["sift", "mixture"]) if D == 128 else "mixture"
        case = dict(kind=kind, data=data, M=M, D=D)
        if kind == "encode":
            case.update(N=_log_int(rng, 1_000, 1_000_000), rotate=rng.random() < 0.5)
            return case
        if kind == "build":
            N = _log_int(rng, 20_000, 1_500_000)
            case.update(N=N, K=_log_int(rng, 16, max(17, min(2_000, N // 100))), iters=rng.randint(1, 3))
            if _cost(case) <= most:
                return case
            continue
        N = _log_int(rng, 2_000, 20_000_000)
        Q = _log_int(rng, 1, 10_000)
        topk = rng.choice([1, 10, 100, 100, 100, 100, 128, 1_000])
        K = _log_int(rng, 16, max(17, min(4_096, N // 50)))
        case.update(N=N, Q=Q, topk=topk)
        if kind == "scan":
            case.update(K=0, L=1)
        elif kind == "query":
            K = 0 if rng.random() < 0.2 else K
            case.update(K=K, L=max(topk, (N // K) * rng.randint(1, 32)) if K else 1)
        elif kind == "lists":
            case.update(K=K, nprobe=min(K, _log_int(rng, 1, 128)))
        else:
            s_max = _log_int(rng, 100, min(N, 1_000_000))
            case.update(K=0, s_min=s_max if rng.random() < 0.5 else _log_int(rng, 10, s_max), s_max=s_max)
            if kind == "filter":
                case.update(K=K, L=max(topk, N // K), s_min=_log_int(rng, 10, s_max), theta=_log_int(rng, 1_000, 100_000))
            if sum(_sizes(case)) > 300_000_000:
                continue
        if _cost(case) <= most:
            return case


# ------------------------------------------------------------------ inputs
def _sizes(case):
    """Target-set sizes of the batch, spread evenly over the logarithm from s_min to s_max."""
    lo, hi, Q = case["s_min"], case["s_max"], case["Q"]
    return [int(round(lo * (hi / lo) ** ((i + 0.5) / Q))) for i in range(Q)]


def _rows(case, seed, r0, r1):
    cfg = replace(workloads.CONFIGS["c5"], D=case["D"], kind=case["data"])
    return workloads.rows(cfg, seed, r0, r1, "cuda")


def _codebooks(case, seed):
    train = _rows(case, 3_000_000 + seed, 0, TRAIN_ROWS).cpu().numpy()
    return rii.rii_train_codebooks(train, case["M"], iters=TRAIN_ITERS, seed=seed)


def _codes(index, case, seed, r0, r1):
    """Codes of database rows r0 .. r1-1, chunk by chunk."""
    for a in range(r0, r1, 2_000_000):
        b = min(r1, a + 2_000_000)
        yield rii.rii_encode_device(index, _rows(case, 1_000_000 + seed, a, b))


def _targets(case, seed):
    """A sorted uniform target set per query (duplicates of the draws dropped), in CSR form."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5_000_000 + seed)
    sizes = _sizes(case)
    order = torch.randperm(len(sizes), generator=g, device="cuda").tolist()  # large and small sets in no order
    N = case["N"]
    parts = []
    for i in order:
        s = sizes[i]
        if 4 * s > N:  # a large share of the database: every identifier with that probability
            hit = torch.rand(N, generator=g, device="cuda") < s / N
            parts.append(hit.nonzero().view(-1).to(torch.int32))
        else:
            parts.append(torch.unique(torch.randint(N, (s,), generator=g, device="cuda", dtype=torch.int32)))
    lengths = [p.numel() for p in parts]
    off = torch.zeros(len(parts) + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.tensor(lengths, dtype=torch.int64), 0)
    return torch.cat(parts), off.cuda(), max(lengths)


def prepare(case, seed):
    kind = case["kind"]
    cb = _codebooks(case, seed)
    index = rii.Index(cb)
    if kind == "encode":
        state = dict(case=case, index=index, x=_rows(case, 1_000_000 + seed, 0, case["N"]), R=None)
        if case["rotate"]:
            g = torch.Generator()
            g.manual_seed(seed)
            q, _ = torch.linalg.qr(torch.randn(case["D"], case["D"], generator=g))
            state["R"] = q.contiguous().cuda()
        return state
    if kind == "build":
        first = case["N"] * 4 // 5
        old = torch.cat(list(_codes(index, case, seed, 0, first)))
        new = torch.cat(list(_codes(index, case, seed, first, case["N"])))
        return dict(case=case, cb=cb, old=old, new=new, seed=seed)
    for codes in _codes(index, case, seed, 0, case["N"]):
        index.add(codes)
    if case["K"]:
        index.reconfigure(case["K"], iters=1, seed=seed)
    state = dict(case=case, index=index, q=_rows(case, 2_000_000 + seed, 0, case["Q"]))
    if kind in ("subset", "filter"):
        state["tids"], state["toff"], state["tmax"] = _targets(case, seed)
    if kind == "filter":
        index.set_threshold(case["theta"])
    return state


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "build":
        index = rii.Index(state["cb"])
        index.add(state["old"])
        index.reconfigure(case["K"], iters=case["iters"], seed=state["seed"])
        index.add(state["new"])
        return index.get_lists()  # what is written to disk beside the codes
    index = state["index"]
    if kind == "encode":
        x = state["x"] if state["R"] is None else rii.rii_rotate(state["R"], state["x"])
        return rii.rii_encode_device(index, x)
    topk = case["topk"]
    if kind == "query":
        return rii.rii_query(index, state["q"], topk, L=case["L"])
    if kind == "filter":
        return rii.rii_query(index, state["q"], topk, state["tids"], state["toff"], state["tmax"], L=case["L"])
    lut = rii.rii_build_lut(index, state["q"])
    if kind == "scan":
        return rii.rii_adc_scan_linear(index, lut, topk)
    if kind == "subset":
        return rii.rii_adc_scan_subset(index, lut, state["tids"], state["toff"], state["tmax"], topk)
    probe, d0 = rii.rii_coarse_assign(index, lut, case["nprobe"])
    return probe, d0, rii.rii_adc_scan_ivf(index, lut, probe, topk)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes: code books, queries, every code row and identifier that is needed once, results.
    Flops: three per coordinate of a table entry, one addition per look-up, as the definitions have it."""
    kind, M, D, N = case["kind"], case["M"], case["D"], case["N"]
    book = 256 * D * 4
    if kind == "encode":
        flops = 3 * 256 * D * N + (2 * D * D * N if case["rotate"] else 0)
        return dict(bytes=book + N * (4 * D + M) + (4 * D * D if case["rotate"] else 0), flops=flops)
    if kind == "build":
        K, first = case["K"], case["N"] * 4 // 5
        scored = case["iters"] * min(first, 100 * K) + N
        return dict(bytes=book + N * (M + M + 4 + 4) + K * (M + 8), flops=scored * K * M)
    Q, K, topk = case["Q"], case["K"], case["topk"]
    size = book + Q * D * 4 + Q * topk * 8
    flops = 3 * 256 * D * Q
    if kind == "scan" or (kind == "query" and not K):
        return dict(bytes=size + N * M, flops=flops + Q * N * M)
    if kind == "subset":
        total = sum(_sizes(case))
        return dict(bytes=size + 4 * total + min(N, total) * M, flops=flops + total * M)
    if kind == "lists":
        rows = Q * case["nprobe"] * N // K
        return dict(bytes=size + K * M + min(N, rows) * M + Q * case["nprobe"] * 8, flops=flops + (Q * K + rows) * M)
    L = min(case["L"], N)
    if kind == "query":
        return dict(bytes=size + K * M + min(N, Q * L) * M, flops=flops + Q * (K + L) * M)
    rows = ids = ranked = 0
    for s in _sizes(case):
        if s < case["theta"]:
            rows, ids = rows + s, ids + s
        else:  # ceil(K L / s) lists of N / K members are walked to find L members of the target set
            rows, ids, ranked = rows + min(L, s), ids + min(N, L * N // s), ranked + 1
    return dict(bytes=size + (K * M if ranked else 0) + 4 * ids + min(N, rows) * M, flops=flops + (ranked * K + rows) * M)


def tolerance(case):
    """Codes, identifiers and lists are whole numbers; distances are defined bit by bit (see above)."""
    return "exact"

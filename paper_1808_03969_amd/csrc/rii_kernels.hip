// HIP kernels (gfx950), their launchers and the device-side entry points of the library.
// The device code lives in the rii_dev_*.inc files included below; this file holds the host
// side: workspace layout, launch shapes (scan_chunks, plan_batch), dispatch on M and the
// extern "C" entry points.
//
// Data flow of one query batch:
//   k_build_lut              q, code books                        -> A [Q][M][256]       (Sec. 3)
//   k_few                    A in LDS, some 10^4 rows at most     -> top-R per query     (all of the following, small)
//   k_pick_members + k_few   lists' members in a target set       -> top-R per query     (Alg. 2, target ids and cap)
//   k_matrix_scan + k_few    A as a vector, codes decoded, MFMA   -> top-R per query     (Alg. 1, whole data, batches)
//   k_scan_w4 / k_scan_w     A in LDS, codes streamed             -> top-R per query     (Alg. 1, whole data)
//   k_scan_w<subset>         A in LDS, codes gathered by id       -> top-R per query     (Alg. 1, target ids)
//   k_rank_lists             A in LDS, coarse codes               -> nearest lists       (Alg. 2, first block)
//   k_ivf_w / k_ivf          A in LDS, probed lists streamed      -> top-R per query     (Alg. 2, second block)
//   k_list_products          A as a vector, lists decoded, MFMA   -> top-R per query     (Alg. 2, second block, batches)
//   k_scan + k_select, k_sort_segments: R above the per-wave kernels' reach, explicit candidates
//
// A candidate is one 64-bit key: order-preserving image of the fp32 distance in the high word,
// identifier in the low word.  Comparing keys as unsigned integers is the (distance,
// identifier) order, so selection is exact and deterministic including ties.

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "rii_internal.h"
#include "rii_bench.h"

#ifndef RII_SUBSET_GENERATION
#define RII_SUBSET_GENERATION 256
#endif

namespace {

// Device code, in dependency order (textual includes: everything shares this namespace).
#include "rii_dev_common.inc"
#include "rii_dev_adc.inc"
#include "rii_dev_scan_common.inc"
#include "rii_dev_scan_w.inc"
#include "rii_dev_scan_batched.inc"
#include "rii_dev_select.inc"
#include "rii_dev_coarse.inc"
#include "rii_dev_ivf.inc"
#include "rii_dev_few.inc"
#include "rii_dev_matrix.inc"
#include "rii_dev_lists.inc"
#include "rii_dev_offline.inc"
#include "rii_dev_bench.inc"

// ------------------------------------------------------------------ host helpers
int ensure_ws(const rii_index* idx, size_t bytes) {
  if (idx->ws_bytes >= bytes) return RII_OK;
  if (idx->ws) (void)hipFree(idx->ws);
  idx->ws = nullptr;
  idx->ws_bytes = 0;
  size_t want = bytes + bytes / 4;
  hipError_t e = hipMalloc(&idx->ws, want);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    e = hipMalloc(&idx->ws, bytes);
    want = bytes;
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return RII_ERR_OOM;
    }
  }
  idx->ws_bytes = want;
  return RII_OK;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

constexpr int64_t kBatchChunkBytes = (int64_t)384 << 20;  // rows of a large batch are scanned in chunks of about this size
constexpr int kCoarseSplitQ = 32, kCoarseSplitK = 8192;  // coarse ranking of few queries over many centres: distances first (see coarse_rank)
constexpr int kSubsetGeneration = RII_SUBSET_GENERATION;  // queries per launch of a subset scan with one block per query


bool m_supported(int M) { return M >= 4 && M <= RII_MAX_M && M % 4 == 0; }

// Per (device, kernel): the dynamic LDS size already granted with hipFuncSetAttribute, and whether
// the kernel was checked to have no static LDS.  Looked up on every launch, written once per
// kernel, so that the online calls make no runtime-attribute calls after their first launch.
struct KernelLdsState {
  size_t granted = 0;
  bool at_zero = false;
};
std::mutex g_lds_mutex;
std::unordered_map<uint64_t, KernelLdsState> g_lds_state;

uint64_t lds_key(const void* kern) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  return (uint64_t)reinterpret_cast<uintptr_t>(kern) * 64u + (uint64_t)(dev & 63);
}

// Allow `kern` to be launched with `bytes` of dynamic LDS.  need_zero: the kernel addresses its
// table as "LDS address 0", so it must not have static LDS in front of the dynamic allocation;
// refuse to launch otherwise (checked once per kernel).
int set_lds_impl(const void* kern, size_t bytes, bool need_zero) {
  std::lock_guard<std::mutex> lock(g_lds_mutex);
  KernelLdsState& st = g_lds_state[lds_key(kern)];
  if (need_zero && !st.at_zero) {
    hipFuncAttributes attr{};
    RII_HIP(hipFuncGetAttributes(&attr, kern));
    if (attr.sharedSizeBytes != 0) return RII_ERR_DEVICE;
    st.at_zero = true;
  }
  if (bytes > 48 * 1024 && bytes > st.granted) {
    RII_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    st.granted = bytes;
  }
  return RII_OK;
}

template <typename Kern>
int set_lds(Kern kern, size_t bytes) { return set_lds_impl(reinterpret_cast<const void*>(kern), bytes, false); }

// set_lds for the kernels whose table must sit at LDS address 0
template <typename Kern>
int set_lds0(Kern kern, size_t bytes) { return set_lds_impl(reinterpret_cast<const void*>(kern), bytes, true); }

#define DISPATCH_M(M, ...)                                  \
  switch (M) {                                              \
    case 8: { constexpr int MT = 8; __VA_ARGS__; } break;   \
    case 16: { constexpr int MT = 16; __VA_ARGS__; } break; \
    case 32: { constexpr int MT = 32; __VA_ARGS__; } break; \
    case 64: { constexpr int MT = 64; __VA_ARGS__; } break; \
    default: { constexpr int MT = 0; __VA_ARGS__; } break;  \
  }

// clear: see k_build_lut
void launch_build_lut(const rii_index* idx, const float* q, int Q, float* lut, hipStream_t st, void* clear = nullptr) {
  const int stride = (int)(align_up((size_t)Q * 4, 256) / 4);
  // Queries per block: enough blocks to fill the chip first (2048 of four waves are a chip-load),
  // then up to 16, where reading the code word no longer shows (10^4 queries, M = 16, 164 MB of
  // tables: 540 us with one query per block, 43 us with 16; at one query the blocks are what counts
  // and per is 1).
  const int per = std::min(16, std::max(1, (int)((int64_t)Q * idx->M / 2048)));
  const dim3 grid((unsigned)idx->M, (unsigned)((Q + per - 1) / per));
#define RII_LUT(DS) k_build_lut<DS><<<grid, 256, 0, st>>>(idx->d_cb, q, idx->D, idx->M, idx->Ds, Q, per, lut, static_cast<uint32_t*>(clear), stride)
  switch (idx->Ds) {
    case 2: RII_LUT(2); break;
    case 3: RII_LUT(3); break;
    case 4: RII_LUT(4); break;
    case 6: RII_LUT(6); break;
    case 8: RII_LUT(8); break;
    case 12: RII_LUT(12); break;
    case 16: RII_LUT(16); break;
    default: RII_LUT(0); break;
  }
#undef RII_LUT
}

// Split max_rows rows per query into equal chunks (one block each): about kWantBlocks blocks
// in total when the batch is small, never chunks shorter than kMinTiles tiles.
void scan_chunks(int Q, int64_t max_rows, int64_t* nchunks_out, int64_t* chunk_rows_out) {
  const int64_t tile = (int64_t)kScanThreads * kRowsPerLane;
  int64_t want = std::max<int64_t>(1, kWantBlocks / Q);  // rounded down: one block over a full round costs a second round
  int64_t most = std::max<int64_t>(1, (max_rows + kMinTiles * tile - 1) / (kMinTiles * tile));
  int64_t nchunks = std::min<int64_t>(std::min(want, most), 65535);
  int64_t chunk_rows = (max_rows + nchunks - 1) / nchunks;
  chunk_rows = std::max<int64_t>(tile, (chunk_rows + tile - 1) / tile * tile);
  *nchunks_out = std::max<int64_t>(1, (max_rows + chunk_rows - 1) / chunk_rows);
  *chunk_rows_out = chunk_rows;
}

// Launch shape of the batched kernel k_scan_w4 for Q queries over `rows` rows: groups of four
// queries (the last may be short) times row chunks.  Returns false when the kernel does not
// apply or would leave most of the chip idle (then the one-query kernels split the rows).
bool plan_batch(int M, int Q, int64_t rows, int topk, int64_t* nchunks_out, int64_t* chunk_rows_out) {
  *nchunks_out = 1;
  *chunk_rows_out = rows;
  if (!rot_m(M) || topk > kWaveK4 || Q < 4 || rows < 1) return false;
  const int64_t tile = (int64_t)kScanThreads * kRowsPerLane;
  const int64_t groups = (Q + 3) / 4;
  int64_t chunk_rows = (rows + tile - 1) / tile * tile, nchunks = 1;
  if (groups < 2 * kWantBlocks) {  // fewer than two full rounds of blocks from the groups alone
    const int64_t want = (kBatchWantBlocks + groups - 1) / groups;
    const int64_t most = std::max<int64_t>(1, rows / (kBatchMinTiles * tile));
    nchunks = std::min<int64_t>(std::min(want, most), 65535);
    // whole rounds of blocks (one block per CU): a part-filled last round takes as long as a full one
    if (groups * nchunks > kWantBlocks) nchunks = std::max<int64_t>(1, groups * nchunks / kWantBlocks * kWantBlocks / groups);
    chunk_rows = (rows + nchunks - 1) / nchunks;
    chunk_rows = (chunk_rows + tile - 1) / tile * tile;
    nchunks = (rows + chunk_rows - 1) / chunk_rows;
  } else if (rows * M > 2 * kBatchChunkBytes) {
    // A large batch over a large array: the rows are cut into chunks of about kBatchChunkBytes
    // all the same, chunk index slowest, so that the blocks resident at one time read the same
    // part of the array and the memory-side cache serves most of them.  With the abandoning
    // tests after every eight look-ups the kernel had become bound by the delivery of the code
    // bytes (10^4 queries over 10^8 rows of 32 bytes: 640 ms in one piece, 545 ms in nine).
    // ... or up to three times as many, so that the blocks make whole rounds of the chip: 625 groups over
    // 960 MB take 8 rounds for 7.3 rounds' worth of blocks in 3 chunks, 10 for 9.8 in 4 (41.7 and 39.5 ms;
    // half a per cent a chunk is what shorter chunks cost).
    const int64_t least = (rows * M + kBatchChunkBytes - 1) / kBatchChunkBytes;
    double best = 0.0;
    for (int64_t c = least; c <= 3 * least; ++c) {
      const double t = (double)((groups * c + kWantBlocks - 1) / kWantBlocks) / (double)c * (1.0 + 0.005 * (double)c);
      if (c == least || t < best) {
        best = t;
        nchunks = c;
      }
    }
    chunk_rows = (rows + nchunks - 1) / nchunks;
    chunk_rows = (chunk_rows + tile - 1) / tile * tile;
    nchunks = (rows + chunk_rows - 1) / chunk_rows;
  }
  if (groups * nchunks < kWantBlocks / 4) return false;  // (a quarter of the CUs busy with four queries each still wins)
  *nchunks_out = nchunks;
  *chunk_rows_out = chunk_rows;
  return true;
}

// Launch shape of k_few for Q queries of about `rows` rows each.
struct FewShape {
  int threads, split, slot, cap;
};
// A block hands over at most `slot` keys.  All of them together stay within kFewHandOver bytes; `tight` (scratch of a
// fixed size that would be exceeded): those of a query within the minima that scan_ws_bytes() counts for it (16 KB,
// 8 KB from four queries on), whatever the rows are.
constexpr int64_t kFewHandOver = (int64_t)16 << 20;
enum class FewRows { linear, targets, lists, capped };
FewShape few_shape(int M, int Q, int64_t rows, int k, FewRows kind, bool tight) {
  FewShape f;
  // By registers four blocks of four waves share a CU (M <= 16), two of eight above that; by LDS fewer for many
  // results (M = 64: one from 500 results on).
  f.threads = kind == FewRows::capped ? 1024 : M <= 16 ? 256 : 512;
  const int round = f.threads * (M == 8 || M == 16 ? 4 : 2);
  f.cap = round + std::max(512, 2 * k);
  f.slot = (k + std::max(k / 4, 16) + 15) / 16 * 16;
  f.split = 1;
  const int64_t rounds = (rows + round - 1) / round;
  if (kind == FewRows::capped || rounds < 4) return f;
  // Several blocks a query cost about 10 us (a launch that clears, handing over, merging), a round of a
  // block that has its CU to itself 2 us: below four rounds splitting loses, and once the queries
  // alone give every other CU a block it has to save four rounds (256 queries, M = 16: 2000 rows 41 us
  // in two blocks, 28 us in one; 32,000 rows 77 and 131 us).  Target sets of very different sizes would
  // leave the largest to run alone when there are few blocks a CU: those of many rounds are cut up
  // all the same (500 sets of up to 25,000: 73 -> 55 us).
  const bool full = Q > kWantBlocks / 2;
  const int64_t per_cu = std::min<int64_t>(M <= 16 ? 4 : 2, (int64_t)(160 * 1024 / few_lds(M, f.cap, 0, false)));
  int64_t want = full ? std::min<int64_t>(rounds / 4, per_cu * kWantBlocks / Q) : std::min<int64_t>(2, per_cu) * kWantBlocks / Q;
  const int64_t least = (Q < 4 ? 16384 : 8192) / (f.slot * 8);  // (few where many results make a block dear)
  if (kind == FewRows::targets && Q < 4 * kWantBlocks && rounds > 16) want = std::max(want, std::min(least, (rounds + 11) / 12));
  want = std::min(std::min(want, rounds), tight ? least : kFewHandOver / ((int64_t)Q * f.slot * 8));
  // A block more takes rounds off the others and gives the last one `slot` keys more to merge, about 1 us a thousand
  // (one query, M = 16, 65,536 rows, top-1000: 94, 82, 85, 102, 142 us in 4, 8, 16, 32, 64 blocks; 10^6 members,
  // top-300: 629, 343, 198, 130, 100 us in 4 .. 64); on a full chip the blocks also take turns at selecting
  // (256 sets of 16,000, M = 8, top-1000: 71 us in one block each, 90 in four; top-300: 61 in two, 80 in four).  The
  // best of the numbers of blocks whose rounds come out even.
  const float per_key = full ? 1.2e-2f : 1e-3f;
  const uint32_t all = (uint32_t)rounds;
  float best = 2.f * (float)all - 3.f;
  for (uint32_t n = 2; n <= (uint32_t)std::max<int64_t>(want, 1); ++n) {
    const uint32_t each = (all + n - 1) / n;
    if ((all + each - 1) / each != n) continue;  // fewer blocks have as many rounds
    const float t = 2.f * (float)each + per_key * (float)n * (float)f.slot;
    if (t < best) {
      best = t;
      f.split = (int)n;
    }
  }
  return f;
}
size_t few_ws_bytes(const FewShape& f, int Q) {
  return kScanArrays * align_up((size_t)Q * 4, 256) + (f.split > 1 ? (size_t)Q * f.split * f.slot * 8 : 0) + 256;
}

// The bounds and counters of a scan in several blocks a query, at the start of its scratch.
void clear_few(const FewShape& f, int Q, void* ws, hipStream_t st) {
  const size_t cstride = align_up((size_t)Q * 4, 256) / 4;
  if (f.split > 1) k_init_scan<<<(Q + 255) / 256, 256, 0, st>>>(static_cast<uint32_t*>(ws), Q, (int)cstride, nullptr, 0);
}

// `ws` holds few_ws_bytes (looked at only when a query has several blocks); cleared: its bounds and counters
// are initialised already.
template <int SRC>
int launch_few(FewArgs a, const FewShape& f, int Q, void* ws, bool cleared, hipStream_t st) {
  a.cap = f.cap;
  a.slot = f.slot;
  a.filter_ids = a.target_ids;
  a.filter_offsets = a.target_offsets;
  if (f.split > 1) {
    const size_t cstride = align_up((size_t)Q * 4, 256) / 4;
    uint32_t* tau = static_cast<uint32_t*>(ws);
    a.tau_g = tau; a.done_cnt = tau + 3 * cstride;
    a.cand = reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(ws) + kScanArrays * cstride * 4);
    if (!cleared) clear_few(f, Q, ws, st);
  }
  const size_t lds = few_lds(a.M, a.cap, a.nprobe, SRC == kFewCapped);
  const dim3 grid((unsigned)f.split, (unsigned)Q);
  DISPATCH_M(a.M, { int rc = set_lds0(k_few<MT, SRC>, lds); if (rc) return rc;
                    k_few<MT, SRC><<<grid, f.threads, lds, st>>>(a); });
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// Rows per query up to which a scan goes to k_few (of lists: what list_rows() says, which for clustered data is about
// twice the mean).  Measured against the streaming kernels (which it would otherwise go to) for batches of 1 .. 4000
// queries, every M, top-1 to top-1000; microseconds there / here.  The streaming kernels lose to their fixed cost and,
// for many results, to their selection; with few results, many queries or M = 32 (rows abandoned half-way) they catch
// up early:
//   whole array  M = 16:  1 query, top-100 64,000 rows 56 / 33, top-1000 200 / 82;  600 queries, top-100 32,000 158 /
//     108, 64,000 186 / 188, top-10 16,000 82 / 62, 32,000 92 / 102;  M = 32:  600 queries, top-100 16,000 151 / 108,
//     32,000 217 / 196
//   lists (mean lengths)  M = 16:  4000 queries, top-100 64,000 members 1431 / 912, top-10 32,000 616 / 514;  1 query,
//     top-300 10^6 1683 / 100;  M = 32:  4000 queries, top-100 32,000 1346 / 1053, top-10 4,000 406 / 278, 16,000
//     643 / 676.  Where the queries make whole rounds of the chip in the streaming kernel it is ahead before the
//     line: M = 16, top-10, 16,000 members, 64 queries 33 / 34, 256 queries 43 / 48 (but 130 queries 59 / 43).
//     Zipf-like lengths, M = 16, 256 queries, two lists, top-1 283 / 969: beyond the line by list_rows()
//   target sets  M = 16:  64 queries, top-100 64,000 ids 126 / 63;  200 queries, top-100 16,000 72 / 57, 32,000
//     95 / 105;  4000 queries, top-100 64,000 2396 / 2424, top-10 16,000 787 / 555, 32,000 1289 / 1230
constexpr int kFewManyResults = 64;
bool few_linear(int M, int Q, int topk, int64_t rows) {
  const bool many = topk >= kFewManyResults;
  if (Q <= 4) return rows <= 65536;
  if (!rot_m(M)) return rows <= (many ? 65536 : 16000);
  if (Q <= kWantBlocks) return rows <= (many ? 65536 : M == 32 ? 12000 : 32000);
  return rows <= (many ? (M == 32 ? 24000 : 40000) : M == 32 ? 10000 : 16000);
}
bool few_lists(int M, int Q, int topk, int64_t rows) {
  if (topk >= kFewManyResults) return rows <= (M == 32 || M == 64 ? 58000 : 110000);
  return rows <= (Q <= 4 ? 120000 : M == 32 ? 20000 : 40000);
}
bool few_subset(int Q, int topk, int64_t rows) {
  const bool many = topk >= kFewManyResults;
  if (Q <= 64) return rows <= 65536;
  if (Q <= 400) return rows <= (many ? 16000 : 12000);
  return rows <= (many ? 50000 : 24000);
}

bool few_scan(int mode, int M, int Q, int topk, int64_t rows) {
  return mode == kLinear ? few_linear(M, Q, topk, rows) : few_subset(Q, topk, rows);
}

// Scan `nrows_max` rows per query (linear: the whole array) and leave per-block partial keys in
// the workspace; then select.  Workspace layout: [tau Q u32][partial Q*nchunks*k u64].
int launch_scan(const rii_index* idx, const uint8_t* codes, int64_t plane, int64_t N, const float* lut, int Q, int mode,
                const int32_t* target_ids, const int64_t* target_offsets, int64_t max_rows, int topk,
                int32_t* ids, float* dist, int out_stride, const int* qmode, int want_mode, void* ws_base,
                hipStream_t st, bool cleared = false, bool tight = false) {
  const int M = idx->M;
  if (Q > 65535) return RII_ERR_UNSUPPORTED;
  const bool timed = mode == kLinear && idx->ev_start && idx->ev_stop && codes == idx->d_codes;
  if (few_scan(mode, M, Q, topk, max_rows) && !idx->bench_half_table) {
    FewArgs f{};
    f.codes = codes; f.plane = plane; f.M = M; f.lut = lut; f.N = N; f.target_ids = target_ids; f.target_offsets = target_offsets;
    f.k = topk; f.ids = ids; f.dist = dist; f.out_stride = out_stride; f.qmode = qmode; f.want_mode = want_mode;
    const FewShape shape = few_shape(M, Q, max_rows, topk, mode == kSubset ? FewRows::targets : FewRows::linear, tight);
    if (mode == kSubset) return launch_few<kFewSubset>(f, shape, Q, ws_base, cleared, st);
    if (!cleared) clear_few(shape, Q, ws_base, st);
    if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_start), st));
    const int rc = launch_few<kFewLinear>(f, shape, Q, ws_base, true, st);
    if (timed && !rc) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_stop), st));
    return rc;
  }
  int64_t nchunks, chunk_rows;
  scan_chunks(Q, max_rows, &nchunks, &chunk_rows);

  // workspace: [tau Q][candidate count Q][prepass counter Q][blocks done Q] u32, then
  // [candidates], then [prepass minima]
  // (the four arrays start 256-byte aligned so that, for a single query, the much-read bound
  // does not share a cache line with the counters the blocks update)
  uint8_t* base = static_cast<uint8_t*>(ws_base);
  const size_t cstride = align_up((size_t)Q * 4, 256) / 4;
  uint32_t* tau = reinterpret_cast<uint32_t*>(base);
  uint32_t* cand_cnt = tau + cstride;
  uint32_t* pre_counter = tau + 2 * cstride;
  uint32_t* done_cnt = tau + 3 * cstride;
  uint64_t* partial = reinterpret_cast<uint64_t*>(base + kScanArrays * cstride * 4);

  ScanArgs a{};
  a.codes = codes; a.plane = plane; a.N = N; a.M = M; a.lut = lut;
  a.target_ids = target_ids; a.target_offsets = target_offsets;
  a.chunk_rows = chunk_rows; a.k = topk; a.partial = partial; a.tau_g = tau;
  int64_t bchunks, brows;
  const bool batched = mode == kLinear && !qmode && plan_batch(M, Q, max_rows, topk, &bchunks, &brows);
  if (!batched) bchunks = 1;
  a.cand_cnt = cand_cnt; a.cand_cap = std::max(nchunks, bchunks) * topk;
  a.nq = Q;
  // [prepass minima] follow the candidates
  uint32_t* minima = reinterpret_cast<uint32_t*>(partial + (size_t)Q * a.cand_cap);
  a.done_cnt = done_cnt; a.ids = ids; a.dist = dist; a.out_stride = out_stride;
  a.qmode = qmode; a.want_mode = want_mode;
  dim3 grid((unsigned)nchunks, (unsigned)Q);
  a.counters = timed ? idx->d_scan_counters : nullptr;
  if (topk <= kWaveK || rot_m(M)) {  // (rotated stored form: k_scan_w up to RII_MAX_TOPK, with a block-level buffer above kWaveK)
    // When a query's rows are split over several blocks, a short first pass over the leading
    // rows seeds the shared bound, so that the main pass starts with few candidates.
    const int64_t tile_rows = (int64_t)kScanThreads * kRowsPerLane;
    const int64_t tiles = (max_rows + tile_rows - 1) / tile_rows;
    int pre_blocks = (int)std::min<int64_t>(kPrepassBlocks, tiles);
    if (Q >= 4) {
      // Many queries: the seeding blocks no longer run side by side, each costs a table fill, and
      // on a small array 256 of them per query would score all of it once more.  A thirty-second
      // of the rows, and never more than 128 blocks, is enough for a useful bound, as long as
      // there are at least topk wave minima.
      const int64_t least = std::min<int64_t>(tiles, (topk + kScanThreads / 64 - 1) / (kScanThreads / 64) + 1);
      pre_blocks = (int)std::max<int64_t>(least, std::min<int64_t>(std::min(pre_blocks, kPrepassBlocks / 2), tiles / 32));
    }
    // The single-query kernel seeds the bound itself when all its blocks run at once and a query
    // has at least topk of them (rotated form only); otherwise a separate pass does it.
    // ... from its blocks' minima (at most 64 kSeedPerLane blocks), or from its waves' when it
    // has fewer than topk blocks but enough waves
    const int waves = kScanThreads / 64;
    const bool resident = nchunks > 1 && rot_m(M) && !batched && (int64_t)Q * nchunks <= kWantBlocks;
    const bool seed_blocks = resident && nchunks >= topk && nchunks <= 64 * kSeedPerLane;
    const bool seed_waves = resident && !seed_blocks && nchunks * waves >= topk && nchunks * waves <= 64 * kSeedPerLane;
    const bool seed_inside = seed_blocks || seed_waves;
    const bool prepass = nchunks > 1 && !seed_inside;
    a.seed_inside = seed_blocks ? 1 : seed_waves ? 2 : 0;
    const int nzero = seed_blocks ? Q * (int)nchunks : seed_waves ? Q * (int)nchunks * waves : 0;
    k_init_scan<<<(std::max(Q, nzero) + 255) / 256, 256, 0, st>>>(tau, Q, (int)cstride, minima, nzero);
    if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_start), st));
    a.minima = minima;
    a.counter = pre_counter;
    ScanArgs pre = a;
    pre.minima = minima;
    pre.counter = pre_counter;
    dim3 pgrid((unsigned)pre_blocks, (unsigned)Q);
    const size_t ldsw = table_bytes(M) + (size_t)(kScanThreads / 64 + 1) * kWaveCap * 8 + kBlockVarsBytes;
    const size_t lds4 = 65536 + 4 * (size_t)(kScanThreads / 64 + 1) * kWaveCap4 * 8 +
                        (size_t)(kScanThreads / 64) * kRescoreCap * 8 + kBlockVarsBytes + 4 * kBins4 * 4;
    const size_t lds2 = 65536 + 2 * (size_t)(kScanThreads / 64 + 1) * kWaveCap * 8 + kBlockVarsBytes;
    if (batched) {
      // Four queries per block with the integer-table filter; the rows are cut into chunks
      // when the groups alone would not fill the chip, and then the bound-seeding pass runs
      // first so that no block starts without a bound.
      ScanArgs a4 = a;
      a4.chunk_rows = brows;
      const dim3 g4((unsigned)((Q + 3) / 4), (unsigned)bchunks);
      // (no seeding pass for a large batch that is chunked for the cache's sake: its first chunk's
      // blocks find their bounds as an unchunked scan does, the later ones read the query's bound)
      const bool pre4 = bchunks > 1 && (Q + 3) / 4 < 2 * kWantBlocks;
      if (pre4) {
        switch (M) {
          case 8: { int rc = set_lds0(k_tau0<8, kLinear>, tau0_lds(M) + kBlockVarsBytes); if (rc) return rc;
                    k_tau0<8, kLinear><<<pgrid, kScanThreads, tau0_lds(M) + kBlockVarsBytes, st>>>(pre); } break;
          case 16: { int rc = set_lds0(k_tau0<16, kLinear>, tau0_lds(M) + kBlockVarsBytes); if (rc) return rc;
                     k_tau0<16, kLinear><<<pgrid, kScanThreads, tau0_lds(M) + kBlockVarsBytes, st>>>(pre); } break;
          default: { int rc = set_lds0(k_tau0<32, kLinear>, tau0_lds(M) + kBlockVarsBytes); if (rc) return rc;
                     k_tau0<32, kLinear><<<pgrid, kScanThreads, tau0_lds(M) + kBlockVarsBytes, st>>>(pre); } break;
        }
      }
      if (idx->bench_half_table) {  // the separately evaluated half-precision table (measurement entry point only)
        switch (M) {
          case 8: { int rc = set_lds0(k_scan_w4<8, true>, lds4); if (rc) return rc;
                    k_scan_w4<8, true><<<g4, kScanThreads, lds4, st>>>(a4); } break;
          case 16: { int rc = set_lds0(k_scan_w4<16, true>, lds4); if (rc) return rc;
                     k_scan_w4<16, true><<<g4, kScanThreads, lds4, st>>>(a4); } break;
          default: { int rc = set_lds0(k_scan_w4<32, true>, lds4); if (rc) return rc;
                     k_scan_w4<32, true><<<g4, kScanThreads, lds4, st>>>(a4); } break;
        }
      } else {
        switch (M) {
          case 8: { int rc = set_lds0(k_scan_w4<8>, lds4); if (rc) return rc;
                    k_scan_w4<8><<<g4, kScanThreads, lds4, st>>>(a4); } break;
          case 16: { int rc = set_lds0(k_scan_w4<16>, lds4); if (rc) return rc;
                     k_scan_w4<16><<<g4, kScanThreads, lds4, st>>>(a4); } break;
          default: { int rc = set_lds0(k_scan_w4<32>, lds4); if (rc) return rc;
                     k_scan_w4<32><<<g4, kScanThreads, lds4, st>>>(a4); } break;
        }
      }
    } else if (mode == kLinear && rot_m(M) && nchunks == 1 && !qmode && Q >= 2 && topk > kWaveK4 && topk <= kWaveK) {
      // Large batch with topk beyond the four-query kernel's reach: two queries per block
      // (k_scan_w2), every block owning its queries' whole scan, and a single-query block for an
      // odd one left over, addressed as query 0 of argument arrays shifted by Q - 1.
      auto shifted = [&](int o) {
        ScanArgs b = a;
        b.lut = lut + (size_t)o * M * 256;
        b.partial = partial + (size_t)o * a.cand_cap;
        b.tau_g = tau + o; b.cand_cnt = cand_cnt + o; b.done_cnt = done_cnt + o;
        b.ids = ids + (size_t)o * out_stride;
        b.dist = dist ? dist + (size_t)o * out_stride : nullptr;
        return b;
      };
      const dim3 g2(1, (unsigned)(Q / 2));
      switch (M) {
        case 8: { int rc = set_lds0(k_scan_w2<8>, lds2); if (rc) return rc;
                  k_scan_w2<8><<<g2, kScanThreads, lds2, st>>>(a); } break;
        case 16: { int rc = set_lds0(k_scan_w2<16>, lds2); if (rc) return rc;
                   k_scan_w2<16><<<g2, kScanThreads, lds2, st>>>(a); } break;
        default: { int rc = set_lds0(k_scan_w2<32>, lds2); if (rc) return rc;
                   k_scan_w2<32><<<g2, kScanThreads, lds2, st>>>(a); } break;
      }
      if (Q & 1) {
        ScanArgs b = shifted(Q - 1);
        switch (M) {
          case 8: { int rc = set_lds0(k_scan_w<8, kLinear>, ldsw); if (rc) return rc;
                    k_scan_w<8, kLinear><<<dim3(1, 1), kScanThreads, ldsw, st>>>(b); } break;
          case 16: { int rc = set_lds0(k_scan_w<16, kLinear>, ldsw); if (rc) return rc;
                     k_scan_w<16, kLinear><<<dim3(1, 1), kScanThreads, ldsw, st>>>(b); } break;
          default: { int rc = set_lds0(k_scan_w<32, kLinear>, ldsw); if (rc) return rc;
                     k_scan_w<32, kLinear><<<dim3(1, 1), kScanThreads, ldsw, st>>>(b); } break;
        }
      }
    } else if (mode == kLinear) {
      DISPATCH_M(M, { int rc = set_lds0(k_scan_w<MT, kLinear>, ldsw); if (rc) return rc;
                      if (prepass) { int rc2 = set_lds0(k_tau0<MT, kLinear>, tau0_lds(M) + kBlockVarsBytes); if (rc2) return rc2; }
                      if (prepass) k_tau0<MT, kLinear><<<pgrid, kScanThreads, tau0_lds(M) + kBlockVarsBytes, st>>>(pre);
                      k_scan_w<MT, kLinear><<<grid, kScanThreads, ldsw, st>>>(a); });
    } else {
      // One block per query and more queries than the chip holds blocks: the queries are launched
      // a chip-load at a time.  Target lists are sorted, so the blocks of one launch walk the code
      // array from its start to its end together, and a memory line that holds rows of several
      // queries' targets is fetched once for all of them while it stays in the memory-side cache
      // (with all queries in one launch the resident blocks are spread over the whole array).
      const int per_launch = nchunks == 1 && Q > kSubsetGeneration ? kSubsetGeneration : Q;
      for (int o = 0; o < Q; o += per_launch) {
        ScanArgs b = a;
        b.lut = lut + (size_t)o * M * 256;
        b.target_offsets = target_offsets + o;
        b.qmode = qmode ? qmode + o : nullptr;
        b.partial = partial + (size_t)o * a.cand_cap;
        b.tau_g = tau + o; b.cand_cnt = cand_cnt + o; b.done_cnt = done_cnt + o;
        b.ids = ids + (size_t)o * out_stride;
        b.dist = dist ? dist + (size_t)o * out_stride : nullptr;
        const dim3 g((unsigned)nchunks, (unsigned)std::min(per_launch, Q - o));
        DISPATCH_M(M, { int rc = set_lds0(k_scan_w<MT, kSubset>, ldsw); if (rc) return rc;
                        if (prepass) { int rc2 = set_lds0(k_tau0<MT, kSubset>, tau0_lds(M) + kBlockVarsBytes); if (rc2) return rc2; }
                        if (prepass) k_tau0<MT, kSubset><<<pgrid, kScanThreads, tau0_lds(M) + kBlockVarsBytes, st>>>(pre);
                        k_scan_w<MT, kSubset><<<g, kScanThreads, ldsw, st>>>(b); });
      }
    }
  } else {
  k_init_scan<<<(Q + 255) / 256, 256, 0, st>>>(tau, Q, (int)cstride, nullptr, 0);
  if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_start), st));
  const size_t lds = (size_t)M * 1024 + (size_t)kSelCap * 8;
  if (mode == kLinear) {
    DISPATCH_M(M, { int rc = set_lds(k_scan<MT, kLinear>, lds); if (rc) return rc;
                    k_scan<MT, kLinear><<<grid, kScanThreads, lds, st>>>(a); });
  } else {
    DISPATCH_M(M, { int rc = set_lds(k_scan<MT, kSubset>, lds); if (rc) return rc;
                    k_scan<MT, kSubset><<<grid, kScanThreads, lds, st>>>(a); });
  }
  }
  if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_stop), st));
  if (topk > kWaveK) {
    SelectArgs s{};
    s.keys = partial; s.nkeys = a.cand_cap; s.key_cnt = cand_cnt; s.k = topk; s.out_stride = out_stride;
    s.ids = ids; s.dist = dist; s.qmode = qmode; s.want_mode = want_mode;
    k_select<><<<Q, kScanThreads, 0, st>>>(s);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// Minima of the bound-seeding pass: it only runs when the rows of a query are cut into chunks,
// which launches of kSeedMaxQ or more queries never do, and with four or more queries it has
// at most kPrepassBlocks / 2 blocks per query (see launch_scan).
constexpr int kSeedMaxQ = 2048;
static_assert(kSeedMaxQ >= 8 * kWantBlocks, "batches that are cut into row chunks have fewer than 2 * kWantBlocks groups of four");
size_t minima_bytes(int Q) {
  const size_t blocks = Q < 4 ? kPrepassBlocks : kPrepassBlocks / 2;
  return (size_t)std::min(Q, kSeedMaxQ) * blocks * (kScanThreads / 64) * 4;
}

// What launch_scan needs.  batch: the call may take the batched kernel (no per-query modes); tight: see few_shape.
size_t scan_ws_bytes(int mode, int M, int Q, int64_t max_rows, int topk, bool batch = true, bool tight = false) {
  int64_t nchunks, chunk_rows;
  scan_chunks(Q, max_rows, &nchunks, &chunk_rows);
  int64_t bchunks = 1, brows;
  if (batch) plan_batch(M, Q, max_rows, topk, &bchunks, &brows);
  const int64_t cap_chunks = std::max(nchunks, bchunks);
  const size_t few = few_scan(mode, M, Q, topk, max_rows)
                         ? few_ws_bytes(few_shape(M, Q, max_rows, topk, mode == kSubset ? FewRows::targets : FewRows::linear, tight), Q) : 0;
  return std::max(few, kScanArrays * align_up((size_t)Q * 4, 256) + (size_t)Q * cap_chunks * topk * 8 + minima_bytes(Q) + 256);
}

// The same for every batch of at most Q queries, at most max_rows rows and at most topk results:
// a bound that grows with each argument (a batch's blocks per query times its queries stay
// below Q + 4 kBatchWantBlocks + kWantBlocks whatever the launch shape is, but for the chunks of a large batch over a
// large array, which only the kernel for up to kWaveK4 results makes).
size_t scan_ws_bound(int M, int Q, int64_t max_rows, int topk) {
  const size_t big_chunks = (size_t)(3 * (max_rows * M / kBatchChunkBytes + 1) + 2);  // (see plan_batch)
  const size_t keys = std::max((size_t)Q * big_chunks * std::min(topk, kWaveK4), (size_t)Q * topk) +
                      (size_t)(4 * kBatchWantBlocks + kWantBlocks + 8) * topk;
  return kScanArrays * align_up((size_t)Q * 4, 256) +
         std::max(keys * 8 + std::max(minima_bytes(Q), minima_bytes(std::min(Q, 3))), (size_t)kFewHandOver) + 256;
}

// ------------------------------------------------------------------ the batched scan by matrix products
// Which calls: see matrix_applies.  Scratch behind launch_left's.
struct MatrixPlan {
  int nf, Qp, cap;
  size_t qfrag, cq, lo, hi, mode, cnt, left, dist, cand, minima, part, total;  // byte offsets, size
};
constexpr int64_t kMatrixMinRows = (int64_t)1 << 18;
constexpr double kMatrixGrowth = 5.0;  // rows of a round against those before it
// From so many queries and rows on (microseconds by look-ups / here, M = 16 and D = 128 unless said; "clustered": rows
// collapsed onto 1000 codes, which list more): the launches of its rounds are 80 us that few queries do not bring back, and it
// looks at 32 queries at a time.
//   64 queries, 4 x 10^6 rows, top-10 318 / 446, top-100 408 / 489;  128 queries, top-10 516 / 495, top-100 600 / 549,
//   270,000 rows top-100 251 / 122, clustered 251 / 141, 1.6 x 10^7 rows top-100 1553 / 1616;  256 queries over 270,000, top-10
//   206 / 107, clustered 230 / 140;  256 over 1.6 x 10^7, top-100 clustered 3122 / 2043;  2048 over 10^6, top-100 1242 / 848
//   many results are scored one query a block: 256 queries, 270,000 rows, top-1000 466 / 459 (M = 8 392 / 453), 10^6 rows
//   863 / 675;  512 queries 887 / 609
//   without a look-up kernel for several queries a block:  M = 64, 512 queries, 10^6 rows 5668 / 392, 64 queries ahead by 1.7
//   from 262,144 rows on;  M = 20 by 1.03;  M = 12, D = 96, 400,000 rows, 64 queries top-10 102 / 118, top-100 157 / 161, 80
//   queries ahead by 1.14, 10^6 rows, 64 queries by 1.2 (D = 48: 0.90 to 1.04 and 1.3 with 64);  M = 4 has so few look-ups that it takes, with D = 128,
//   384 queries below 786,432 rows (256: 0.81 to 1.3, 384: 1.5 and more), 192 from there (128: 0.83, 192: 1.38), 96 from 2^21
//   (2.5 x 10^6: 64 queries 253 / 362, 96 ahead by 1.17), with D = 64 half of each.  (More than 512 results and M = 4, D = 128: from
//   0.75, 70 queries over 524,800 rows 332 / 440, to 1.5, 192 over 10^6.)
//   A batch that fills one round of the four-query kernel's blocks, M = 8, 400,000 rows:  top-10 640 queries 0.97 times as
//   fast here, 1024 0.77;  top-100 768 1.01, 1024 0.87;  M = 16 top-10 900 0.97.  (D = 64 and less: 0.97 and more.)
bool matrix_applies(const rii_index* idx, int Q, int topk, int64_t rows) {
  const int M = idx->M, D = idx->D;
  if (!idx->mx_book || idx->bench_half_table || rows < kMatrixMinRows) return false;
  if (topk > kWaveK && Q < 512 && rows < 2 * kMatrixMinRows) return false;
  const bool many = topk >= kFewManyResults;
  if (!rot_m(M)) {
    int least = 64;
    if (M == 4 && topk <= 512) least = std::max(80, (D > 64 ? 384 : 192) >> (rows >= 8 * kMatrixMinRows ? 2 : rows >= 3 * kMatrixMinRows ? 1 : 0));
    else if (M <= 12 && topk <= kWaveK && D > 64 && rows < 4 * kMatrixMinRows) least = 80;
    return Q >= least;
  }
  if (Q < (many && rows <= 32 * kMatrixMinRows ? 128 : 256)) return false;
  int64_t chunks, chunk_rows;
  if (M <= 16 && D > 64 && topk <= kWaveK4 && Q <= 4 * kWantBlocks && rows < 3 * kMatrixMinRows &&
      plan_batch(M, Q, rows, topk, &chunks, &chunk_rows) && chunks == 1)
    return Q <= (M == 8 ? (many ? 800 : 576) : many || D <= 96 ? 4 * kWantBlocks : 864);
  return true;
}
// Places of a query's list.  A round is expected to list five to ten times topk rows; where clusters have collapsed onto few
// codes, all rows that share the bound's distance with them, which is what the places above the least are for: as many
// as 512 MB of lists allow, an eighth of the rows at most.  Microseconds by look-ups / with lists of
// the least and N / 1024 places / here (M = 16, top-100):  250 clusters of 1.6 x 10^7 rows, 2048 queries 26,700 / 35,200 /
// 14,100, 256 queries 4240 / 5840 / 3080;  1000 clusters of 10^8, 1024 queries 53,900 / 73,300 / 30,500;  100 clusters of
// 10^6, 256 queries 750 / 930 / 570.
constexpr size_t kMatrixLists = (size_t)512 << 20;
int matrix_least(const rii_index* idx, int topk) { return 16 * topk + 4096 + (int)std::min<int64_t>(idx->N / 1024, 32768); }
int matrix_most(const rii_index* idx, int Q, int topk) {
  const int64_t least = matrix_least(idx, topk);
  return (int)std::max(least, std::min<int64_t>(least + idx->N / 8, kMatrixLists / 4 / Q));
}
MatrixPlan matrix_plan(const rii_index* idx, int Q, int topk, int cap) {
  const int D = idx->D, M = idx->M;
  MatrixPlan p;
  p.nf = (D + 31) / 32 * 2;
  p.Qp = (Q + 31) / 32 * 32;
  p.cap = cap;
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t o = at; at += align_up(bytes, 256); return o; };
  p.qfrag = take((size_t)p.Qp * p.nf * 32);
  p.cq = take((size_t)p.Qp * 4);
  p.lo = take((size_t)p.Qp * 4);
  p.hi = take((size_t)p.Qp * 4);
  p.mode = take((size_t)p.Qp * 4);
  p.cnt = take((size_t)p.Qp * kMxCntStride * 4);
  p.left = take(256 + (size_t)Q * 4);
  p.dist = take((size_t)Q * topk * 4);
  p.cand = take((size_t)Q * p.cap * 4);
  // (the fit's partial results are read before the groups' maxima are written)
  p.minima = p.part = take(std::max((size_t)kMxSeedGroups * 4, (size_t)M * 16) * p.Qp);
  p.total = at;
  return p;
}

// ---- what it leaves
// Row chunks of two rounds' groups of four and more (as plan_batch has them for the whole batch), 1 where there are none.
int64_t left_big(const rii_index* idx, int Q, int topk) {
  int64_t chunks = 1, rows;
  const bool many = (Q + 3) / 4 >= 2 * kWantBlocks;
  return rot_m(idx->M) && topk <= kWaveK4 && many && plan_batch(idx->M, Q, idx->N, topk, &chunks, &rows) ? chunks : 1;
}
// Bounds and counters by place, then candidates.
size_t left_ws_bytes(const rii_index* idx, int Q, int topk) {
  return kScanArrays * align_up((size_t)Q * 4, 256) + (size_t)left_lists(Q, left_big(idx, Q, topk)) * topk * 8;
}
// The linear scan for the queries that are entered in `left` (up to Q; their number is known on the device only, and usually
// 0): by the kernels of launch_scan, spread over the chip as their number asks for.  A launch of the whole batch's shape
// with the other queries' blocks gone left a query to one block, or dragged in its group's others (whole call, that way / here):
// one of 512 queries over 10^6 rows, M = 64, top-100 3240 / 507 us (none left: 392);  16 of 256 over 10^7, M = 16 2441 / 1332;
// 512 of 2048 over 10^6, M = 16 1906 / 1278, all of them 1751 / 1751;  one of 1024, top-300 1168 / 701.
// `big`: left_big of the batch that the scratch was sized for (a smaller one, its last piece, may ask for more chunks).
int launch_left(const rii_index* idx, const float* lut, int Q, int64_t big, int topk, int32_t* ids, float* dist, int out_stride,
                const LeftOut& left, hipStream_t st) {
  const int M = idx->M;
  ScanArgs a{};
  a.codes = idx->d_codes; a.plane = idx->plane_codes; a.N = idx->N; a.M = M; a.lut = lut; a.k = topk;
  a.tau_g = left.arrays; a.cand_cnt = left.arrays + left.stride; a.done_cnt = left.arrays + 3 * left.stride;
  a.partial = reinterpret_cast<uint64_t*>(left.arrays + kScanArrays * left.stride);
  a.ids = ids; a.dist = dist; a.out_stride = out_stride;
  a.left_n = left.n; a.left_q = left.q; a.left_big = (int)big; a.left_most = 0xFFFFFFFFu;
  auto blocks = [&](int per) { return (unsigned)left_blocks(per, Q, a.left_big); };
  const size_t ldsw = table_bytes(M) + (size_t)(kScanThreads / 64 + 1) * kWaveCap * 8 + kBlockVarsBytes;
  if (rot_m(M) && topk <= kWaveK4) {
    const size_t lds4 = 65536 + 4 * (size_t)(kScanThreads / 64 + 1) * kWaveCap4 * 8 +
                        (size_t)(kScanThreads / 64) * kRescoreCap * 8 + kBlockVarsBytes + 4 * kBins4 * 4;
#define RII_LEFT4(MT) { int rc = set_lds0(k_scan_w4<MT, false, true>, lds4); if (rc) return rc; \
                        k_scan_w4<MT, false, true><<<blocks(4), kScanThreads, lds4, st>>>(a); } break
    switch (M) {
      case 8: RII_LEFT4(8);
      case 16: RII_LEFT4(16);
      default: RII_LEFT4(32);
    }
#undef RII_LEFT4
  } else if (topk <= kWaveK || rot_m(M)) {
    if (rot_m(M) && topk <= kWaveK && Q > kWantBlocks) {  // more than a round of single queries: two a block
      a.left_most = kWantBlocks;
      const size_t lds2 = 65536 + 2 * (size_t)(kScanThreads / 64 + 1) * kWaveCap * 8 + kBlockVarsBytes;
#define RII_LEFT2(MT) { int rc = set_lds0(k_scan_w2<MT, true>, lds2); if (rc) return rc; \
                        k_scan_w2<MT, true><<<blocks(2), kScanThreads, lds2, st>>>(a); } break
      switch (M) {
        case 8: RII_LEFT2(8);
        case 16: RII_LEFT2(16);
        default: RII_LEFT2(32);
      }
#undef RII_LEFT2
    }
    DISPATCH_M(M, { int rc = set_lds0(k_scan_w<MT, kLeft>, ldsw); if (rc) return rc;
                    k_scan_w<MT, kLeft><<<blocks(1), kScanThreads, ldsw, st>>>(a); });
  } else {
    const size_t lds = (size_t)M * 1024 + (size_t)kSelCap * 8;
    if (M == 64) {
      int rc = set_lds(k_scan<64, kLeft>, lds); if (rc) return rc;
      k_scan<64, kLeft><<<blocks(1), kScanThreads, lds, st>>>(a);
    } else {
      int rc = set_lds(k_scan<0, kLeft>, lds); if (rc) return rc;
      k_scan<0, kLeft><<<blocks(1), kScanThreads, lds, st>>>(a);
    }
  }
  if (topk > kWaveK) {
    SelectArgs s{};
    s.keys = a.partial; s.key_cnt = a.cand_cnt; s.k = topk; s.out_stride = out_stride; s.ids = ids; s.dist = dist;
    s.left_n = left.n; s.left_q = left.q; s.left_rows = idx->N;
    k_select<true><<<Q, kScanThreads, 0, st>>>(s);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// What `q` queries of a batch need, what is left of them included.
size_t matrix_need(const rii_index* idx, int q, int topk, int cap) {
  return align_up(left_ws_bytes(idx, q, topk), 256) + matrix_plan(idx, q, topk, cap).total;
}

// Where a batch's products have their scratch, and how many queries fit it at a time; q = 0: the batch goes by look-ups.
struct MatrixScratch {
  int q = 0;    // queries at a time
  int cap = 0;  // places of a list
  void* at = nullptr;
};
// Queries at a time in `room` bytes, pieces of equal size as long as they are worth it, and the places that there is room for.
MatrixScratch matrix_fit(const rii_index* idx, int Q, int topk, size_t room) {
  MatrixScratch s;
  const int least = matrix_least(idx, topk);
  for (int pieces = 1;; ++pieces) {
    const int q = std::min(Q, ((Q + pieces - 1) / pieces + 31) / 32 * 32);
    if (!matrix_applies(idx, q, topk, idx->N)) return s;
    const size_t need = matrix_need(idx, q, topk, least);
    if (need > room) continue;
    s.q = q;
    s.cap = (int)std::min<size_t>(matrix_most(idx, q, topk), least + (room - need) / 256 * 256 / 4 / q);  // (areas are multiples of 256)
    return s;
  }
}
// The handle holds the `lead` bytes in front and what the look-up kernels need (`reserved`: and held them before the call, by
// rii_index_reserve_workspace); the products' scratch is an allocation of its own of 1 GB at most, so that asking for it, or
// asking in vain, leaves alone what served the look-ups, and what a captured graph of theirs reads.  It is not asked for in a
// reserved handle or while a graph is captured, and not moved once a graph holds it: pieces that fit what is there, or
// look-ups.  A device without room is asked for half as long as that is enough, and then for nothing in the next 64 calls.
constexpr size_t kMatrixScratch = (size_t)1 << 30;
constexpr int kMatrixPatience = 64;
MatrixScratch matrix_scratch(const rii_index* idx, int Q, int topk, size_t lead, bool reserved, hipStream_t st) {
  MatrixScratch s;
  if (!matrix_applies(idx, Q, topk, idx->N)) return s;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
  if (capturing) (void)hipGetLastError();
  const size_t behind = idx->ws_bytes - lead;
  if (!reserved && !capturing && !idx->mx_held && idx->mx_wait == 0) {
    for (size_t room = kMatrixScratch;; room /= 2) {
      const MatrixScratch fit = matrix_fit(idx, Q, topk, room);
      const size_t need = fit.q ? matrix_need(idx, fit.q, topk, fit.cap) : 0;
      if (need <= std::max(behind, idx->mx_ws_bytes)) break;
      void* bigger = nullptr;
      if (need <= idx->mx_most && hipMalloc(&bigger, need) == hipSuccess) {
        if (idx->mx_ws) (void)hipFree(idx->mx_ws);  // (waits for the device)
        idx->mx_ws = bigger;
        idx->mx_ws_bytes = need;
        break;
      }
      (void)hipGetLastError();
      idx->mx_wait = kMatrixPatience;
    }
  } else if (idx->mx_wait > 0) {
    --idx->mx_wait;
  }
  const bool own = idx->mx_ws_bytes > behind;
  s = matrix_fit(idx, Q, topk, own ? idx->mx_ws_bytes : behind);
  s.at = own ? idx->mx_ws : static_cast<uint8_t*>(idx->ws) + lead;
  if (s.q && own && capturing) idx->mx_held = true;
  return s;
}

// Scratch that a call can do without: behind the `lead` bytes of the handle's, else an allocation of its kind's own (`own`; see
// matrix_scratch for when it is asked for); NULL: there is none.  One that a captured graph holds stays as it is, a larger call gets a
// second one: a small captured call must not send all later ones the slower way.
void* extra_scratch(const rii_index* idx, rii_extra& own, size_t need, size_t lead, bool reserved, hipStream_t st) {
  if (need > kMatrixScratch) return nullptr;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone;
  if (capturing) (void)hipGetLastError();
  const size_t behind = idx->ws_bytes > lead ? idx->ws_bytes - lead : 0;
  if (need <= behind) return static_cast<uint8_t*>(idx->ws) + lead;
  if (need > own.bytes) {
    if (reserved || capturing || (own.held && own.n_kept == 64)) return nullptr;
    if (own.wait > 0) {
      --own.wait;
      return nullptr;
    }
    // (a quarter more than needed, as in ensure_ws: calls that vary a little would wait for the device again and again)
    void* bigger = nullptr;
    size_t ask = std::min(need + need / 4, kMatrixScratch);
    if (ask > idx->mx_most || hipMalloc(&bigger, ask) != hipSuccess) {
      (void)hipGetLastError();
      ask = need;
      if (ask > idx->mx_most || hipMalloc(&bigger, ask) != hipSuccess) {
        (void)hipGetLastError();
        own.wait = kMatrixPatience;
        return nullptr;
      }
    }
    if (own.held) {
      own.kept[own.n_kept++] = own.at;
      own.kept_bytes += own.bytes;
      own.held = false;
    } else if (own.at) {
      (void)hipFree(own.at);  // (waits for the device)
    }
    own.at = bigger;
    own.bytes = ask;
  }
  if (capturing) own.held = true;
  return own.at;
}

// Whether rii_adc_scan_linear takes the products for such a batch (a device that has not refused is taken to have room).
bool matrix_taken(const rii_index* idx, int Q, int topk) {
  if (!matrix_applies(idx, Q, topk, idx->N)) return false;
  const size_t look_ups = scan_ws_bytes(kLinear, idx->M, Q, idx->N, topk);
  const bool fixed = (idx->ws_reserved && idx->ws_bytes >= look_ups) || idx->mx_held || idx->mx_wait > 0;
  return !fixed || matrix_fit(idx, Q, topk, std::max(std::max(idx->ws_bytes, look_ups), idx->mx_ws_bytes)).q > 0;
}

void launch_fit(const rii_index* idx, const float* lut, int Q, int Qp, int nf, bool by_query, uint16_t* qfrag, float4* part, uint32_t* left_n,
                hipStream_t st) {
  const int M = idx->M;
  // groups of 16 queries a wave goes through: one round of blocks (three a CU by their registers)
  const int per = std::max(1, (int)(((int64_t)(Qp / 16) * M + 12 * kWantBlocks - 1) / (12 * kWantBlocks)));
  const dim3 grid((unsigned)((Qp / 16 + 4 * per - 1) / (4 * per)), (unsigned)M);
#define RII_FIT(DSP) k_fit_tables<DSP><<<grid, 256, 0, st>>>(lut, idx->mx_fit, idx->mx_ch, by_query ? idx->mx_bh : idx->mx_b, idx->mx_scale, M, idx->Ds, nf, Q, Qp, per, by_query, qfrag, part, left_n)
  switch (idx->mx_dsp) {
    case 4: RII_FIT(4); break;
    case 8: RII_FIT(8); break;
    case 16: RII_FIT(16); break;
    default: RII_FIT(32); break;
  }
#undef RII_FIT
}

template <int NF, bool SEED>
int launch_matrix_round(const MatrixArgs& a, dim3 grid, hipStream_t st) {
  const int rc = set_lds(k_matrix_scan<NF, SEED>, mx_lds<NF>());
  if (rc) return rc;
  k_matrix_scan<NF, SEED><<<grid, 64 * kMxWaves, mx_lds<NF>(), st>>>(a);
  return RII_OK;
}

int launch_matrix_scan(const rii_index* idx, const float* lut, int Q, int cap, int64_t big, int topk, int32_t* ids, float* dist, int out_stride,
                       void* scan_ws, size_t scan_bytes, hipStream_t st) {
  const int M = idx->M;
  const MatrixPlan p = matrix_plan(idx, Q, topk, cap);
  uint8_t* w = static_cast<uint8_t*>(scan_ws) + align_up(scan_bytes, 256);
  float* cq = reinterpret_cast<float*>(w + p.cq);
  float* lo = reinterpret_cast<float*>(w + p.lo);
  float* hi = reinterpret_cast<float*>(w + p.hi);
  int* mode = reinterpret_cast<int*>(w + p.mode);
  MatrixArgs a{};
  a.codes = idx->d_codes; a.plane = idx->plane_codes; a.N = idx->N; a.M = M; a.Ds = idx->Ds; a.D = idx->D;
  a.book = idx->mx_book; a.b = idx->mx_b;
  a.qfrag = reinterpret_cast<const mx_u32x4*>(w + p.qfrag); a.cq = cq; a.Qp = p.Qp;
  a.tiles = (idx->N + kMxRows - 1) / kMxRows;
  // tiles in an order that spreads every round over the whole array (rows may be stored in some order of their own)
  a.step = (int64_t)((double)a.tiles * 0.6180339887) | 1;
  auto gcd = [](int64_t x, int64_t y) { while (y) { const int64_t t = x % y; x = y; y = t; } return x; };
  while (gcd(a.step, a.tiles) != 1) ++a.step;
  a.minima = reinterpret_cast<float*>(w + p.minima);
  a.cnt = reinterpret_cast<uint32_t*>(w + p.cnt);
  a.cand = reinterpret_cast<int32_t*>(w + p.cand);
  a.cap = p.cap;
  uint16_t* qfrag = reinterpret_cast<uint16_t*>(w + p.qfrag);
  float4* part = reinterpret_cast<float4*>(w + p.part);
  LeftOut left{};
  left.n = reinterpret_cast<uint32_t*>(w + p.left); left.q = reinterpret_cast<int32_t*>(w + p.left + 256);
  left.arrays = static_cast<uint32_t*>(scan_ws); left.stride = (int64_t)(align_up((size_t)Q * 4, 256) / 4);
  left.counters = idx->ev_start && idx->ev_stop ? idx->d_scan_counters : nullptr;
  launch_fit(idx, lut, Q, p.Qp, p.nf, false, qfrag, part, left.n, st);
  k_fit_sums<<<(p.Qp + 255) / 256, 256, 0, st>>>(part, M, p.nf, Q, p.Qp, cq, lo, hi, mode, a.cnt, left, nullptr, 0);
  // Tables that no query made are known after the fit: with many of them the products are not worth it, and all queries go by look-ups.
  // (2048 queries over 10^6 rows, M = 16, top-100: products 0.7 of the look-ups' time; 512 over 10^6, M = 64: 0.07)
  const uint32_t most_left = rot_m(M) && topk <= kWaveK4 ? (uint32_t)Q * 3 / 8 : (uint32_t)Q * 3 / 4;
  a.left_n = left.n; a.counters = left.counters;
  auto scan = [&](bool seed, int64_t first, int64_t last) {
    a.first = first;
    a.left_most = seed ? most_left : (uint32_t)Q - 1;
    const int qtiles = p.Qp / 32;
    const int64_t n = last - first;
    int splits = (int)std::max<int64_t>(1, std::min<int64_t>((8 * kWantBlocks + n - 1) / n, qtiles / 32));
    a.per_split = (int)align_up((size_t)(qtiles + splits - 1) / splits, kMxStage);
    const dim3 grid((unsigned)n, (unsigned)((qtiles + a.per_split - 1) / a.per_split));
    switch (p.nf * 2 + (seed ? 1 : 0)) {
      case 4: return launch_matrix_round<2, false>(a, grid, st);
      case 5: return launch_matrix_round<2, true>(a, grid, st);
      case 8: return launch_matrix_round<4, false>(a, grid, st);
      case 9: return launch_matrix_round<4, true>(a, grid, st);
      case 12: return launch_matrix_round<6, false>(a, grid, st);
      case 13: return launch_matrix_round<6, true>(a, grid, st);
      case 16: return launch_matrix_round<8, false>(a, grid, st);
      default: return launch_matrix_round<8, true>(a, grid, st);
    }
  };
  int rc = scan(true, 0, kMxSeedTiles);
  if (rc) return rc;
  const int spare = kMxSeedGroups / (8 * topk);  // groups to a result, in eights
#define RII_SEED(FOLD) k_matrix_seed<FOLD><<<p.Qp / 32, 512, 0, st>>>(a.minima, Q, p.Qp, topk, lo, hi, mode, cq, left, most_left)
  if (spare >= 8) RII_SEED(8);
  else if (spare >= 4) RII_SEED(4);
  else if (spare >= 2) RII_SEED(2);
  else RII_SEED(1);
#undef RII_SEED
  const double ratio = (double)a.tiles / kMxSeedTiles;
  const int rounds = std::max(1, (int)std::ceil(std::log(ratio) / std::log(kMatrixGrowth)));
  int64_t from = 0;
  for (int r = 1; r <= rounds; ++r) {
    const int64_t to = r == rounds ? a.tiles : std::min<int64_t>(a.tiles, (int64_t)(kMxSeedTiles * std::pow(ratio, (double)r / rounds)));
    rc = scan(false, from, to);
    if (rc) return rc;
    from = to;
    // what is listed, scored as defined: the k best so far
    FewArgs f{};
    f.codes = idx->d_codes_rows; f.plane = idx->plane_rows; f.M = M; f.lut = lut; f.N = idx->N;
    f.listed = a.cand; f.listed_cnt = a.cnt; f.listed_cap = p.cap; f.listed_cnt_stride = kMxCntStride;
    f.k = topk; f.ids = ids; f.out_stride = out_stride; f.qmode = mode; f.want_mode = 0;
    f.dist = dist ? dist : reinterpret_cast<float*>(w + p.dist);
    FewShape shape = few_shape(M, Q, p.cap, topk, FewRows::targets, false);
    shape.split = 1;
    rc = launch_few<kFewListed>(f, shape, Q, nullptr, true, st);
    if (rc) return rc;
    k_matrix_next<<<(Q + 3) / 4, 256, 0, st>>>(ids, f.dist, Q, topk, out_stride, p.cap, idx->mx_scale, lo, cq, a.cnt, a.cand, mode, left);
  }
  return launch_left(idx, lut, Q, big, topk, ids, dist, out_stride, left, st);
}

// The index's tables are made by the first call that reads them, on its own stream (35 us; at the index's creation, with
// the wait for them, they were 4 to 7 % of building one of 100,000 codes).  A call that is being captured makes them
// for itself at every replay: nothing has run when the next call is issued.
int matrix_books(const rii_index* idx, hipStream_t st) {
  if (idx->mx_ready) return RII_OK;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(st, &capture) == hipSuccess;
  if (!known) (void)hipGetLastError();
  k_matrix_scale<<<1, 1024, 0, st>>>(idx->d_cb, idx->M, idx->Ds, idx->mx_scale);
  k_matrix_books<<<idx->M, 256, 0, st>>>(idx->d_cb, idx->mx_scale, idx->Ds, idx->mx_dsp, idx->mx_book, idx->mx_fit, idx->mx_ch, idx->mx_b, idx->mx_bh);
  RII_HIP(hipGetLastError());
  idx->mx_ready = known && capture == hipStreamCaptureStatusNone;
  return RII_OK;
}

// The whole batch, as many queries at a time as the scratch is for.
int launch_matrix_batches(const rii_index* idx, const float* lut, int Q, const MatrixScratch& scratch, int topk, int32_t* ids, float* dist,
                          int out_stride, hipStream_t st) {
  const int q = scratch.q;
  const bool timed = idx->ev_start && idx->ev_stop;
  const size_t scan_bytes = matrix_need(idx, q, topk, scratch.cap) - matrix_plan(idx, q, topk, scratch.cap).total;
  int rc = matrix_books(idx, st);
  if (rc) return rc;
  if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_start), st));
  for (int o = 0; o < Q; o += q) {
    rc = launch_matrix_scan(idx, lut + (size_t)o * idx->M * 256, std::min(q, Q - o), scratch.cap, left_big(idx, q, topk), topk, ids + (size_t)o * out_stride,
                                      dist ? dist + (size_t)o * out_stride : nullptr, out_stride, scratch.at, scan_bytes, st);
    if (rc) return rc;
  }
  if (timed) RII_HIP(hipEventRecord(static_cast<hipEvent_t>(idx->ev_stop), st));
  return RII_OK;
}

// ------------------------------------------------------------------ lists by matrix products
// Scratch of a batch (rii_dev_lists.inc), from `at` on: byte offsets.
struct ListPlan {
  int nf, Qp, cap;
  int64_t items;  // most work items
  FewShape few;   // for long lists of candidates
  size_t query, cq, lo, hi, mode, cnt, left, part, counts, starts, groups_n, pairs, by_list, items_at, groups, cand, few_ws, total;
};
bool list_shape(int M, int Ds) {
#define RII_SHAPE(MT, DS) if (M == MT && Ds == DS) return true;
  RII_LIST_SHAPES(RII_SHAPE)
#undef RII_SHAPE
  return false;
}
int64_t list_members(const rii_index* idx, int nprobe, int64_t L) {  // that a query probes, in lists of the mean length
  const int64_t rows = idx->N / idx->K * nprobe;
  return L > 0 && L < rows ? L : rows;
}
ListPlan list_plan(const rii_index* idx, int Q, int nprobe, int64_t L, int topk) {
  const int M = idx->M, K = idx->K;
  ListPlan p;
  p.nf = lp_frags(M, idx->Ds);
  p.Qp = (Q + 31) / 32 * 32;
  const int64_t pairs = (int64_t)Q * nprobe;
  p.items = idx->N / kLpRows + K + pairs / kLpQueries * (idx->max_list_len / kLpRows + 1);
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t o = at; at += align_up(bytes, 256); return o; };
  p.query = take((size_t)p.Qp * p.nf * 32);
  p.cq = take((size_t)p.Qp * 4);
  p.lo = take((size_t)p.Qp * 4);
  p.hi = take((size_t)p.Qp * 4);
  p.mode = take((size_t)p.Qp * 4);
  p.cnt = take((size_t)p.Qp * kMxCntStride * 4);
  p.left = take(256 + (size_t)(1 + kScanArrays) * p.Qp * 4);
  p.part = take((size_t)M * p.Qp * 16);
  p.counts = take((size_t)(K + 2) * 4);
  p.starts = take((size_t)K * 4);
  p.groups_n = take((size_t)Q * 4);
  p.pairs = take((size_t)pairs * sizeof(ListPair));
  p.by_list = take((size_t)pairs * sizeof(ListPair));
  p.items_at = take((size_t)p.items * sizeof(ListItem));
  p.groups = take((size_t)Q * kLpGroups * 4);
  // An eighth of the scratch there may be.  More for members that a bound of the nearest kLpSeen of them will list: four times as many as there
  // would be if the others were no farther away (clusters that share codes list three times that), up to half of the scratch.
  p.cap = (int)std::min<int64_t>(std::max<int64_t>((int64_t)kMatrixScratch / 8 / 4 / Q, kLpLeast), kLpMost);
  const int64_t more = std::min<int64_t>(4 * topk * (list_members(idx, nprobe, L) / kLpSeen), kLpMostSeen);
  const int64_t room = std::min<int64_t>((int64_t)kMatrixScratch / 2, (int64_t)kMatrixScratch * 3 / 4 - (int64_t)at) / 4 / Q;
  p.cap = (int)std::max<int64_t>(p.cap, std::min(more, room));
  // (scored before what is left of the batch needs its candidates there: topk a block)
  p.cand = take(std::max((size_t)Q * p.cap * 4, (size_t)std::max(Q, kWantBlocks) * kWaveK * 8));
  p.few = few_shape(M, Q, p.cap, topk, FewRows::targets, false);
  p.few_ws = take(few_ws_bytes(p.few, Q));
  p.total = at;
  return p;
}
// Which batches: from so many members on, all queries together, as pay for the launches (90 us), for decoding the lists twice and for what
// the filter lists.  The line lies where it no longer loses on rows in clusters that share codes (they list most, and their members
// look alike to the bound), measured over the shapes that there are kernels for, 100,000 to 16 x 10^6 rows, 20 to 4096 lists, 4 to 100 of
// them, top-10 and top-100.  Microseconds query by query / here, the lists in parentheses; "mixture": rows in clusters.
//   at the line, mixture, top-100:  M = 8, N = 10^6 (8 of 1000) 399 / 359, 4 x 10^6 (16 of 2048) 536 / 522;  M = 16, 10^6 (8 of 1000) 310 / 286,
//   4 x 10^6 (16 of 2048) 433 / 421;  M = 32, 10^6 (8 of 1000) 289 / 232;  M = 12, 100,000 (4 of 20) 102 / 100;  M = 64, 10^6 (8 of
//   1000) 449 / 426, with 0.7 times the queries 319 / 366
//   many short lists (the term with K):  M = 16, 10^6 (100 of 4096), 2653 queries top-10 303 / 248, top-100 239 / 274, 4421 368 / 348,
//   4 x 10^6 (64 of 4096) 1818 queries top-100 354 / 383, 2160 437 / 401;  M = 8, 10^6 (100 of 4096) 2959 queries top-100 286 / 310, 4181 406 /
//   370;  M = 12, 10^6 (100 of 4096) 704 queries top-10 146 / 174
//   top-10 and rows that share little are ahead by 1.1 to 4 at the same points, M = 64 in long lists by 2 to 4
//   lists of more than 12,000, mixture, top-100 (the bound is taken of the nearest 18,432 members only, which M = 8 lists most by):  M = 8, 6.5 x 10^6
//   (8 of 72) 291 queries 1359 / 1320, 489 1600 / 1580, (27 of 72) 86 queries 873 / 1330, 145 1568 / 1490, 8 x 10^6 (8 of 100) 395 queries
//   1635 / 1663, (32 of 250) 416 2151 / 1780;  top-10 and M = 16 are ahead from where shorter lists are:  M = 8, (27 of 72) 83 queries 769 / 749,
//   (32 of 250) 239 1030 / 970;  M = 16, 6.5 x 10^6 (8 of 72) 202 queries top-100 937 / 715, (27 of 72) 60 873 / 730, 8 x 10^6 (32 of 250) 174
//   1159 / 980;  M = 12, (8 of 72) 94 986 / 796.  Under 250,000 members a query:  M = 12, 300,000 (4 of 20) 182 queries top-100 121 / 124
//   below the line, left to the look-ups:  M = 16, N = 10^6 (8 of 1000), 1500 queries 107 / 109;  D = 96, 4 x 10^6 (8 of 2048), 4000
//   queries 241 / 264;  M = 64, 500,000, 500 queries 142 / 142, N = 10^6, mixture, 1500 182 / 202.  And, ahead by the products on rows that
//   share little, 1500 queries (8 lists of 1000), M = 64, N = 500,000 339 / 167, M = 12 243 / 146, 4000 queries, N = 10^6, M = 16 210 / 153,
//   M = 32 249 / 176, M = 8 199 / 147: what the rows are like is not known here.
bool list_products_apply(const rii_index* idx, int Q, int nprobe, int64_t L, int topk) {
  const int M = idx->M;
  if (!idx->mx_book || !list_shape(M, idx->Ds) || topk > kWaveK || nprobe > kIvfMaxProbe || idx->K > kLpMaxLists || Q > 65535) return false;
  const int64_t rows = list_members(idx, nprobe, L);
  if (rows < 32 * (int64_t)topk) return false;  // (a bound is taken of groups of four and more members)
  const bool many = topk >= kFewManyResults;
  const bool lengthy = idx->N / idx->K > 12000 && (rows < 250000 || (M == 8 && many));
  const double share = M == 8 ? (lengthy ? 2.6 : 1.5) : M == 16 ? (lengthy ? 1.6 : 1.0) : M == 32 ? 1.0 : M == 64 || lengthy ? 0.6 : 0.5;
  const double lists = M == 64 ? 8000.0 : M == 16 ? (many ? 12000.0 : 4500.0) : M == 8 ? (many ? 8000.0 : 0.0) : M == 12 ? 2500.0 : 0.0;
  const double more = lists * idx->K + (M == 16 ? 1.5 * (double)idx->N : 0.0);
  return (double)Q * (double)rows >= share * (16e6 + 18.0 * (double)idx->N) + more;
}
// Their scratch; NULL: query by query.
void* list_scratch(const rii_index* idx, int Q, int nprobe, int64_t L, int topk, size_t lead, bool reserved, hipStream_t st) {
  if (!list_products_apply(idx, Q, nprobe, L, topk)) return nullptr;
  return extra_scratch(idx, idx->lists_extra, list_plan(idx, Q, nprobe, L, topk).total, lead, reserved, st);
}
template <int M, int DS, bool SEED>
int launch_list_round(const ListProductsArgs& a, hipStream_t st) {
  const int rc = set_lds0(k_list_products<M, DS, SEED>, lp_lds(M, DS));
  if (rc) return rc;
  k_list_products<M, DS, SEED><<<kWantBlocks, 64 * kLpWaves, lp_lds(M, DS), st>>>(a);
  return RII_OK;
}
// All but the queries that are left: their mode is 1 afterwards.
struct ListLeft {
  int* mode;
  LeftOut out;
  uint64_t* cand;  // for k_ivf_w
};
int launch_list_products(const rii_index* idx, const float* lut, int Q, const int32_t* probe, int probe_stride, int nprobe, int64_t L,
                         int topk, int32_t* ids, float* dist, void* scratch, ListLeft* left_out, hipStream_t st) {
  int rc = matrix_books(idx, st);
  if (rc) return rc;
  const int M = idx->M, K = idx->K;
  const ListPlan p = list_plan(idx, Q, nprobe, L, topk);
  uint8_t* w = static_cast<uint8_t*>(scratch);
  auto floats = [&](size_t o) { return reinterpret_cast<float*>(w + o); };
  auto words = [&](size_t o) { return reinterpret_cast<uint32_t*>(w + o); };
  int* mode = reinterpret_cast<int*>(w + p.mode);
  float4* part = reinterpret_cast<float4*>(w + p.part);
  LeftOut left{};
  left.n = words(p.left); left.q = reinterpret_cast<int32_t*>(w + p.left + 256);
  left.arrays = words(p.left + 256) + p.Qp; left.stride = p.Qp;
  left.counters = idx->ev_start && idx->ev_stop ? idx->d_scan_counters : nullptr;
  launch_fit(idx, lut, Q, p.Qp, p.nf, true, reinterpret_cast<uint16_t*>(w + p.query), part, left.n, st);
  uint32_t* counts = words(p.counts);
  k_fit_sums<<<(p.Qp + 255) / 256, 256, 0, st>>>(part, M, p.nf, Q, p.Qp, floats(p.cq), floats(p.lo), floats(p.hi), mode, words(p.cnt), left, counts, K + 2);
  ListPair* pairs = reinterpret_cast<ListPair*>(w + p.pairs);
  ListPair* by_list = reinterpret_cast<ListPair*>(w + p.by_list);
  ListItem* items = reinterpret_cast<ListItem*>(w + p.items_at);
  const int per_block = std::max(16, (Q + kWantBlocks / 2 - 1) / (kWantBlocks / 2));
  rc = set_lds(k_pair_count, (size_t)K * 4);
  if (rc) return rc;
  k_pair_count<<<(Q + per_block - 1) / per_block, 1024, (size_t)K * 4, st>>>(probe, probe_stride, nprobe, idx->d_list_off, K, Q, per_block, L, counts, pairs, words(p.groups_n));
  k_pair_place<<<(K + 63) / 64, 256, 0, st>>>(counts, idx->d_list_off, K, words(p.starts), counts + K, items);
  const int64_t n = (int64_t)Q * nprobe;
  k_pair_fill<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(pairs, n, nprobe, words(p.starts), by_list);
  ListProductsArgs a{};
  a.codes = idx->d_codes_list; a.plane = idx->plane_list; a.book = idx->mx_book;
  a.query = reinterpret_cast<const uint16_t*>(w + p.query); a.cq = floats(p.cq); a.pairs = by_list;
  a.list_ids = idx->d_list_ids; a.items = items; a.n_items = counts + K + 1; a.groups = floats(p.groups); a.cnt = words(p.cnt); a.cand = reinterpret_cast<int32_t*>(w + p.cand); a.cap = p.cap;
  a.left_n = left.n; a.left_most = (uint32_t)Q * 3 / 8;
#define RII_SEED_ROUND(MT, DS) if (M == MT && idx->Ds == DS) rc = launch_list_round<MT, DS, true>(a, st);
#define RII_LIST_ROUND(MT, DS) if (M == MT && idx->Ds == DS) rc = launch_list_round<MT, DS, false>(a, st);
  RII_LIST_SHAPES(RII_SEED_ROUND)
  if (rc) return rc;
  k_list_bound<<<(Q + 3) / 4, 256, 0, st>>>(a.groups, words(p.groups_n), Q, topk, floats(p.lo), floats(p.hi), mode, floats(p.cq), left, a.left_most);
  RII_LIST_SHAPES(RII_LIST_ROUND)
#undef RII_SEED_ROUND
#undef RII_LIST_ROUND
  if (rc) return rc;
  DISPATCH_M(M, k_list_score<MT><<<Q, kLpRanked, 0, st>>>(idx->d_codes_rows, idx->plane_rows, M, lut, a.cnt, a.cand, p.cap, topk, ids, dist, mode, left,
                                                        p.few.split > 1 ? words(p.few_ws) : nullptr, (int)(align_up((size_t)Q * 4, 256) / 4)));
  FewArgs f{};
  f.codes = idx->d_codes_rows; f.plane = idx->plane_rows; f.M = M; f.lut = lut; f.N = idx->N;
  f.listed = a.cand; f.listed_cnt = a.cnt; f.listed_cap = p.cap; f.listed_cnt_stride = kMxCntStride; f.listed_alone = kLpAlone;
  f.k = topk; f.ids = ids; f.dist = dist; f.out_stride = topk; f.qmode = mode; f.want_mode = 2;
  rc = launch_few<kFewListed>(f, p.few, Q, w + p.few_ws, true, st);
  *left_out = ListLeft{mode, left, reinterpret_cast<uint64_t*>(w + p.cand)};
  return rc;
}

// ------------------------------------------------------------------ lists with target set and candidate cap
// Scratch of k_pick_members, then that of the scan that follows.
struct PickPlan {
  int cap;              // most members that are scored
  bool joint;
  FewShape few;
  size_t cnt, few_ws, total;
};
// lin_rows: identifiers that the batch's other queries may have; they are done in the same launch where all of it is a small scan
// (joint), 0: there are none.
PickPlan pick_plan(const rii_index* idx, int Q, int nprobe, int64_t L, int64_t lin_rows, int topk) {
  PickPlan p;
  p.cap = (int)std::min(L, (int64_t)nprobe * idx->max_list_len);
  p.joint = lin_rows > 0 && few_scan(kSubset, idx->M, Q, topk, std::max<int64_t>(lin_rows, p.cap));
  p.few = few_shape(idx->M, Q, std::max<int64_t>(p.joint ? lin_rows : 1, p.cap), topk, FewRows::targets, false);
  p.cnt = align_up((size_t)Q * p.cap * 4, 256);
  p.few_ws = p.cnt + align_up((size_t)Q * 4, 256);
  p.total = p.few_ws + few_ws_bytes(p.few, Q);
  return p;
}
// Lists of so few members and sets so small that k_few's capped form is done in the time that two kernels take (12 us of one query where these
// take 15), up to a round of blocks.  What the sets' size is only the device knows: `largest` may be a guess.  Microseconds of rii_adc_scan_ivf
// in the capped form / members first:  M = 32, 300,000 codes in lists of 1000, one list, L = 20, 20 queries with sets of 24,000 12.4 / 16.0, 300,000 13.1 / 16.0, 200 queries 13.1 / 17.0 and 31 / 17;  M = 16, 10^6 codes, one
// query, L = 5, sets of 10,000 12.6 / 14.8, 160,000 15.0 / 14.7;  M = 64, 20 queries, two lists, L = 50, 40,000 16.9 / 18.5, three
// lists, 20,000 24.2 / 16.9;  M = 8, 100,000 codes, two lists, L = 50, 4000 13.6 / 15.1, five lists, 2000, L = 100 21.4 / 15.5.
bool pick_small(int M, int Q, int64_t members, int64_t L, double largest) {
  return Q <= kWantBlocks && members + 10 * std::min<int64_t>(L, 1 << 20) <= (M == 8 || M == 16 ? 5000 : 3000) &&
         Q * largest <= (M >= 32 ? 6e6 : 2e6) && largest <= (M >= 32 ? 3e5 : 1e5);
}
bool pick_applies(const rii_index* idx, int Q, int nprobe, int64_t L, int topk, double largest) {
  if (pick_small(idx->M, Q, idx->N / idx->K * nprobe, L, largest)) return false;
  return nprobe <= kIvfMaxProbe && Q <= 65535 && few_scan(kSubset, idx->M, Q, topk, std::min(L, idx->N));
}
int launch_pick(const rii_index* idx, const PickPlan& p, int Q, const int32_t* probe, int probe_stride, int nprobe, const int* nprobe_q,
                const int32_t* target_ids, const int64_t* target_offsets, int64_t L, const int* qmode, void* scratch, FewArgs* f,
                hipStream_t st) {
  uint8_t* w = static_cast<uint8_t*>(scratch);
  PickArgs a{};
  a.list_ids = idx->d_list_ids; a.list_off = idx->d_list_off; a.probe = probe; a.probe_stride = probe_stride; a.nprobe = nprobe;
  a.nprobe_q = nprobe_q; a.target_ids = target_ids; a.target_offsets = target_offsets; a.qmode = qmode; a.Lcap = L; a.N = idx->N;
  a.cand = reinterpret_cast<int32_t*>(w); a.cnt = reinterpret_cast<uint32_t*>(w + p.cnt); a.cap = p.cap;
  // as many bits as there are identifiers, 128 KB of them at most, half of it where more than 1000 lists want their place in LDS
  const int64_t bits = std::min<int64_t>((idx->N + 127) / 128 * 128, nprobe <= 1000 ? 1 << 20 : 1 << 19);
  a.words = (int)(bits / 32);
  while (((idx->N - 1) >> a.shift) >= bits) ++a.shift;
  const size_t lds = pick_lds(a.words, nprobe);
  const int rc = set_lds(k_pick_members, lds);
  if (rc) return rc;
  k_pick_members<<<Q, kPickThreads, lds, st>>>(a);
  f->listed = a.cand; f->listed_cnt = a.cnt; f->listed_cap = p.cap; f->listed_cnt_stride = 1;
  return RII_OK;
}

}  // namespace

// ====================================================================== entry points
extern "C" {

int rii_build_lut(const rii_index_t* idx, const float* q, int Q, float* lut, void* stream) {
  if (!idx || !q || !lut || Q < 1) return RII_ERR_INVALID_ARG;
  if (Q > 65535) return RII_ERR_UNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  launch_build_lut(idx, q, Q, lut, st);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_scan_linear_plan(const rii_index_t* idx, int Q, int topk, int* queries_per_block, int64_t* row_chunks) {
  if (!idx || !queries_per_block || !row_chunks || Q < 1 || topk < 1) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  int64_t nchunks, chunk_rows, bchunks, brows;
  scan_chunks(Q, idx->N, &nchunks, &chunk_rows);
  if (matrix_taken(idx, Q, topk)) {
    *queries_per_block = 32;  // (a tile of them at a time, past a block's rows)
    *row_chunks = (idx->N + kMxRows - 1) / kMxRows;
  } else if (few_linear(idx->M, Q, topk, idx->N)) {
    *queries_per_block = 1;
    *row_chunks = few_shape(idx->M, Q, idx->N, topk, FewRows::linear, false).split;
  } else if (topk <= kWaveK && plan_batch(idx->M, Q, idx->N, topk, &bchunks, &brows)) {
    *queries_per_block = 4;
    *row_chunks = bchunks;
  } else if (topk <= kWaveK && rot_m(idx->M) && nchunks == 1 && Q >= 2 && topk > kWaveK4) {
    *queries_per_block = 2;
    *row_chunks = 1;
  } else {
    *queries_per_block = 1;
    *row_chunks = nchunks;
  }
  return RII_OK;
}

int rii_bench_lds_lookups(int width, int blocks, int threads, int iters, int lds_bytes, uint32_t* sink, void* stream) {
  if ((width != 4 && width != 8 && width != 64) || blocks < 1 || iters < 1 || !sink) return RII_ERR_INVALID_ARG;
  if (threads < 64 || threads > kScanThreads || threads % 64 != 0) return RII_ERR_INVALID_ARG;
  if (lds_bytes < 65536 || lds_bytes > 160 * 1024) return RII_ERR_INVALID_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (width == 64) {
    int rc = set_lds0(k_lds_lookups<64>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_lookups<64><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  } else if (width == 8) {
    int rc = set_lds0(k_lds_lookups<8>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_lookups<8><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  } else {
    int rc = set_lds0(k_lds_lookups<4>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_lookups<4><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_bench_scan_linear_half(rii_index_t* idx, const float* lut, int Q, int topk, int32_t* ids, float* dist,
                               void* stream) {
  if (!idx) return RII_ERR_INVALID_ARG;
  if (Q < 1 || topk < 1) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  int64_t chunks = 0, rows = 0;
  // only the four-queries-per-block kernel has the variant (and it runs at any number of rows that kernel can take)
  if (topk > kWaveK || !plan_batch(idx->M, Q, idx->N, topk, &chunks, &rows)) return RII_ERR_UNSUPPORTED;
  idx->bench_half_table = true;
  int rc = rii_adc_scan_linear(idx, lut, Q, topk, ids, dist, stream);
  idx->bench_half_table = false;
  return rc;
}

int rii_bench_lds_reads(int width, int blocks, int threads, int iters, int lds_bytes, uint32_t* sink, void* stream) {
  if ((width != 4 && width != 8 && width != 16) || blocks < 1 || iters < 1 || !sink) return RII_ERR_INVALID_ARG;
  if (threads < 64 || threads > kScanThreads || threads % 64 != 0) return RII_ERR_INVALID_ARG;
  if (lds_bytes < 65536 || lds_bytes > 160 * 1024) return RII_ERR_INVALID_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (width == 4) {
    int rc = set_lds(k_lds_reads<4>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_reads<4><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  } else if (width == 8) {
    int rc = set_lds(k_lds_reads<8>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_reads<8><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  } else {
    int rc = set_lds(k_lds_reads<16>, (size_t)lds_bytes);
    if (rc) return rc;
    k_lds_reads<16><<<blocks, threads, (size_t)lds_bytes, st>>>(iters, sink);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_adc_scan_linear(const rii_index_t* idx, const float* lut, int Q, int topk, int32_t* ids, float* dist,
                        void* stream) {
  if (!idx || !lut || !ids || !dist || Q < 1 || topk < 1) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  if (idx->N < 1) return RII_ERR_INVALID_ARG;
  const size_t need = scan_ws_bytes(kLinear, idx->M, Q, idx->N, topk);
  const bool reserved = idx->ws_reserved && idx->ws_bytes >= need;
  int rc = ensure_ws(idx, need);
  if (rc) return rc;
  const MatrixScratch products = matrix_scratch(idx, Q, topk, 0, reserved, static_cast<hipStream_t>(stream));
  if (products.q) return launch_matrix_batches(idx, lut, Q, products, topk, ids, dist, topk, static_cast<hipStream_t>(stream));
  return launch_scan(idx, idx->d_codes, idx->plane_codes, idx->N, lut, Q, kLinear, nullptr, nullptr, idx->N, topk, ids, dist, topk,
                     nullptr, 0, idx->ws, static_cast<hipStream_t>(stream));
}

int rii_check_target_ids(const rii_index_t* idx, const int32_t* target_ids, const int64_t* target_offsets, int Q,
                         void* stream) {
  if (!idx || !target_offsets || Q < 1) return RII_ERR_INVALID_ARG;
  if (Q > 65535) return RII_ERR_UNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  int rc = ensure_ws(idx, 256);
  if (rc) return rc;
  uint32_t* flag = static_cast<uint32_t*>(idx->ws);
  RII_HIP(hipMemsetAsync(flag, 0, 4, st));
  k_check_targets<<<Q, 256, 0, st>>>(target_ids, target_offsets, idx->N, flag);
  RII_HIP(hipGetLastError());
  uint32_t h = 0;
  RII_HIP(hipMemcpyAsync(&h, flag, 4, hipMemcpyDeviceToHost, st));
  RII_HIP(hipStreamSynchronize(st));
  if (h & 2u) return RII_ERR_INVALID_ARG;
  return h ? RII_ERR_UNSORTED_IDS : RII_OK;
}

int rii_adc_scan_subset(const rii_index_t* idx, const float* lut, int Q, const int32_t* target_ids,
                        const int64_t* target_offsets, int64_t max_targets, int topk, int32_t* ids, float* dist,
                        void* stream) {
  if (!idx || !lut || !ids || !dist || !target_offsets || Q < 1 || topk < 1 || max_targets < 0)
    return RII_ERR_INVALID_ARG;
  if (!target_ids && max_targets > 0) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  if (max_targets > idx->N) max_targets = idx->N;
  int64_t rows = std::max<int64_t>(max_targets, 1);
  int rc = ensure_ws(idx, scan_ws_bytes(kSubset, idx->M, Q, rows, topk));
  if (rc) return rc;
  return launch_scan(idx, idx->d_codes_rows, idx->plane_rows, idx->N, lut, Q, kSubset, target_ids, target_offsets, rows, topk, ids, dist,
                     topk, nullptr, 0, idx->ws, static_cast<hipStream_t>(stream));
}

int rii_topk(const float* cand_dist, const int32_t* cand_ids, const int64_t* cand_offsets, int Q,
             int64_t max_segment, int topk, int32_t* ids, float* dist, void* stream) {
  if (!cand_dist || !cand_offsets || !ids || Q < 1 || topk < 1 || max_segment < 0) return RII_ERR_INVALID_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  SelectArgs s{};
  s.cand_dist = cand_dist; s.cand_ids = cand_ids; s.cand_offsets = cand_offsets;
  s.k = topk; s.out_stride = topk; s.ids = ids; s.dist = dist;
  if (topk <= RII_MAX_TOPK) {
    k_select<><<<Q, kScanThreads, 0, st>>>(s);
  } else {
    if (topk > RII_MAX_SORT || max_segment < 1 || max_segment > RII_MAX_SORT) return RII_ERR_UNSUPPORTED;
    size_t lds = (size_t)RII_MAX_SORT * 8;
    int rc = set_lds(k_sort_segments, lds);
    if (rc) return rc;
    k_sort_segments<<<Q, kScanThreads, lds, st>>>(s);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// Coarse ranking into caller buffers; `ws` must hold what coarse_ws_bytes() says.  Which way:
//   n <= RII_MAX_TOPK, K <= kRankMaxRows: k_rank_lists, the distances computed in the kernel --
//     except for few queries over many centres, where a chip-wide k_adc_all computes them first
//     (K = 16384, M = 32: 19 us against 32 for one query, 26 against 32 for 32 queries; at K = 4096
//     the second launch costs what it saves: 14 against 12);
//   n <= RII_MAX_TOPK, more centres than a block's LDS holds: the scan kernels over the stored form;
//   n above that: all distances sorted (k_sort_segments, K <= RII_MAX_SORT).
static bool coarse_in_lds(int K, int nprobe) { return nprobe <= RII_MAX_TOPK && K <= kRankMaxRows; }
static bool coarse_split(int Q, int K) { return Q <= kCoarseSplitQ && K >= kCoarseSplitK; }

static size_t coarse_ws_bytes(const rii_index* idx, int Q, int nprobe, bool tight = false) {
  if (coarse_in_lds(idx->K, nprobe)) return coarse_split(Q, idx->K) ? align_up((size_t)Q * idx->K * 4, 256) : 256;
  if (nprobe <= RII_MAX_TOPK) return scan_ws_bytes(kLinear, idx->M, Q, idx->K, nprobe, true, tight);
  return align_up((size_t)Q * idx->K * 4, 256) + align_up((size_t)(Q + 1) * 8, 256);
}

static int coarse_rank(const rii_index* idx, const float* lut, int Q, int nprobe, int32_t* list_ids, float* list_d0,
                       int out_stride, const int* qmode, int want_mode, void* ws, hipStream_t st, bool tight = false,
                       const RankTables& tables = RankTables{}) {
  const int M = idx->M, K = idx->K;
  const bool in_lds = coarse_in_lds(K, nprobe);
  if (nprobe <= RII_MAX_TOPK && !in_lds) {
    return launch_scan(idx, idx->d_coarse_st, idx->plane_coarse, K, lut, Q, kLinear, nullptr, nullptr, K, nprobe, list_ids, list_d0,
                       out_stride, qmode, want_mode, ws, st, false, tight);
  }
  float* d0 = static_cast<float*>(ws);
  const bool split = !in_lds || coarse_split(Q, K);
  if (split) {
    const size_t lds = (size_t)M * 1024;
    const dim3 grid((K + 255) / 256, Q);
    DISPATCH_M(M, { int rc = set_lds(k_adc_all<MT>, lds); if (rc) return rc;
                    k_adc_all<MT><<<grid, 256, lds, st>>>(idx->d_coarse, K, M, lut, d0, qmode, want_mode); });
  }
  if (in_lds) {
    const size_t lds = rank_lds(M, K, nprobe, !split);
    // one block per query: small blocks, several to a CU, when the queries fill the chip, of as many threads
    // as fill it however few the LDS leaves room for (M = 64: 777 queries, K = 1000, 36 us with 256)
    const int per_cu = (int)(160 * 1024 / lds);
    const int threads = Q < kWantBlocks || per_cu <= 2 ? 1024 : per_cu <= 4 || K > 2048 ? 512 : 256;
    if (split) {
      int rc = set_lds(k_rank_lists<0, true>, lds);
      if (rc) return rc;
      k_rank_lists<0, true><<<Q, threads, lds, st>>>(nullptr, K, M, nullptr, d0, nprobe, out_stride, list_ids, list_d0, qmode, want_mode, tables);
    } else {
      // (two kernels: the choice in one cost calls that have their tables)
#define RII_RANK(TABLES) DISPATCH_M(M, { int rc = set_lds(k_rank_lists<MT, false, TABLES>, lds); if (rc) return rc; \
                                         k_rank_lists<MT, false, TABLES><<<Q, threads, lds, st>>>(idx->d_coarse, K, M, lut, nullptr, nprobe, out_stride, \
                                                                                                  list_ids, list_d0, qmode, want_mode, tables); })
      if (tables.q) { RII_RANK(true); }
      else { RII_RANK(false); }
#undef RII_RANK
    }
    RII_HIP(hipGetLastError());
    return RII_OK;
  }
  int64_t* off = reinterpret_cast<int64_t*>(static_cast<uint8_t*>(ws) + align_up((size_t)Q * K * 4, 256));
  k_iota_offsets<<<(Q + 256) / 256, 256, 0, st>>>(off, Q, K);
  SelectArgs s{};
  s.cand_dist = d0; s.cand_offsets = off; s.k = nprobe; s.out_stride = out_stride;
  s.ids = list_ids; s.dist = list_d0; s.qmode = qmode; s.want_mode = want_mode;
  size_t lds2 = (size_t)RII_MAX_SORT * 8;
  int rc = set_lds(k_sort_segments, lds2);
  if (rc) return rc;
  k_sort_segments<<<Q, kScanThreads, lds2, st>>>(s);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_coarse_assign(const rii_index_t* idx, const float* lut, int Q, int nprobe, int32_t* list_ids, float* list_d0,
                      void* stream) {
  if (!idx || !lut || !list_ids || Q < 1) return RII_ERR_INVALID_ARG;
  if (idx->K < 1) return RII_ERR_NOT_BUILT;
  if (nprobe < 1 || nprobe > idx->K) return RII_ERR_INVALID_ARG;
  if (!m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  if (nprobe > RII_MAX_TOPK && idx->K > RII_MAX_SORT) return RII_ERR_UNSUPPORTED;
  int rc = ensure_ws(idx, coarse_ws_bytes(idx, Q, nprobe));
  if (rc) return rc;
  return coarse_rank(idx, lut, Q, nprobe, list_ids, list_d0, nprobe, nullptr, 0, idx->ws,
                     static_cast<hipStream_t>(stream));
}

// How many members the `nprobe` lists of a query may well have, the candidate cap taken into account.  Queries come
// from where the data are, so a list is probed about in proportion to its length, and the lists count with the
// length that a member's list has; one of them may be the longest, and a batch waits for its longest query.  (Lists
// by Zipf's law, M = 16, 256 queries, two lists of 2 x 10^6 members in 1000, top-1: 283 us in the streaming kernel, 969
// in k_few, where the mean length alone sent them.)
static int64_t list_rows(const rii_index* idx, int nprobe, int64_t L) {
  const int64_t mean = idx->N / idx->K * nprobe + (idx->N % idx->K) * nprobe / idx->K;
  const int64_t rows = std::min(idx->N, std::max(mean, idx->member_list_len * nprobe) + idx->max_list_len);
  return L > 0 && L < rows ? L : rows;
}

// Blocks per query of the multi-block inverted-index scan.
static int ivf_split(int Q, int nprobe) {
  int split = (kWantBlocks + Q - 1) / Q;
  if (split > nprobe) split = nprobe;
  return split < 1 ? 1 : split;
}

static size_t ivf_ws_bytes(const rii_index* idx, int Q, int nprobe, int64_t L, int topk, bool targets, bool tight = false) {
  const FewShape f = few_shape(idx->M, Q, list_rows(idx, nprobe, L), topk, targets && L > 0 ? FewRows::capped : FewRows::lists, tight);
  const size_t few = few_ws_bytes(f, Q);
  if (topk > kWaveK) return few;
  return std::max(few, kScanArrays * align_up((size_t)Q * 4, 256) + (size_t)Q * ivf_split(Q, nprobe) * topk * 8 + 256);
}

constexpr int64_t kLeftFewRows = 32768;
constexpr uint32_t kLeftFewQueries = 64;
static int launch_ivf(const rii_index* idx, const float* lut, int Q, const int32_t* probe, int probe_stride,
                      int nprobe, const int* nprobe_q, const int32_t* target_ids, const int64_t* target_offsets,
                      int64_t L, int topk, int32_t* ids, float* dist, const int* qmode, int want_mode, void* ws,
                      hipStream_t st, bool cleared = false, bool tight = false, void* products = nullptr) {
  const int M = idx->M;
  const bool capped = L > 0 && target_ids;
  const int64_t rows = list_rows(idx, nprobe, capped ? 0 : L);
  const bool few = nprobe <= kIvfMaxProbe && Q <= 65535 && (capped || topk > kWaveK || few_lists(M, Q, topk, rows));
  if (products) {  // (no target sets, one branch and one number of lists for all queries); below: what it leaves
    ListLeft left;
    int rc = launch_list_products(idx, lut, Q, probe, probe_stride, nprobe, L, topk, ids, dist, products, &left, st);
    if (rc) return rc;
    // Many members: queries that are left share the chip, where k_few would take them up to kLeftFewQueries of them (so many that each
    // has four blocks; all others by k_few).  Few members: a block of k_few has done them as soon.
    if (!few || rows > kLeftFewRows) {
      IvfArgs a{};
      a.codes_list = idx->d_codes_list; a.plane = idx->plane_list; a.list_ids = idx->d_list_ids; a.list_off = idx->d_list_off; a.M = M;
      a.lut = lut; a.probe = probe; a.probe_stride = probe_stride; a.nprobe = nprobe; a.Lcap = L; a.k = topk; a.ids = ids; a.dist = dist;
      a.tau_g = left.out.arrays; a.cand_cnt = left.out.arrays + left.out.stride; a.done_cnt = left.out.arrays + 3 * left.out.stride; a.cand = left.cand;
      a.left_n = left.out.n; a.left_q = left.out.q; a.left_most = few ? kLeftFewQueries : 0xFFFFFFFFu; a.left_mode = left.mode;
      const size_t lds = ivf_w_lds(M, nprobe);
      const unsigned blocks = (unsigned)(few ? kWantBlocks : std::max(Q, kWantBlocks));
      DISPATCH_M(M, { rc = set_lds0(k_ivf_w<MT, true>, lds); if (rc) return rc;
                      k_ivf_w<MT, true><<<blocks, kScanThreads, lds, st>>>(a); });
      RII_HIP(hipGetLastError());
      if (!few) return RII_OK;
    }
    qmode = left.mode;
    want_mode = 1;
  }
  if (few) {
    FewArgs f{};
    f.codes = idx->d_codes_list; f.plane = idx->plane_list; f.M = M; f.lut = lut; f.N = idx->N;
    f.target_ids = target_ids; f.target_offsets = target_offsets; f.list_ids = idx->d_list_ids; f.list_off = idx->d_list_off;
    f.probe = probe; f.probe_stride = probe_stride; f.nprobe = nprobe; f.nprobe_q = nprobe_q; f.Lcap = L;
    f.k = topk; f.ids = ids; f.dist = dist; f.out_stride = topk; f.qmode = qmode; f.want_mode = want_mode;
    const FewShape shape = few_shape(M, Q, rows, topk, capped ? FewRows::capped : FewRows::lists, tight);
    return capped ? launch_few<kFewCapped>(f, shape, Q, ws, cleared, st) : launch_few<kFewLists>(f, shape, Q, ws, cleared, st);
  }
  IvfArgs a{};
  a.codes_list = idx->d_codes_list; a.plane = idx->plane_list; a.list_ids = idx->d_list_ids; a.list_off = idx->d_list_off; a.M = M;
  a.lut = lut; a.probe = probe; a.probe_stride = probe_stride; a.nprobe = nprobe; a.nprobe_q = nprobe_q;
  a.target_ids = target_ids; a.target_offsets = target_offsets; a.Lcap = L; a.k = topk;
  a.ids = ids; a.dist = dist; a.qmode = qmode; a.want_mode = want_mode;
  if ((L == 0 || !target_ids) && topk <= kWaveK && nprobe <= kIvfMaxProbe && Q <= 65535) {
    // no candidate cap, or a cap without a target set: who scores which member does not matter,
    // so the members of the probed lists are dealt to the waves of one or more blocks per query
    const int split = ivf_split(Q, nprobe);
    const size_t cstride = align_up((size_t)Q * 4, 256) / 4;
    uint32_t* tau = static_cast<uint32_t*>(ws);
    a.tau_g = tau; a.cand_cnt = tau + cstride; a.done_cnt = tau + 3 * cstride;
    a.cand = reinterpret_cast<uint64_t*>(static_cast<uint8_t*>(ws) + kScanArrays * cstride * 4);
    a.cand_cap = (int64_t)split * topk;
    k_init_scan<<<(Q + 255) / 256, 256, 0, st>>>(tau, Q, (int)cstride, nullptr, 0);
    const size_t ldsw = ivf_w_lds(M, nprobe);
    dim3 grid((unsigned)split, (unsigned)Q);
    DISPATCH_M(M, { int rc = set_lds0(k_ivf_w<MT>, ldsw); if (rc) return rc;
                    k_ivf_w<MT><<<grid, kScanThreads, ldsw, st>>>(a); });
    RII_HIP(hipGetLastError());
    return RII_OK;
  }
  const size_t lds = ivf_lds_main(M) + kBlockVarsBytes;
  DISPATCH_M(M, { int rc = set_lds(k_ivf<MT>, lds); if (rc) return rc;
                  k_ivf<MT><<<Q, kScanThreads, lds, st>>>(a); });
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_adc_scan_ivf(const rii_index_t* idx, const float* lut, int Q, const int32_t* probe_lists, int nprobe,
                     const int32_t* target_ids, const int64_t* target_offsets, int64_t L, int topk, int32_t* ids,
                     float* dist, void* stream) {
  if (!idx || !lut || !probe_lists || !ids || !dist || Q < 1 || topk < 1 || L < 0) return RII_ERR_INVALID_ARG;
  if (idx->K < 1) return RII_ERR_NOT_BUILT;
  if (nprobe < 1 || nprobe > idx->K) return RII_ERR_INVALID_ARG;
  if ((target_ids == nullptr) != (target_offsets == nullptr)) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M)) return RII_ERR_UNSUPPORTED;
  if (L >= idx->N) L = 0;  // such a cap never cuts anything
  const size_t need = ivf_ws_bytes(idx, Q, nprobe, L, topk, target_ids != nullptr);
  const bool reserved = idx->ws_reserved && idx->ws_bytes >= need;
  int rc = ensure_ws(idx, need);
  if (rc) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // (the largest set for which Alg. 3 asks for so many lists; for a single one half-way, by their logarithms, from the smallest to everything)
  const double all = (double)idx->N, one = std::min(all, (double)idx->K * (double)L);
  const double largest = nprobe > 1 ? std::min(all, one / (nprobe - 1)) : std::sqrt(one * all);
  if (target_ids && L > 0 && pick_applies(idx, Q, nprobe, L, topk, largest)) {
    const PickPlan p = pick_plan(idx, Q, nprobe, L, 0, topk);
    if (void* pick = extra_scratch(idx, idx->pick_extra, p.total, align_up(need, 256), reserved, st)) {
      FewArgs f{};
      rc = launch_pick(idx, p, Q, probe_lists, nprobe, nprobe, nullptr, target_ids, target_offsets, L, nullptr, pick, &f, st);
      if (rc) return rc;
      f.codes = idx->d_codes_rows; f.plane = idx->plane_rows; f.M = idx->M; f.lut = lut; f.N = idx->N;
      f.k = topk; f.ids = ids; f.dist = dist; f.out_stride = topk;
      return launch_few<kFewListed>(f, p.few, Q, static_cast<uint8_t*>(pick) + p.few_ws, false, st);
    }
  }
  void* products = target_ids ? nullptr : list_scratch(idx, Q, nprobe, L, topk, align_up(need, 256), reserved, st);
  return launch_ivf(idx, lut, Q, probe_lists, nprobe, nprobe, nullptr, target_ids, target_offsets, L, topk, ids,
                    dist, nullptr, 0, idx->ws, st, false, false, products);
}

// Scratch layout of the query procedure: tables, per-query plan, probed lists, then the stage
// scratch that the scan, the coarse ranking and the inverted-index scan use one after the other.
struct QueryPlan {
  int64_t theta = 0;     // target sets from this size on go through the lists
  int pmax = 1;          // most lists any inverted-index query of the batch can ask for
  int64_t lin_rows = 1;  // most rows any linear-scan query of the batch can have
  size_t lut_b = 0, plan_b = 0, probe_b = 0, total = 0;
  // Without target sets every query has the same |S| = N: the host takes Alg. 3's decision and k_plan and
  // the per-query modes fall away, which also lets a batch into the batched scan.
  bool uniform = false;
  bool tight = false;  // small scans get the least scratch (see few_shape)
  bool no_lists = false;  // all target sets are below theta
  MatrixScratch products;  // of the linear scan by matrix products, where it goes that way
  void* lists = nullptr;   // the same of the inverted index
  void* pick = nullptr;    // of lists with target sets, whose members are found first
};

// `limit` > 0: a plan beyond that many bytes gives up the small scans' room, then the batched scan.  whole: see theta.
static int plan_query(const rii_index* idx, int Q, int topk, bool targets, int64_t max_targets, int64_t L,
                      QueryPlan* p, size_t limit = 0, bool whole = true) {
  const int M = idx->M, K = idx->K;
  const bool has_lists = K > 0;
  // Largest number of lists any inverted-index query of this batch can ask for: such a query
  // has |S| >= max(theta, 1), and |S| = N when there is no target set.
  // A target set of at most L members asks for all K lists and its cap is never met: the members scored are the set, which the
  // linear scan does without walking every list (6317 sets of 410 to 10,827 identifiers, 43 lists of 147,000, M = 64: 307 ms, 0.8).
  p->theta = targets && has_lists && whole ? std::max<int64_t>(idx->theta, L + 1) : idx->theta;
  p->pmax = 1;
  if (has_lists) {
    auto lists = [&](int64_t theta) {
      const int64_t smin = targets ? std::max<int64_t>(theta, 1) : idx->N;
      return (int)std::min<int64_t>(((int64_t)K * L + smin - 1) / smin, K);
    };
    if (lists(idx->theta) > RII_MAX_TOPK && K > RII_MAX_SORT) return RII_ERR_UNSUPPORTED;
    p->pmax = lists(p->theta);
  }
  p->no_lists = targets && has_lists && max_targets < p->theta;
  // linear-scan queries have |S| < theta (and at most max_targets, N)
  int64_t lin_rows = targets ? std::min<int64_t>(max_targets, idx->N) : idx->N;
  if (has_lists && p->theta > 0) lin_rows = std::min<int64_t>(lin_rows, p->theta - 1);
  if (has_lists && p->theta <= 0) lin_rows = 0;
  if (!targets && has_lists && idx->N >= p->theta) lin_rows = 0;
  p->lin_rows = std::max<int64_t>(lin_rows, 1);
  p->lut_b = align_up((size_t)Q * M * 256 * 4, 256);
  p->plan_b = align_up((size_t)Q * 4, 256);
  p->probe_b = align_up((size_t)Q * p->pmax * 4, 256);
  const int scan_mode = targets ? kSubset : kLinear;
  auto size = [&](bool uniform, bool tight) {
    p->uniform = uniform;
    p->tight = tight;
    const size_t scan_b = align_up(scan_ws_bytes(scan_mode, M, Q, p->lin_rows, topk, uniform, tight), 256);
    const size_t coarse_b = has_lists ? align_up(coarse_ws_bytes(idx, Q, p->pmax, tight), 256) : 0;
    const size_t ivf_b = has_lists ? align_up(ivf_ws_bytes(idx, Q, p->pmax, L, topk, targets, tight), 256) : 0;
    p->total = p->lut_b + 2 * p->plan_b + p->probe_b + std::max(scan_b, std::max(coarse_b, ivf_b));
  };
  size(!targets, false);
  if (limit && p->total > limit) size(!targets, true);
  if (limit && p->total > limit) size(false, true);
  // (sets up to the cap are larger ones for the linear scan, which may want more scratch than the lists)
  if (limit && p->total > limit && p->theta != idx->theta) return plan_query(idx, Q, topk, targets, max_targets, L, p, limit, false);
  return RII_OK;
}

static int check_query_args(const rii_index_t* idx, const float* q, int Q, int topk, const int32_t* target_ids,
                            const int64_t* target_offsets, int64_t max_targets, int64_t L, const int32_t* ids,
                            const float* dist) {
  if (!idx || !q || !ids || !dist || Q < 1 || topk < 1 || L < 1 || max_targets < 0) return RII_ERR_INVALID_ARG;
  if ((target_ids == nullptr) != (target_offsets == nullptr)) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || !m_supported(idx->M) || Q > 65535) return RII_ERR_UNSUPPORTED;
  if (idx->N < 1) return RII_ERR_INVALID_ARG;
  return RII_OK;
}

// Alg. 3 with its scratch at `ws` (p.total bytes).
static int run_query(const rii_index* idx, const QueryPlan& p, const float* q, int Q, int topk,
                     const int32_t* target_ids, const int64_t* target_offsets, int64_t L, int32_t* ids, float* dist,
                     void* ws, hipStream_t st) {
  const int K = idx->K;
  const bool has_lists = K > 0;
  uint8_t* w = static_cast<uint8_t*>(ws);
  float* lut = reinterpret_cast<float*>(w); w += p.lut_b;
  int* qmode = reinterpret_cast<int*>(w); w += p.plan_b;
  int* nprobe_q = reinterpret_cast<int*>(w); w += p.plan_b;
  int32_t* probe = reinterpret_cast<int32_t*>(w); w += p.probe_b;
  void* stage_ws = w;

  // One branch for all queries, and that the lists: the ranking makes the tables where it reads them in LDS (with few queries a block's 16,384
  // entries of M = 64 take a microsecond longer than the launch that they save).
  const bool untouched = has_lists && coarse_in_lds(K, p.pmax) && !coarse_split(Q, K);  // (the ranking leaves the stage scratch alone then)
  const bool by_rank = p.uniform && untouched && idx->N >= idx->theta && idx->Ds <= kRankTableDs && (idx->M <= 32 || Q > 32);
  if (!by_rank) launch_build_lut(idx, q, Q, lut, st, p.uniform ? stage_ws : nullptr);
  // No set is as large as those that go through the lists: the ranking and the lists' scan would find no query of theirs (138 sets
  // of up to 1844 identifiers, 28 lists of 184, M = 32: they took 10 of 41 us).
  if (has_lists && p.no_lists)
    return launch_scan(idx, idx->d_codes_rows, idx->plane_rows, idx->N, lut, Q, kSubset, target_ids, target_offsets, p.lin_rows, topk, ids, dist,
                       topk, nullptr, 0, stage_ws, st, false, p.tight);
  PickPlan pick{};
  uint8_t* pick_ws = static_cast<uint8_t*>(p.pick);
  if (p.pick) pick = pick_plan(idx, Q, p.pmax, L, p.lin_rows, topk);
  if (p.uniform) qmode = nprobe_q = nullptr;  // (one branch for all queries; every query's lists are p.pmax then)
  else k_plan<<<(Q + 255) / 256, 256, 0, st>>>(target_offsets, idx->N, Q, p.theta, K, L, p.pmax, qmode, nprobe_q,
                                               p.pick ? reinterpret_cast<uint32_t*>(pick_ws + pick.few_ws) : nullptr,
                                               (int)(align_up((size_t)Q * 4, 256) / 4));
  int rc = RII_OK;
  if (p.pick) {
    if (!pick.joint) {
      rc = launch_scan(idx, idx->d_codes_rows, idx->plane_rows, idx->N, lut, Q, kSubset, target_ids, target_offsets, p.lin_rows, topk,
                       ids, dist, topk, qmode, 0, stage_ws, st, false, p.tight);
      if (rc) return rc;
    }
    rc = coarse_rank(idx, lut, Q, p.pmax, probe, nullptr, p.pmax, qmode, 1, stage_ws, st, p.tight);
    if (rc) return rc;
    FewArgs f{};
    rc = launch_pick(idx, pick, Q, probe, p.pmax, p.pmax, nprobe_q, target_ids, target_offsets, L, qmode, p.pick, &f, st);
    if (rc) return rc;
    f.codes = idx->d_codes_rows; f.plane = idx->plane_rows; f.M = idx->M; f.lut = lut; f.N = idx->N;
    f.k = topk; f.ids = ids; f.dist = dist; f.out_stride = topk; f.qmode = qmode;
    if (pick.joint) {  // both branches in one scan by identifiers: the target sets (mode 0), their first L members in the lists (mode 1)
      f.target_ids = target_ids; f.target_offsets = target_offsets;
      return launch_few<kFewJoint>(f, pick.few, Q, pick_ws + pick.few_ws, true, st);
    }
    f.want_mode = 1;
    return launch_few<kFewListed>(f, pick.few, Q, pick_ws + pick.few_ws, true, st);
  }
  // linear-scan branch (mode 0)
  const bool all_linear = !target_ids && (!has_lists || idx->N < idx->theta);
  if (target_ids) {
    rc = launch_scan(idx, idx->d_codes_rows, idx->plane_rows, idx->N, lut, Q, kSubset, target_ids, target_offsets, p.lin_rows, topk,
                     ids, dist, topk, qmode, 0, stage_ws, st, false, p.tight);
  } else if (all_linear && p.products.q) {
    rc = launch_matrix_batches(idx, lut, Q, p.products, topk, ids, dist, topk, st);
  } else if (all_linear) {
    rc = launch_scan(idx, idx->d_codes, idx->plane_codes, idx->N, lut, Q, kLinear, nullptr, nullptr, idx->N, topk, ids, dist, topk,
                     qmode, 0, stage_ws, st, p.uniform, p.tight);
  }
  if (rc) return rc;
  // inverted-index branch (mode 1); the scratch of the scan stage is reused in stream order
  if (has_lists && !all_linear) {
    RankTables tables{};
    if (by_rank) tables = RankTables{q, idx->d_cb, idx->D, idx->Ds, lut, static_cast<uint32_t*>(stage_ws), (int)(align_up((size_t)Q * 4, 256) / 4)};
    rc = coarse_rank(idx, lut, Q, p.pmax, probe, nullptr, p.pmax, qmode, 1, stage_ws, st, p.tight, tables);
    if (rc) return rc;
    rc = launch_ivf(idx, lut, Q, probe, p.pmax, p.pmax, nprobe_q, target_ids, target_offsets, L, topk, ids, dist, qmode,
                    1, stage_ws, st, p.uniform && untouched, p.tight, p.lists);
    if (rc) return rc;
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_query(const rii_index_t* idx, const float* q, int Q, int topk, const int32_t* target_ids,
              const int64_t* target_offsets, int64_t max_targets, int64_t L, int32_t* ids, float* dist,
              void* stream) {
  int rc = check_query_args(idx, q, Q, topk, target_ids, target_offsets, max_targets, L, ids, dist);
  if (rc) return rc;
  // L >= N asks for all K lists and never cuts the candidates: N says the same, and K * L then
  // stays far from overflow here and in k_plan
  if (L > idx->N) L = idx->N;
  QueryPlan p;
  rc = plan_query(idx, Q, topk, target_ids != nullptr, max_targets, L, &p);
  if (rc) return rc;
  const bool reserved = idx->ws_reserved && idx->ws_bytes >= p.total;
  rc = ensure_ws(idx, p.total);
  if (rc) return rc;
  if (!target_ids && (idx->K == 0 || idx->N < idx->theta))
    p.products = matrix_scratch(idx, Q, topk, p.lut_b + 2 * p.plan_b + p.probe_b, reserved, static_cast<hipStream_t>(stream));
  else if (!target_ids)
    p.lists = list_scratch(idx, Q, p.pmax, L, topk, p.total, reserved, static_cast<hipStream_t>(stream));
  else if (idx->K > 0 && !p.no_lists) {
    const PickPlan pick = pick_plan(idx, Q, p.pmax, L, p.lin_rows, topk);
    // (joint: the members are found in a kernel more and the sets of both branches scanned in one less, which few members earn as well: M = 8,
    // four sets of 85 to 1839, 95 lists of 160, L = 160 34.7 us in the capped form, 26.5 here)
    if (pick_applies(idx, Q, p.pmax, L, topk, pick.joint ? HUGE_VAL : (double)std::min(max_targets, idx->N)))
      p.pick = extra_scratch(idx, idx->pick_extra, pick.total, p.total, reserved, static_cast<hipStream_t>(stream));
  }
  return run_query(idx, p, q, Q, topk, target_ids, target_offsets, L, ids, dist, idx->ws, static_cast<hipStream_t>(stream));
}

int rii_index_reserve_workspace(rii_index_t* idx, int Q, int topk, int64_t max_targets, int nprobe) {
  if (!idx || Q < 1 || topk < 1 || max_targets < 0 || nprobe < 0) return RII_ERR_INVALID_ARG;
  if (topk > RII_MAX_TOPK || Q > 65535) return RII_ERR_UNSUPPORTED;
  const int M = idx->M, K = idx->K;
  nprobe = std::min(nprobe, std::max(K, 1));
  // every stage's need, as bounds that grow with Q and topk (so smaller batches fit as well)
  size_t stage = scan_ws_bound(M, Q, idx->N, topk);
  if (K > 0 && nprobe > 0) {
    const size_t coarse = coarse_in_lds(K, nprobe)   ? align_up((size_t)std::min(Q, kCoarseSplitQ) * K * 4, 256) + 256
                          : nprobe <= RII_MAX_TOPK ? scan_ws_bound(M, Q, K, nprobe)
                                                   : align_up((size_t)Q * K * 4, 256) + align_up((size_t)(Q + 1) * 8, 256);
    const size_t ivf = kScanArrays * align_up((size_t)Q * 4, 256) + ((size_t)Q + kWantBlocks) * topk * 8 + 256;
    stage = std::max(stage, std::max(coarse, ivf));
  }
  const size_t query = align_up((size_t)Q * M * 256 * 4, 256) + 2 * align_up((size_t)Q * 4, 256) +
                       align_up((size_t)Q * std::max(nprobe, 1) * 4, 256) + align_up(stage, 256);
  idx->ws_reserved = true;
  return ensure_ws(idx, query);
}

// ---- the query procedure without any allocation ---------------------------------------------
// Scratch of rii_query_noalloc: one array per GPU, in the library's own device image.  In host
// code the array's name only stands for it; its device address is asked for once per device
// (with that device current) and kept.
static __device__ __align__(256) unsigned char scratch[RII_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

static int scratch_of_current_device(void** out) {
  int dev = -1;
  RII_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return RII_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    RII_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return RII_ERR_DEVICE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return RII_OK;
}

int rii_query_noalloc(const rii_index_t* idx, const float* q, int Q, int topk, const int32_t* target_ids,
                      const int64_t* target_offsets, int64_t max_targets, int64_t L, int32_t* ids, float* dist,
                      void* stream) {
  int rc = check_query_args(idx, q, Q, topk, target_ids, target_offsets, max_targets, L, ids, dist);
  if (rc) return rc;
  if (L > idx->N) L = idx->N;
  int dev = -1;
  RII_HIP(hipGetDevice(&dev));
  if (dev != idx->device) return RII_ERR_INVALID_ARG;  // the handle's arrays live on another GPU
  QueryPlan p;
  rc = plan_query(idx, Q, topk, target_ids != nullptr, max_targets, L, &p, RII_NOALLOC_SCRATCH_BYTES);
  if (rc) return rc;
  if (p.total > (size_t)RII_NOALLOC_SCRATCH_BYTES) return RII_ERR_UNSUPPORTED;  // beyond the static scratch
  void* ws = nullptr;
  rc = scratch_of_current_device(&ws);
  if (rc) return rc;
  return run_query(idx, p, q, Q, topk, target_ids, target_offsets, L, ids, dist, ws, static_cast<hipStream_t>(stream));
}

int rii_encode_device(const rii_index_t* idx, const float* x, int64_t n, uint8_t* codes_out, void* stream) {
  if (!idx || n < 0 || (n > 0 && (!x || !codes_out))) return RII_ERR_INVALID_ARG;
  if (n == 0) return RII_OK;
  const int Ds = idx->Ds, M = idx->M;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // The code book's fragments are 16 ceil(Ds / 4) registers a lane: up to Ds = 16 they and the rest
  // of k_encode_mfma stay in registers, above that the kernel with the code book in LDS runs.
  if (Ds <= 16 && (M + 3) / 4 <= 65535) {
    // a wave keeps its sub-space: two or three blocks of four sub-spaces run on a CU (by its registers), each
    // over every gridDim.x-th 64 vectors
    const int64_t tiles = (n + 63) / 64, groups = (M + 3) / 4;
    const int64_t want = std::max<int64_t>(1, (int64_t)kWantBlocks * (Ds <= 4 ? 3 : 2) / groups);
    const dim3 grid((unsigned)std::min(tiles, want), (unsigned)groups);
#define RII_ENCODE(S)                                                                                        \
  if (Ds == 4 * S) k_encode_mfma<S, true><<<grid, 256, 0, st>>>(idx->d_cb, x, n, idx->D, M, Ds, codes_out);  \
  else k_encode_mfma<S, false><<<grid, 256, 0, st>>>(idx->d_cb, x, n, idx->D, M, Ds, codes_out)
    switch ((Ds + 3) / 4) {
      case 1: RII_ENCODE(1); break;
      case 2: RII_ENCODE(2); break;
      case 3: RII_ENCODE(3); break;
      default: RII_ENCODE(4); break;
    }
#undef RII_ENCODE
    RII_HIP(hipGetLastError());
    return RII_OK;
  }
  size_t lds = (size_t)512 * Ds * 4;
  if (lds > 160 * 1024) return RII_ERR_UNSUPPORTED;
  int rc = set_lds(k_encode, lds);
  if (rc) return rc;
  const int64_t max_rows = (int64_t)1 << 30;
  for (int64_t r0 = 0; r0 < n; r0 += max_rows) {
    int64_t cnt = std::min(max_rows, n - r0);
    dim3 grid((unsigned)((cnt + 255) / 256), (unsigned)idx->M);
    k_encode<<<grid, 256, lds, st>>>(idx->d_cb, x + r0 * idx->D, cnt, idx->D, idx->M, Ds, codes_out + r0 * idx->M);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_rotate(const float* R, int D, const float* x, int64_t n, float* y, void* stream) {
  if (!R || D < 1 || n < 0 || (n > 0 && (!x || !y)) || x == y) return RII_ERR_INVALID_ARG;
  if (n == 0) return RII_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // Outputs per thread: the fewest blocks of at most 128 outputs, as narrow as they may be.  Rows per
  // thread: 8 as soon as that gives every CU its two blocks; below, where the call takes as long as
  // one block, 2 (and 2 outputs): 128 coordinates, 10,000 rows 28.6 -> 17.2 us, 60,000 141 -> 74 us; from
  // 70,000 on (159 -> 103 us) the larger tiles are at least level.
  const int cols = (D + 127) / 128, ot = (D + 16 * cols - 1) / (16 * cols);
  const bool few = (n + 127) / 128 * cols < 2 * kWantBlocks;
  const int64_t rows_per_launch = (int64_t)128 << 22;
  for (int64_t i0 = 0; i0 < n; i0 += rows_per_launch) {
    const int64_t cnt = std::min(rows_per_launch, n - i0);
    const float* xi = x + i0 * D;
    float* yi = y + i0 * D;
#define RII_ROTATE(RT, OT)                                                                                 \
  k_rotate<RT, OT><<<dim3((unsigned)((cnt + 16 * RT - 1) / (16 * RT)), (unsigned)((D + 16 * OT - 1) / (16 * OT))), \
                     256, 0, st>>>(R, D, xi, cnt, yi)
    if (few) RII_ROTATE(2, 2);
    else if (ot <= 2) RII_ROTATE(8, 2);
    else if (ot <= 4) RII_ROTATE(8, 4);
    else if (ot <= 6) RII_ROTATE(8, 6);
    else RII_ROTATE(8, 8);
#undef RII_ROTATE
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// The tables of the scan by matrix products: their place behind the code books (made by launch_matrix_batches).
static int matrix_dsp(int Ds) { return Ds <= 4 ? 4 : Ds <= 8 ? 8 : Ds <= 16 ? 16 : 32; }
size_t rii_internal_matrix_bytes(int M, int Ds) {
  if (!m_supported(M) || M * Ds > kMxMaxD || Ds > kMxMaxDs) return 0;
  return (size_t)M * 256 * (mx_entry_bytes(Ds) + 2 * matrix_dsp(Ds) * 4 + 8) + 256;
}
int rii_internal_matrix_books(rii_index* idx, void* where) {
  const int M = idx->M, Ds = idx->Ds;
  idx->mx_dsp = matrix_dsp(Ds);
  idx->mx_book = static_cast<uint8_t*>(where);
  idx->mx_fit = reinterpret_cast<float*>(idx->mx_book + (size_t)M * 256 * mx_entry_bytes(Ds));
  idx->mx_ch = idx->mx_fit + (size_t)M * idx->mx_dsp * 256;
  idx->mx_b = idx->mx_ch + (size_t)M * idx->mx_dsp * 256;
  idx->mx_bh = idx->mx_b + (size_t)M * 256;
  idx->mx_scale = idx->mx_bh + (size_t)M * 256;
  return RII_OK;
}

// lazily build the symmetric table
int rii_internal_sym_table(const rii_index* cidx, hipStream_t st) {
  rii_index* idx = const_cast<rii_index*>(cidx);
  if (idx->d_sym) return RII_OK;
  RII_HIP(hipMalloc(&idx->d_sym, (size_t)idx->M * 256 * 256 * 4));
  k_sym_table<<<dim3(256, idx->M), 256, 0, st>>>(idx->d_cb, idx->Ds, idx->d_sym);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// a(n) by brute force.  rot_base >= 0: `codes` is the base of a stored array (planes `plane`
// apart) and the items are its rows rot_base .. rot_base+n-1; rot_base < 0: n plain codes.  `open` not NULL:
// only those of the items that it lists (see k_assign).
int rii_internal_assign(const rii_index* idx, const uint8_t* codes, int64_t n, int64_t rot_base, int64_t plane,
                        const uint8_t* coarse, int K, int32_t* assign_out, const uint32_t* open, hipStream_t st) {
  if (!m_supported(idx->M)) return RII_ERR_UNSUPPORTED;
  if (n == 0) return RII_OK;
  if (!rot_m(idx->M) && rot_base >= 0) { codes += rot_base * idx->M; rot_base = -1; }
  int rc = rii_internal_sym_table(idx, st);
  if (rc) return rc;
  const int M = idx->M;
  const size_t lds = (size_t)M * 1024;
  int blocks = (int)std::min<int64_t>(n, open ? 256 * 8 : 256 * 16);
  DISPATCH_M(M, { int rc2 = set_lds(k_assign<MT>, lds); if (rc2) return rc2;
                  k_assign<MT><<<blocks, 256, lds, st>>>(idx->d_sym, codes, n, rot_base, plane, M, coarse, K, assign_out, open); });
  RII_HIP(hipGetLastError());
  return RII_OK;
}

int rii_assign(const rii_index_t* idx, const uint8_t* codes, int64_t n, const uint8_t* coarse, int K,
               int32_t* assign_out, void* stream) {
  if (!idx || n < 0 || K < 1 || !coarse || (n > 0 && (!codes || !assign_out))) return RII_ERR_INVALID_ARG;
  return rii_internal_assign(idx, codes, n, -1, 0, coarse, K, assign_out, nullptr, static_cast<hipStream_t>(stream));
}

// a(n) by matrix products (see k_assign_matrix), as far as they decide it; all pointers device.  Items as in
// rii_internal_assign, at most 2^31 of them; scratch: rii_internal_assign_matrix_bytes, or 0 when the dimension is
// beyond the kernel.  *open_out: the undecided items, for rii_internal_assign or rii_internal_assign_pruned.
size_t rii_internal_assign_matrix_bytes(const rii_index* idx, int64_t n, int K) {
  const int steps = (idx->D + 31) / 32, tiles = (K + 15) / 16;
  if (steps > 4 || !m_supported(idx->M)) return 0;
  return (size_t)tiles * steps * 2 * 64 * 16 + align_up((size_t)tiles * 64, 256) + align_up((size_t)idx->D * 1024, 256) + 256 +
         align_up((size_t)(n + 1) * 4, 256);
}

// The margin the products are used with, as a share of |x|^2 + max |c|^2 (see assign_margin).
float rii_internal_assign_margin(int M, int Ds) { return assign_margin((M * Ds + 31) / 32 * 32, M, Ds); }

// The margin of the scan's filter by matrix products, as a share of its magnitudes (see k_fit_sums).
float rii_internal_matrix_margin(int M, int Ds) { return mx_margin((M * Ds + 31) / 32 * 2, M); }

// What the device is taken to have room for at the most, for the products' scratch (tests of a full device).
void rii_internal_matrix_room(rii_index* idx, size_t most) {
  idx->mx_most = most;
  idx->mx_wait = idx->lists_extra.wait = idx->pick_extra.wait = 0;
}

// What the launches for left-over queries ask for (see left_chunks).
int64_t rii_internal_left_chunks(int per, int64_t groups, int64_t rows, int64_t big) { return left_chunks(per, groups, rows, big); }
int64_t rii_internal_left_blocks(int per, int64_t Q, int64_t big) { return left_blocks(per, Q, big); }
int64_t rii_internal_left_lists(int64_t Q, int64_t big) { return left_lists(Q, big); }
int64_t rii_internal_ivf_left_parts(int64_t n) { return ivf_left_parts((uint32_t)n); }

int rii_internal_assign_matrix(const rii_index* idx, const uint8_t* codes, int64_t n, int64_t rot_base, int64_t plane,
                               const uint8_t* coarse, int K, int32_t* assign_out, void* scratch, const uint32_t** open_out,
                               hipStream_t st) {
  const int M = idx->M, Ds = idx->Ds, steps = (idx->D + 31) / 32, tiles = (K + 15) / 16;
  if (!rot_m(M) && rot_base >= 0) { codes += rot_base * M; rot_base = -1; }
  uint8_t* w = static_cast<uint8_t*>(scratch);
  bf16x8_t* frag = reinterpret_cast<bf16x8_t*>(w); w += (size_t)tiles * steps * 2 * 64 * 16;
  float* c2 = reinterpret_cast<float*>(w); w += align_up((size_t)tiles * 64, 256);
  float* books = reinterpret_cast<float*>(w); w += align_up((size_t)idx->D * 1024, 256);
  uint32_t* cmax = reinterpret_cast<uint32_t*>(w); w += 256;
  uint32_t* open = reinterpret_cast<uint32_t*>(w);
  k_centred_books<<<dim3((unsigned)M, (unsigned)Ds), 256, 0, st>>>(idx->d_cb, M, Ds, coarse, K, books, cmax, open);
  k_centre_frags<<<tiles, 64, 0, st>>>(books, M, Ds, coarse, K, steps, frag, c2, cmax);
#define RII_ASSIGN(S, T)                                                                              \
  k_assign_matrix<S, T><<<(unsigned)((n + 64 * T - 1) / (64 * T)), 256, 0, st>>>(books, M, Ds, codes, n, rot_base, plane, \
                                                                                 frag, c2, cmax, tiles, assign_out, open)
  switch (steps) {
    case 1: RII_ASSIGN(1, 4); break;
    case 2: RII_ASSIGN(2, 4); break;
    case 3: RII_ASSIGN(3, 2); break;
    default: RII_ASSIGN(4, 2); break;
  }
#undef RII_ASSIGN
  RII_HIP(hipGetLastError());
  *open_out = open;
  return RII_OK;
}

// a(n) with pruning (see k_assign_pruned); all pointers device; `open` as in rii_internal_assign.  visited_total may be NULL.
int rii_internal_assign_pruned(const rii_index* idx, const uint8_t* codes, int64_t n, int64_t rot_base, int64_t plane,
                               const uint8_t* super, int G,
                               const float* radius, const uint8_t* coarse_g, const int32_t* perm_g,
                               const int32_t* group_off, int32_t* assign_out, const uint32_t* open,
                               unsigned long long* visited_total, hipStream_t st) {
  if (n == 0) return RII_OK;
  if (!rot_m(idx->M) && rot_base >= 0) { codes += rot_base * idx->M; rot_base = -1; }
  int rc = rii_internal_sym_table(idx, st);
  if (rc) return rc;
  const int M = idx->M;
  const size_t lds = (size_t)M * 1024 + (size_t)G * 4;
  if (lds > 150 * 1024) return RII_ERR_UNSUPPORTED;
  int blocks = (int)std::min<int64_t>(n, 256 * 32);
  DISPATCH_M(M, { int rc2 = set_lds(k_assign_pruned<MT>, lds); if (rc2) return rc2;
                  k_assign_pruned<MT><<<blocks, 256, lds, st>>>(idx->d_sym, codes, n, rot_base, plane, M, super, G, radius,
                                                               coarse_g,
                                                               perm_g, group_off, assign_out, open, visited_total); });
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// Posting lists (off [K+1], ids [n], ascending inside a list) of device-resident a(n).  Scratch:
// rii_internal_lists_bytes, 0 when K is beyond what a block counts in LDS.
static int64_t list_chunk(int64_t n, int K) {
  const int64_t most = std::max<int64_t>(1, ((int64_t)1 << 26) / K);  // chunks: at most 256 MB of counts
  return std::max<int64_t>(4096, ((n + most - 1) / most + 63) / 64 * 64);
}
size_t rii_internal_lists_bytes(int64_t n, int K) {
  if ((size_t)K * 4 > 150 * 1024 || n < 1) return 0;
  const int64_t chunks = (n + list_chunk(n, K) - 1) / list_chunk(n, K);
  return align_up((size_t)chunks * K * 4, 256) + align_up((size_t)K * 4, 256);
}
int rii_internal_build_lists(const int32_t* assign, int64_t n, int K, int64_t* off, int32_t* ids, void* scratch, hipStream_t st) {
  const int64_t chunk = list_chunk(n, K);
  const int chunks = (int)((n + chunk - 1) / chunk);
  uint32_t* counts = static_cast<uint32_t*>(scratch);
  uint32_t* lengths = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(scratch) + align_up((size_t)chunks * K * 4, 256));
  const size_t lds = (size_t)K * 4;
  int rc = set_lds(k_list_count, lds);
  if (!rc) rc = set_lds(k_list_fill, lds);
  if (rc) return rc;
  int bits = 0;
  while (bits < 31 && (K - 1) >> bits) ++bits;
  k_list_count<<<chunks, 256, lds, st>>>(assign, n, chunk, K, counts);
  k_list_starts<<<(K + 63) / 64, 64, 0, st>>>(counts, chunks, K, lengths);
  k_list_offsets<<<1, 1024, 0, st>>>(lengths, K, off);
  k_list_fill<<<chunks, 64, lds, st>>>(assign, n, chunk, K, bits, counts, off, ids);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// One update round of the clustering in code space (see k_update_centres); all pointers device.
int rii_internal_update_centres(const rii_index* idx, const uint8_t* sample, const int64_t* off, const int32_t* ids, int K,
                                uint8_t* coarse, hipStream_t st) {
  int rc = rii_internal_sym_table(idx, st);
  if (rc) return rc;
  k_update_centres<<<dim3((unsigned)K, (unsigned)idx->M), 256, 0, st>>>(idx->d_sym, sample, idx->M, off, ids, coarse);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// a(n) of every stored item from the installed posting lists (device buffer of N entries)
int rii_internal_assign_from_lists(const rii_index* idx, int32_t* d_out, hipStream_t st) {
  if (idx->N == 0) return RII_OK;
  const int64_t per = (int64_t)1 << 30;
  if (idx->N > per * 2 - 1) return RII_ERR_UNSUPPORTED;
  k_assign_from_lists<<<(unsigned)((idx->N + 255) / 256), 256, 0, st>>>(idx->d_list_off, idx->d_list_ids, idx->K, idx->N, d_out);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// used by the threshold calibration in rii_index.hip
int rii_internal_spread_ids(int32_t* ids, int64_t* offsets, int nq, int64_t S, int64_t N, hipStream_t st) {
  int64_t total = std::max<int64_t>((int64_t)nq * S, nq + 1);
  k_spread_ids<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(ids, offsets, nq, S, N);
  RII_HIP(hipGetLastError());
  return RII_OK;
}

// used by rii_index.hip: see k_copy_rows.  For M without a stored form the rotation arguments only
// select the first row of the (plain) arrays.
int rii_internal_copy_rows(const uint8_t* in, int64_t in_rot, int64_t in_plane, const int32_t* ids, int64_t n, int M,
                           uint8_t* out, int64_t out_rot, int64_t out_plane, hipStream_t st) {
  if (n == 0) return RII_OK;
  if (!rot_m(M)) {
    if (in_rot > 0) in += in_rot * M;
    if (out_rot > 0) out += out_rot * M;
    in_rot = out_rot = -1;
  }
  const int M4 = M / 4;
  const int64_t per = ((int64_t)1 << 30) / M4;  // rows per launch
  for (int64_t r0 = 0; r0 < n; r0 += per) {
    int64_t cnt = std::min<int64_t>(per, n - r0);
    int64_t dw = cnt * M4;
    // rows r0.. of this call: shift the row bases of stored arrays, the pointers of plain ones
    const bool seq = !ids;  // source rows follow the output rows
    k_copy_rows<<<(unsigned)((dw + 255) / 256), 256, 0, st>>>(
        seq && in_rot < 0 ? in + r0 * M : in, seq && in_rot >= 0 ? in_rot + r0 : in_rot, in_plane,
        ids ? ids + r0 : nullptr, cnt, M, out_rot < 0 ? out + r0 * M : out, out_rot >= 0 ? out_rot + r0 : out_rot,
        out_plane);
  }
  RII_HIP(hipGetLastError());
  return RII_OK;
}

}  // extern "C"

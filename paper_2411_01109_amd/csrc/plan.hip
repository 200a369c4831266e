// Status strings, graph validation and the plan of the discretized SpMM
// (paper section 5.2.1: edges are dealt out in storage order in fixed-size batches,
// observation rules 1-3).  Integer work only; everything here is one-off set-up.
#include <stdarg.h>
#include <stdio.h>

#include <hsa/hsa.h>

#include <algorithm>
#include <mutex>

#include "ranges.h"

namespace hgnn {

static thread_local char g_err[512] = "";

// ---- cache sizes of the current device ----------------------------------------------------------------
// L2 (per XCD) from the HIP device attribute; the last-level cache behind the L2s (the Infinity Cache) is not a
// HIP attribute, so it is read from the HSA agent's cache list (level 3).  Either falls back to the MI355X
// figure (4 MB, 256 MB) when the query gives nothing.
struct CacheQuery {
  int want;      // ordinal of the GPU agent looked for
  int seen;      // GPU agents met so far
  int64_t l3;    // largest level-3 cache of that agent
};

static hsa_status_t cache_cb(hsa_cache_t cache, void* data) {
  CacheQuery* q = static_cast<CacheQuery*>(data);
  uint8_t level = 0;
  uint32_t size = 0;
  if (hsa_cache_get_info(cache, HSA_CACHE_INFO_LEVEL, &level) == HSA_STATUS_SUCCESS &&
      hsa_cache_get_info(cache, HSA_CACHE_INFO_SIZE, &size) == HSA_STATUS_SUCCESS && level == 3) {
    // the attribute is specified in bytes; runtimes have been seen to hand through the driver's KiB figure.  No
    // last-level cache is below 1 MiB and none is 2^30 KiB, so the unit can be told from the value
    int64_t bytes = int64_t(size);
    if (bytes < (int64_t(1) << 20)) bytes <<= 10;
    if (bytes > q->l3) q->l3 = bytes;
  }
  return HSA_STATUS_SUCCESS;
}

static hsa_status_t agent_cb(hsa_agent_t agent, void* data) {
  CacheQuery* q = static_cast<CacheQuery*>(data);
  hsa_device_type_t type;
  if (hsa_agent_get_info(agent, HSA_AGENT_INFO_DEVICE, &type) != HSA_STATUS_SUCCESS || type != HSA_DEVICE_TYPE_GPU)
    return HSA_STATUS_SUCCESS;
  if (q->seen++ == q->want) (void)hsa_agent_iterate_caches(agent, cache_cb, q);
  return HSA_STATUS_SUCCESS;
}

void device_cache_bytes(int64_t* l2, int64_t* llc) {
  *l2 = int64_t(4) << 20;
  *llc = int64_t(256) << 20;
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess) return;
  // asked once per device: compute calls consult the sizes too
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static bool known[kMaxDev];
  static int64_t kept[kMaxDev][2];
  std::lock_guard<std::mutex> lock(mu);
  if (dev >= 0 && dev < kMaxDev && known[dev]) {
    *l2 = kept[dev][0];
    *llc = kept[dev][1];
    return;
  }
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeL2CacheSize, dev) == hipSuccess && v > 0) *l2 = v;
  if (hsa_init() == HSA_STATUS_SUCCESS) {
    CacheQuery q{dev, 0, 0};
    (void)hsa_iterate_agents(agent_cb, &q);
    (void)hsa_shut_down();
    if (q.l3 > 0) *llc = q.l3;
  }
  if (dev >= 0 && dev < kMaxDev) {
    kept[dev][0] = *l2;
    kept[dev][1] = *llc;
    known[dev] = true;
  }
}

hgnn_status fail(hgnn_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return s;
}
void clear_error() { g_err[0] = 0; }

hgnn_status check_csr_args(const hgnn_csr* g, const char* who) {
  HGNN_REQUIRE(g != nullptr, HGNN_EINVAL, "%s: graph is NULL", who);
  HGNN_REQUIRE(g->nrows >= 0 && g->ncols >= 0 && g->nnz >= 0, HGNN_EINVAL, "%s: negative graph size", who);
  HGNN_REQUIRE(g->nnz < (int64_t(1) << 31), HGNN_EINVAL, "%s: nnz = %lld does not fit int32", who, (long long)g->nnz);
  HGNN_REQUIRE(g->rowptr != nullptr, HGNN_EINVAL, "%s: rowptr is NULL", who);
  HGNN_REQUIRE(g->nnz == 0 || g->col != nullptr, HGNN_EINVAL, "%s: col is NULL", who);
  return HGNN_OK;
}

// ---- validation ---------------------------------------------------------------------------------
// Results of the passes over a graph that the host waits for, zeroed before the first one.
struct GraphFacts {
  int bad;                        // 8 - the smallest number of the offset array's rules (1-3) that is broken, 0 = none
  int bad_edge;                   // the same for rules 4-6
  int n_split, n_big, n_mid;      // rows in the three lists of a plan
  int n_chunks;                   // chunks of kHubEdges of the long rows
  unsigned long long listed;      // non-zeros of the long and middle rows
  unsigned long long drops;       // positions whose column is below their predecessor's
  unsigned long long drops_ok;    // rows whose first column is below the column before it
};
static_assert(sizeof(GraphFacts) <= kMailBytes, "GraphFacts goes through a mail slot");

// The offset array first (rules 1-3); the per-edge rules only count on a graph that passed them, because they index with
// values that are in range only when it is monotone and has the right end points.
__global__ void validate_rowptr_kernel(hgnn_csr g, GraphFacts* f) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  int bad = 0;
  if (i == 0) {
    if (g.rowptr[0] != 0) bad = 1;
    else if (int64_t(g.rowptr[g.nrows]) != g.nnz) bad = 2;
  }
  if (!bad && i < g.nrows && g.rowptr[i] > g.rowptr[i + 1]) bad = 3;
  if (bad) atomicMax(&f->bad, 8 - bad);
}

template <int THREADS>
__device__ __forceinline__ void add_block_total(int v, unsigned long long* total) {  // blockDim.x == THREADS
  __shared__ int part[THREADS / kWave];
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off);
  if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int w = 0; w < THREADS / kWave; ++w) t += part[w];
    if (t) atomicAdd(total, (unsigned long long)t);
  }
}

// Rules 4-7.  A column id may only drop where a new row starts (rule 7): the positions where it drops are counted over the
// stream of column ids, the row starts among them over the rows, and the two numbers are equal exactly when no drop lies
// inside a row (43 us with a search of the row of every drop at 5.5 M non-zeros).  Few workgroups, each adding its total
// once: thousands of additions to one address took longer than the pass (51 us).
constexpr int kEdgesPerThread = 8;
constexpr int kFactBlocks = 512;  // most workgroups that add to a fact: of 1024 lanes, all that the chip holds (with 256 lanes
                                  // 16 us at 5.5 M non-zeros, 29 with an edge-id map; 14 and 16)
constexpr int kFactThreads = 1024;
__global__ __launch_bounds__(kFactThreads) void validate_edges_kernel(hgnn_csr g, GraphFacts* f, int64_t edge_blocks, int64_t row_blocks,
                                                                    RangeLists ranges) {
  if (f->bad) return;  // written by the launch before
  // windows whose long rows are cut beside the checks come first: theirs are the longest chains
  const int64_t b = int64_t(blockIdx.x) - ranges.nwin;
  if (b < 0) {
    range_cut<kFactThreads>(ranges, int(blockIdx.x));
    return;
  }
  if (b >= edge_blocks) {
    int ok = 0;
    for (int64_t r = (b - edge_blocks) * kFactThreads + threadIdx.x; r < g.nrows; r += row_blocks * kFactThreads) {
      const int p = g.rowptr[r], e = g.rowptr[r + 1];
      if (p < e && p > 0) ok += g.col[p - 1] > g.col[p];
    }
    add_block_total<kFactThreads>(ok, &f->drops_ok);
    return;
  }
  int bad = 0, drops = 0;
  for (int64_t i0 = b * (kFactThreads * kEdgesPerThread) + threadIdx.x; i0 < g.nnz;
       i0 += edge_blocks * (kFactThreads * kEdgesPerThread)) {
    int c[kEdgesPerThread], before[kEdgesPerThread], e[kEdgesPerThread];
#pragma unroll
    for (int u = 0; u < kEdgesPerThread; ++u) {
      const int64_t i = i0 + u * kFactThreads;
      c[u] = i < g.nnz ? g.col[i] : 0;
      before[u] = i < g.nnz && i > 0 ? g.col[i - 1] : -1;
      e[u] = g.eid && i < g.nnz ? g.eid[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < kEdgesPerThread; ++u) {
      const int64_t i = i0 + u * kFactThreads;
      if (i >= g.nnz) break;
      int b = 0;
      if (c[u] < 0 || c[u] >= g.ncols) b = 4;
      if (!b && (e[u] < 0 || int64_t(e[u]) >= g.nnz)) b = 5;
      if (!b && g.row) {
        const int r = g.row[i];
        if (r < 0 || r >= g.nrows) b = 6;
        else if (!(int64_t(g.rowptr[r]) <= i && i < int64_t(g.rowptr[r + 1]))) b = 6;
      }
      if (i > 0) drops += before[u] > c[u];
      if (b && (bad == 0 || b < bad)) bad = b;
    }
  }
  if (bad) atomicMax(&f->bad_edge, 8 - bad);
  add_block_total<kFactThreads>(drops, &f->drops);
}

static const char* const kRule[] = {"ok",
                                    "rowptr[0] != 0",
                                    "rowptr[nrows] != nnz",
                                    "rowptr decreases",
                                    "a column id is outside [0, ncols)",
                                    "an edge id is outside [0, nnz)",
                                    "a COO row id disagrees with rowptr",
                                    "column ids are not ascending inside a row"};

// ranges.nwin windows beside the checks (0: none)
static hipError_t launch_validate_edges(const hgnn_csr* g, GraphFacts* facts, const RangeLists& ranges, hipStream_t s) {
  if (g->nnz > 0) {
    const int64_t eb = std::min<int64_t>(kFactBlocks, ceil_div(g->nnz, int64_t(kFactThreads) * kEdgesPerThread));
    const int64_t rb = std::min<int64_t>(kFactBlocks / 2, ceil_div(g->nrows, kFactThreads));
    validate_edges_kernel<<<dim3(unsigned(eb + rb + ranges.nwin)), kFactThreads, 0, s>>>(*g, facts, eb, rb, ranges);
  }
  return hipGetLastError();
}

static hipError_t launch_validate(const hgnn_csr* g, GraphFacts* facts, hipStream_t s) {
  hipError_t e = hipMemsetAsync(facts, 0, sizeof(GraphFacts), s);
  if (e != hipSuccess) return e;
  validate_rowptr_kernel<<<dim3(unsigned(ceil_div(int64_t(g->nrows) + 1, kBlock))), kBlock, 0, s>>>(*g, facts);
  return launch_validate_edges(g, facts, RangeLists{}, s);
}

static hgnn_status check_facts(const GraphFacts& f) {
  const int rule = f.bad ? 8 - f.bad : (f.bad_edge ? 8 - f.bad_edge : (f.drops != f.drops_ok ? 7 : 0));
  if (rule) return fail(HGNN_EINVAL, "hgnn_csr_validate: %s", kRule[rule > 0 && rule < 8 ? rule : 0]);
  return HGNN_OK;
}

// ---- first and last row of every segment: binary searches in the offset array ------------------------
__device__ __forceinline__ void seg_rows(const int* __restrict__ rowptr, int nrows, int64_t nnz, int S, int64_t nseg, int64_t k,
                                         int* __restrict__ lo, int* __restrict__ hi) {
  if (k >= nseg) return;
  int64_t e0 = k * S, e1 = e0 + S < nnz ? e0 + S : nnz;
  lo[k] = row_of_edge(rowptr, nrows, e0);
  hi[k] = row_of_edge(rowptr, nrows, e1 - 1);
}

// ---- the row lists of a plan ------------------------------------------------------------------------------
// split: first and last edge of the row fall in different segments; big: longer than big_deg; mid: longer than mid_deg and
// not big.  One pass counts the members of all three per workgroup (and the chunks of the long rows and the non-zeros of
// the two length lists), one workgroup turns the counts into offsets and hands the totals to the host, one pass writes
// the lists in row order.
struct RowLists {
  const int* rowptr;
  int nrows, S, big_deg, mid_deg;
};

constexpr int kRowsPerThread = 4;
constexpr int kRowsPerBlock = kBlock * kRowsPerThread;
enum { kSplitList, kBigList, kMidList, kChunkList, kLists };

__device__ __forceinline__ void row_memberships(const RowLists& q, int r, int (&m)[kLists], int& len) {
  const int b = q.rowptr[r], e = q.rowptr[r + 1];
  len = e - b;
  m[kSplitList] = e > b && (b / q.S) != ((e - 1) / q.S);
  m[kBigList] = len > q.big_deg;
  m[kMidList] = len > q.mid_deg && len <= q.big_deg;
  m[kChunkList] = m[kBigList] ? pieces_of(len, kHubEdges) : 0;
}

// exclusive scan of one value per thread over the workgroup (blockDim.x == kBlock)
__device__ inline int block_exclusive_scan(int v, int* total) {
  __shared__ int wsum[kBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int incl = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int t = __shfl_up(incl, d);
    if (lane >= d) incl += t;
  }
  __syncthreads();  // a previous scan has been read
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) {
    if (w < wave) before += wsum[w];
    all += wsum[w];
  }
  *total = all;
  return before + incl - v;
}

// A workgroup per window of rows (kRowsPerBlock = kTaskWindow): the rules of the offset array, the members of the row lists and the
// pieces of the row tasks.  The three as launches of their own took 14 us at 262 144 rows, this one 9.
static_assert(kRowsPerBlock == kTaskWindow && kBlock == kTaskThreads, "row lists and row tasks share their windows");
template <bool MIDS>
__global__ __launch_bounds__(kBlock) void plan_count_kernel(hgnn_csr g, RowLists q, TaskSource tq, int nblk, int* __restrict__ counts,
                                                            int* __restrict__ task_counts, GraphFacts* f) {
  constexpr int kListed = kLists + kTaskAll, kSums = kListed + 1;
  __shared__ int s_total[kSums], s_sample;
  if (threadIdx.x < kSums) s_total[threadIdx.x] = 0;
  if (MIDS && threadIdx.x == 0) s_sample = 0;
  __syncthreads();
  const int64_t base = int64_t(blockIdx.x) * kRowsPerBlock + threadIdx.x * kRowsPerThread;
  int bad = 0;
  if (base == 0) {
    if (g.rowptr[0] != 0) bad = 1;
    else if (int64_t(g.rowptr[g.nrows]) != g.nnz) bad = 2;
  }
  const MidSample<MIDS> sample(tq);
  int c[kLists] = {0, 0, 0, 0}, n[kTaskAll] = {}, listed = 0;
  for (int u = 0; u < kRowsPerThread; ++u) {
    if (base + u >= q.nrows) break;
    const int r = int(base) + u;
    int m[kLists], len;
    row_memberships(q, r, m, len);
    if (!bad && len < 0) bad = 3;
    for (int i = 0; i < kLists; ++i) c[i] += m[i];
    if (m[kBigList] || m[kMidList]) listed += len;
    task_count_row<true, MIDS>(tq, g.rowptr, r, n);
  }
  if (bad) atomicMax(&f->bad, 8 - bad);
#pragma unroll
  for (int i = 0; i < kSums; ++i) {
    const int v = wave_sum(i < kLists ? c[i < kLists ? i : 0] : (i < kListed ? n[i < kListed && i >= kLists ? i - kLists : 0] : listed));
    if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(&s_total[i], v);
  }
  sample.add(&s_sample);
  __syncthreads();
  if (nblk == 0) return;  // no rows
  const int i = threadIdx.x;
  const int counters = tq.range_min == kNoRanges ? kTaskCounters : kTaskAll;
  if (i < kLists) counts[i * nblk + blockIdx.x] = s_total[i];
  else if (i < kLists + counters)
    task_counts[int64_t(i - kLists) * nblk + blockIdx.x] = task_counter<true, MIDS>(s_total + kLists, i - kLists, MIDS && MidSample<MIDS>::many(tq, s_sample));
  else if (i == kListed && s_total[i]) atomicAdd(&f->listed, (unsigned long long)s_total[i]);
}

// one workgroup: exclusive scans of the n block counts of every list in place; the totals and what earlier passes left in
// `facts` go to `out` (host memory)
__device__ __forceinline__ void row_lists_scan(int* __restrict__ counts, int n, const GraphFacts* __restrict__ facts, GraphFacts* out) {
  int carry[kLists] = {0, 0, 0, 0};
  for (int base = 0; base < n; base += kBlock) {
    const int i = base + threadIdx.x;
    for (int l = 0; l < kLists; ++l) {
      const int v = i < n ? counts[l * n + i] : 0;
      int tot;
      const int ex = block_exclusive_scan(v, &tot);
      if (i < n) counts[l * n + i] = carry[l] + ex;
      carry[l] += tot;
    }
  }
  if (threadIdx.x == 0) {
    GraphFacts r = *facts;
    r.n_split = carry[kSplitList];
    r.n_big = carry[kBigList];
    r.n_mid = carry[kMidList];
    r.n_chunks = carry[kChunkList];
    *out = r;
  }
}

// two workgroups: the row lists and the row tasks; a third: the pieces at column ranges
__global__ __launch_bounds__(kBlock) void plan_scan_kernel(TaskSource tq, int n, int* __restrict__ counts, const GraphFacts* __restrict__ facts,
                                                          GraphFacts* out, int* __restrict__ task_counts, int* __restrict__ sums,
                                                          hgnn_task_sec* __restrict__ sec, TaskTotals* totals, RangeLists ranges,
                                                          int* n_range) {
  if (blockIdx.x == 0) {
    row_lists_scan(counts, n, facts, out);
  } else if (blockIdx.x == 1) {
    task_scan(tq, n, task_counts, sums, sec, totals);
  } else {
    const int all = range_scan_all(ranges);
    if (threadIdx.x == 0) *n_range = all;
  }
}

struct RowListArrays {
  int *split_row, *split_lo, *split_hi, *big_row, *big_first, *mid_row, *chunk_row, *chunk_first, *chunk_count;
};

__device__ __forceinline__ void row_lists_write(const RowLists& q, int b, int nblk, const int* __restrict__ offsets, const RowListArrays& o) {
  const int base = b * kRowsPerBlock + threadIdx.x * kRowsPerThread;
  int m[kRowsPerThread][kLists], c[kLists] = {0, 0, 0, 0}, pos[kLists];
  for (int u = 0; u < kRowsPerThread; ++u) {
    for (int i = 0; i < kLists; ++i) m[u][i] = 0;
    int len;
    if (base + u < q.nrows) row_memberships(q, base + u, m[u], len);
    for (int i = 0; i < kLists; ++i) c[i] += m[u][i];
  }
  for (int i = 0; i < kLists; ++i) {
    int total;
    pos[i] = offsets[i * nblk + b] + block_exclusive_scan(c[i], &total);
  }
  for (int u = 0; u < kRowsPerThread; ++u) {
    const int r = base + u;
    if (m[u][kSplitList]) {
      const int k = pos[kSplitList]++;
      o.split_row[k] = r;
      o.split_lo[k] = q.rowptr[r] / q.S;
      o.split_hi[k] = (q.rowptr[r + 1] - 1) / q.S;
    }
    if (m[u][kMidList]) o.mid_row[pos[kMidList]++] = r;
    if (m[u][kBigList]) {
      const int k = pos[kBigList]++, first = pos[kChunkList], nch = m[u][kChunkList];
      o.big_row[k] = r;
      o.big_first[k] = first;
      for (int j = 0; j < nch; ++j) {
        o.chunk_row[first + j] = r;
        o.chunk_first[first + j] = first;
        o.chunk_count[first + j] = nch;
      }
      pos[kChunkList] += nch;
    }
  }
}

// Workgroups for the windows of the row tasks, then (with members) for those of the row lists and of the rows cut at column ranges, then
// for the segments: none needs
// what another one writes, and as launches of their own they took 25 us at 5.5 M non-zeros, mostly latency, in one 11.
template <bool MIDS>
__global__ __launch_bounds__(kBlock) void plan_write_kernel(TaskSource tq, int n, const int* __restrict__ task_counts, const int* __restrict__ sums,
                                                           hgnn_task_sec* __restrict__ sec, int4* __restrict__ task, int* __restrict__ zrow,
                                                           int4* __restrict__ split, RowLists q, int list_blocks,
                                                           const int* __restrict__ offsets, RowListArrays o, int64_t nseg,
                                                           int* __restrict__ seg_lo, int* __restrict__ seg_hi, RangeLists ranges,
                                                           int range_blocks, const int* __restrict__ split_at, int4* __restrict__ rtask,
                                                           int4* __restrict__ rsplit) {
  // (those of the column ranges, the longest chains, come first)
  const int b = int(blockIdx.x) - range_blocks;
  if (b < 0) {
    const int w = int(blockIdx.x) * kRangeGroup;
    RangePlace at;
#pragma unroll
    for (int x = 0; x < kRanges; ++x) at.task[x] = ranges.count[x * ranges.nwin + w];
    at.slot = ranges.slots[w];
    at.split = split_at[w];
    range_write(ranges, w, at, rtask, rsplit);
  } else if (b < n) {
    task_write<false, true, MIDS>(tq, b, 0, n, task_counts, sums, sec, nullptr, task, zrow, split, 0);
  } else if (b < n + list_blocks) {
    row_lists_write(q, b - n, n, offsets, o);
  } else {
    seg_rows(q.rowptr, q.nrows, tq.nnz, q.S, nseg, (int64_t(b) - n - list_blocks) * kBlock + threadIdx.x, seg_lo, seg_hi);
  }
}

// Which plans have long rows cut at column ranges, beside the ordinary pieces of those rows (at_ranges in task.h says which a call takes).  A
// segment size is the least length because such rows leave staged partial rows (fp16, as ever) in any case: as many at S, more at the
// ranges, and the sum of their roundings no larger (rows of 257, 1000, 4000 non-zeros 2.04e-4 against 2.06e-4, 2.11 against 2.07, 2.10
// against 2.12 relative to float64).  us a call, rows in pieces of S / at column ranges (F = 64 and one head if not said; power law unless log-normal):
//   table, non-zeros                  SpMM, edge values   behind a map   SDDMM       attention fwd (saving), bwd
//   614 MB, 62 M, F = 128               1711 / 1285        2683 / 2043
//   307 MB, 62 M, F = 64 by degrees      870 / 740
//   154 MB, 31 M                         359 / 328          772 / 624    350 / 332
//   256 MB, 13 M, F = 256                747 / 618         1012 / 783
//   77 MB, 60 M, F = 16                  738 / 611         1640 / 1422
//   77 MB, 12 M                          129 / 118          280 / 222    125 / 115
//   134 MB, 26 M log-normal, 4 heads     930 / 819         1183 / 1169   937 / 802
//   67 MB, 5.5 M, F = 128                                                            179 / 166, 213 / 195
//   34 MB, 21 M                          142 / 135          352 / 312    136 / 128
//   34 MB, 5.5 M, 4 heads                 59 / 59           123 / 114     59 / 59    105 / 102, 132 / 124
//   13 MB, 8 M                            58 / 61           106 / 101     52 / 52
//   8 MB, 8 M                             56 / 64            96 / 94      50 / 53
//   34 MB, 2.1 M, F = 128: GIN layer forward 44 / 46; 10 MB, 1.3 M: by degrees 30 / 48
// The cuts ride beside the checks of the columns and the lists beside the others (a plan of 5.5 M non-zeros 72 -> 82 us), so the line lies
// where the calls begin to gain: at four L2s.
static int range_min_row(int64_t nnz, int64_t ncols, int max_F, int S, int64_t l2) {
  constexpr int64_t kLeastNnz = int64_t(4) << 20;
  return nnz > kLeastNnz && ncols * max_F * 2 > 4 * l2 ? S + 1 : kNoRanges;
}

// Validates the graph g and builds the segment arrays, row lists and row tasks of p for it (p->S, p->nseg, p->max_F set by the
// caller).  The host waits twice: for the totals of the lists (which size the allocations) and for the arrays.
hgnn_status plan_build_arrays(hgnn_plan* p, const hgnn_csr* g, bool blocks, SetupStream& s) {
  const int64_t E = g->nnz;
  const int nblk = int(ceil_div(g->nrows, kRowsPerBlock));
  DevTemp facts_buf(s), counts_buf(s);
  HostMail mail(s);
  HGNN_HIP(facts_buf.alloc(2 * sizeof(GraphFacts)));
  HGNN_HIP(counts_buf.alloc(sizeof(int) * kLists * (size_t(nblk) + 1)));
  GraphFacts* facts = facts_buf.as<GraphFacts>();
  GraphFacts* totals = mail.data ? reinterpret_cast<GraphFacts*>(mail.data) : facts + 1;
  int* counts = counts_buf.as<int>();
  const RowLists q{g->rowptr, g->nrows, p->S, p->big_deg, p->mid_deg};
  const TaskSource tq{g->rowptr, nullptr, g->nrows, 1, p->S, task_group_max(g->nnz), g->nnz,
                      blocks ? kNoRanges : range_min_row(E, g->ncols, p->max_F, p->S, p->l2_bytes)};
  TaskCounts tc(s);
  hgnn_status st = task_prepare(tq, tc);
  if (st != HGNN_OK) return st;
  HGNN_HIP(hipMemsetAsync(facts, 0, sizeof(GraphFacts), s));
  const bool mids = has_mids(tq);
  const auto count_kernel = mids ? plan_count_kernel<true> : plan_count_kernel<false>;
  count_kernel<<<dim3(unsigned(nblk > 0 ? nblk : 1)), kBlock, 0, s>>>(*g, q, tq, nblk, counts, tc.count, facts);
  RangeLists ranges{};
  DevTemp range_mem(s);
  tc.ranges = tq.range_min != kNoRanges && nblk > 0;
  if (tc.ranges) {
    const size_t cut_bytes = range_cut_bytes(g->nrows, E, tq.range_min);
    HGNN_HIP(range_mem.alloc(cut_bytes + sizeof(int) * (kRanges + 1) * size_t(nblk)));
    int* const count = reinterpret_cast<int*>(static_cast<char*>(range_mem.p) + cut_bytes);
    ranges = range_lists(tq, g->col, g->ncols, nblk, range_mem.as<int>(), count, count + kRanges * size_t(nblk), nullptr);
  }
  HGNN_HIP(launch_validate_edges(g, facts, ranges, s));
  plan_scan_kernel<<<tc.ranges ? 3 : 2, kBlock, 0, s>>>(tq, nblk, counts, facts, totals, tc.count, tc.sums, tc.sec, tc.totals, ranges, tc.n_range);
  HGNN_LAUNCH_CHECK("plan_count_kernel / plan_scan_kernel");
  GraphFacts f;
  if (!mail.data) HGNN_HIP(hipMemcpyAsync(&f, totals, sizeof(f), hipMemcpyDeviceToHost, s));
  HGNN_HIP(s.wait());
  if (mail.data) f = *totals;
  st = check_facts(f);
  if (st != HGNN_OK) return st;
  p->n_split = f.n_split;
  p->n_big = f.n_big;
  p->n_mid = f.n_mid;
  p->n_hub_chunks = f.n_chunks;
  p->listed_nnz = int64_t(f.listed);
  if (E > 0) {
    HGNN_HIP(dev_malloc(&p->seg_row_lo, sizeof(int) * size_t(p->nseg)));
    HGNN_HIP(dev_malloc(&p->seg_row_hi, sizeof(int) * size_t(p->nseg)));
  }
  if (p->n_split > 0) {
    HGNN_HIP(dev_malloc(&p->split_row, sizeof(int) * size_t(p->n_split)));
    HGNN_HIP(dev_malloc(&p->split_seg_lo, sizeof(int) * size_t(p->n_split)));
    HGNN_HIP(dev_malloc(&p->split_seg_hi, sizeof(int) * size_t(p->n_split)));
  }
  if (p->n_mid > 0) HGNN_HIP(dev_malloc(&p->mid_row, sizeof(int) * size_t(p->n_mid)));
  if (p->n_big > 0) {  // the long rows and their chunk table
    const size_t nc = size_t(p->n_hub_chunks);
    HGNN_HIP(dev_malloc(&p->big_row, sizeof(int) * size_t(p->n_big)));
    HGNN_HIP(dev_malloc(&p->big_first, sizeof(int) * size_t(p->n_big)));
    HGNN_HIP(dev_malloc(&p->hub_chunk_row, sizeof(int) * nc));
    HGNN_HIP(dev_malloc(&p->hub_chunk_first, sizeof(int) * nc));
    HGNN_HIP(dev_malloc(&p->hub_chunk_count, sizeof(int) * nc));
    HGNN_HIP(dev_malloc(&p->hub_part, sizeof(float) * 2 * nc * size_t(p->max_H)));
  }
  st = task_allocate(tq, tc, p->max_F, p->max_H, &p->tasks);
  if (st != HGNN_OK) return st;
  const int list_blocks = p->n_split + p->n_mid + p->n_big > 0 ? nblk : 0;
  const int range_blocks = tc.got.n_range > 0 ? int(ceil_div(nblk, kRangeGroup)) : 0;
  const int64_t grid = int64_t(nblk) + list_blocks + range_blocks + ceil_div(p->nseg, kBlock);
  hgnn_row_tasks* const t = p->tasks;
  if (grid > 0) {
    const auto write_kernel = mids ? plan_write_kernel<true> : plan_write_kernel<false>;
    write_kernel<<<dim3(unsigned(grid)), kBlock, 0, s>>>(
        tq, nblk, tc.count, tc.sums, t->sec, t->task, t->zrow, t->split, q, list_blocks, counts,
        RowListArrays{p->split_row, p->split_seg_lo, p->split_seg_hi, p->big_row, p->big_first, p->mid_row, p->hub_chunk_row,
                      p->hub_chunk_first, p->hub_chunk_count},
        p->nseg, p->seg_row_lo, p->seg_row_hi, ranges, range_blocks, tc.split_at, t->rtask, t->split + t->n_split);
    HGNN_LAUNCH_CHECK("plan_write_kernel");
  }
  const size_t nv = (size_t(g->nrows) + size_t(g->ncols)) * size_t(p->max_H);
  if (nv > 0) HGNN_HIP(dev_malloc(&p->vscratch, sizeof(float) * nv));
  if (g->nrows > 0) HGNN_HIP(dev_malloc(&p->vtab, sizeof(float) * 4 * size_t(g->nrows) * size_t(p->max_H)));
  HGNN_HIP(s.wait());
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

extern "C" {

const char* hgnn_status_str(hgnn_status s) {
  switch (s) {
    case HGNN_OK: return "HGNN_OK";
    case HGNN_EINVAL: return "HGNN_EINVAL: invalid argument";
    case HGNN_EUNSUPPORTED: return "HGNN_EUNSUPPORTED: shape not supported";
    case HGNN_ENOMEM: return "HGNN_ENOMEM: out of memory";
    case HGNN_EHIP: return "HGNN_EHIP: HIP runtime error";
  }
  return "unknown hgnn_status";
}

const char* hgnn_last_error(void) { return g_err; }

hgnn_status hgnn_plan_set_vector_halves(hgnn_plan* p, int32_t halves) {
  clear_error();
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "hgnn_plan_set_vector_halves: plan is NULL");
  HGNN_REQUIRE(halves == 2 || halves == 4 || halves == 8, HGNN_EINVAL, "hgnn_plan_set_vector_halves: %d is not 2, 4 or 8", halves);
  p->vec_halves = halves;
  if (p->fine) p->fine->vec_halves = halves;
  return HGNN_OK;
}

int32_t hgnn_plan_vector_halves(const hgnn_plan* p) { return p ? p->vec_halves : 0; }

hgnn_status hgnn_csr_validate(const hgnn_csr* g, void* stream) {
  clear_error();
  hgnn_status st = check_csr_args(g, "hgnn_csr_validate");
  if (st != HGNN_OK) return st;
  SetupStream s(stream);
  DevTemp facts(s);
  GraphFacts f;
  HGNN_HIP(facts.alloc(sizeof(GraphFacts)));
  hipError_t e = launch_validate(g, facts.as<GraphFacts>(), s);
  if (e == hipSuccess) e = hipMemcpyAsync(&f, facts.p, sizeof(f), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = s.wait();
  if (e != hipSuccess) return fail(HGNN_EHIP, "hgnn_csr_validate: %s", hipGetErrorString(e));
  return check_facts(f);
}

int64_t hgnn_plan_num_segments(const hgnn_plan* p) { return p ? p->nseg : 0; }
int32_t hgnn_plan_num_split_rows(const hgnn_plan* p) { return p ? p->n_split : 0; }
int32_t hgnn_plan_seg_edges(const hgnn_plan* p) { return p ? p->S : 0; }

int32_t hgnn_plan_col_blocks(const hgnn_plan* p) { return p ? p->nb : 0; }
int32_t hgnn_plan_col_blocks_fine(const hgnn_plan* p) { return p ? (p->fine ? p->fine->nb : p->nb) : 0; }

void hgnn_plan_cache_bytes(const hgnn_plan* p, int64_t* l2_bytes, int64_t* llc_bytes) {
  if (l2_bytes) *l2_bytes = p ? p->l2_bytes : 0;
  if (llc_bytes) *llc_bytes = p ? p->llc_bytes : 0;
}

}  // extern "C"

// idle: nothing that uses the plan is in flight
static void destroy_plan(hgnn_plan* p, bool idle) {
  if (!p) return;
  destroy_plan(p->fine, idle);
  destroy_tasks(p->tasks, idle);
  destroy_tasks(p->btasks, idle);
  dev_put(p->brp, idle);
  dev_put(p->bcol, idle);
  dev_put(p->bcol16, idle);
  dev_put(p->beid, idle);
  dev_put(p->bdelta, idle);
  dev_put(p->bstage, idle);
  dev_put(p->bsum, idle);
  dev_put(p->seg_row_lo, idle);
  dev_put(p->seg_row_hi, idle);
  dev_put(p->split_row, idle);
  dev_put(p->split_seg_lo, idle);
  dev_put(p->split_seg_hi, idle);
  dev_put(p->big_row, idle);
  dev_put(p->hub_chunk_row, idle);
  dev_put(p->hub_chunk_first, idle);
  dev_put(p->hub_chunk_count, idle);
  dev_put(p->big_first, idle);
  dev_put(p->hub_part, idle);
  dev_put(p->mid_row, idle);
  dev_put(p->vscratch, idle);
  dev_put(p->vtab, idle);
  dev_put(p->goff, idle);
  dev_put(p->moff, idle);
  dev_put(p->grp_row, idle);
  dev_put(p->gstage, idle);
  dev_put(p->scut, idle);
  dev_put(p->slice_share, idle);
  dev_put(p->col_part, idle);
  dev_put(p->col_poison, idle);
  delete p;
}

extern "C" {

void hgnn_plan_destroy(hgnn_plan* p) {
  if (!p) return;
  destroy_plan(p, device_idle(p->device));  // calls that use the plan may be in flight, and its memory is handed to the next plan
}

hgnn_status hgnn_plan_create(const hgnn_csr* g, int32_t seg_edges, int32_t max_F, int32_t max_H, int32_t col_blocks,
                             hgnn_plan** out, void* stream) {
  clear_error();
  HGNN_REQUIRE(out != nullptr, HGNN_EINVAL, "hgnn_plan_create: out is NULL");
  *out = nullptr;
  hgnn_status st = check_csr_args(g, "hgnn_plan_create");
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(seg_edges >= 1 && seg_edges <= 2048, HGNN_EINVAL, "hgnn_plan_create: seg_edges = %d outside [1, 2048]",
               seg_edges);
  HGNN_REQUIRE(max_F >= 8 && max_F % 8 == 0, HGNN_EINVAL, "hgnn_plan_create: max_F = %d must be a positive multiple of 8",
               max_F);
  HGNN_REQUIRE(max_H >= 1, HGNN_EINVAL, "hgnn_plan_create: max_H = %d must be positive", max_H);
  HGNN_REQUIRE(col_blocks >= 0 && col_blocks <= 64, HGNN_EINVAL, "hgnn_plan_create: col_blocks = %d outside [0, 64]",
               col_blocks);
  hgnn_plan* p = new (std::nothrow) hgnn_plan();
  HGNN_REQUIRE(p != nullptr, HGNN_ENOMEM, "hgnn_plan_create: host allocation failed");
  if (hipGetDevice(&p->device) != hipSuccess) {
    delete p;
    return fail(HGNN_EHIP, "hgnn_plan_create: no current device");
  }
  p->nrows = g->nrows;
  p->ncols = g->ncols;
  p->nnz = g->nnz;
  p->S = seg_edges;
  p->nseg = ceil_div(g->nnz, seg_edges);
  p->max_F = max_F;
  p->max_H = max_H;
  p->big_deg = 2048;
  p->mid_deg = 32;
  device_cache_bytes(&p->l2_bytes, &p->llc_bytes);
  SetupStream s(stream);
  int nb = col_blocks;
  bool narrow_only = false;  // every pass over blocks takes the finer cut
  p->auto_blocks = nb == 0;
  if (nb == 0) {
    // automatic: block only when the feature table is too large for an XCD's L2 (beyond three times its size)
    // but fits the last-level cache with room for the streams (three quarters of it), and rows are long enough
    // that a row piece per block still amortises its partial vector; about two L2 sizes of feature rows per block
    const double table = double(g->ncols) * max_F * 2.0;
    const double mean_deg = g->nrows > 0 ? double(g->nnz) / g->nrows : 0.0;
    nb = 1;
    if (table > 3.0 * double(p->l2_bytes) && table < 0.75 * double(p->llc_bytes) && mean_deg >= 128.0) {
      nb = int(table / (2.0 * double(p->l2_bytes)) + 0.5);
      if (nb < 2) nb = 2;
      if (nb > 16) nb = 16;
      // all passes walk the finer cut below where a row still has 32 non-zeros or more in each of its blocks on
      // average: slices of 3.7 MB come from L2 at 26 TB/s, of 7.5 MB at 15 TB/s, but every piece of a row costs a
      // partial row written and read again, as much as some ten gathers.  233 000 columns x 64, 4 -> 8 blocks: at 489
      // non-zeros a row 1.2 times as fast, at 172 slower (attention forward 524 -> 646 us, backward 552 -> 586).
      narrow_only = mean_deg >= 64.0 * nb && g->ncols >= 2 * nb;
    }
  }
  const bool blocks = nb > 1 && g->nnz > 0 && g->ncols >= nb;
  st = plan_build_arrays(p, g, blocks, s);
  if (st == HGNN_OK) {
    if (blocks) {
      p->nb = nb;
      p->block_width = int(ceil_div(g->ncols, nb));
      p->block_eid = g->eid != nullptr;
      if (!narrow_only) st = build_col_blocks(p, g, nb, s);
    }
    // A call that reads edge values through the edge-id map gathers from two tables at once: the feature rows of the
    // block's columns and, for each of those columns, the 128-byte line of the edge tensor that the walk is currently
    // passing (the slots of one source row are consecutive).  Both sets grow with the block's width, so such calls get
    // blocks of half the width.  So does the SDDMM, which leaves no partial row per block behind and only gains from
    // the narrower slice.
    if (st == HGNN_OK && p->auto_blocks && p->nb > 1 && g->ncols >= 2 * p->nb) {
      hgnn_plan* f = new (std::nothrow) hgnn_plan();
      if (f == nullptr) {
        st = fail(HGNN_ENOMEM, "hgnn_plan_create: host allocation failed");
      } else {
        p->fine = f;
        f->nrows = p->nrows;
        f->ncols = p->ncols;
        f->nnz = p->nnz;
        f->S = p->S;
        f->nseg = p->nseg;
        f->max_F = p->max_F;
        f->max_H = p->max_H;
        f->big_deg = p->big_deg;
        f->mid_deg = p->mid_deg;
        f->l2_bytes = p->l2_bytes;
        f->llc_bytes = p->llc_bytes;
        f->auto_blocks = true;
        st = build_col_blocks(f, g, 2 * p->nb, s);
      }
    }
    if (st == HGNN_OK && p->nb > 1 && !narrow_only) st = build_block_tasks(p, s);
    if (st == HGNN_OK && p->fine) st = build_block_tasks(p->fine, s);
    // column slices for the per-edge passes over per-vertex scalars: where a row's share of a slice still is a piece
    // of 16 non-zeros or more on average
    if (st == HGNN_OK && col_blocks == 0 && g->nrows > 0 && g->nnz > 0) {
      const int64_t ns = ceil_div(g->ncols, kSliceMaxCols);
      if (double(g->nnz) / g->nrows >= 16.0 * double(ns)) st = build_col_slices(p, g, kSliceMaxCols, false, s);
    }
  }
  if (st != HGNN_OK) {
    hgnn_plan_destroy(p);
    return st;
  }
  *out = p;
  return HGNN_OK;
}

hgnn_status hgnn_plan_export(const hgnn_plan* p, int32_t* seg_row_lo, int32_t* seg_row_hi, int32_t* split_row,
                             int32_t* split_seg_lo, int32_t* split_seg_hi) {
  clear_error();
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "hgnn_plan_export: plan is NULL");
  HGNN_HIP(hipDeviceSynchronize());
  if (p->nseg > 0) {
    if (seg_row_lo) HGNN_HIP(hipMemcpy(seg_row_lo, p->seg_row_lo, sizeof(int) * size_t(p->nseg), hipMemcpyDeviceToHost));
    if (seg_row_hi) HGNN_HIP(hipMemcpy(seg_row_hi, p->seg_row_hi, sizeof(int) * size_t(p->nseg), hipMemcpyDeviceToHost));
  }
  if (p->n_split > 0) {
    size_t b = sizeof(int) * size_t(p->n_split);
    if (split_row) HGNN_HIP(hipMemcpy(split_row, p->split_row, b, hipMemcpyDeviceToHost));
    if (split_seg_lo) HGNN_HIP(hipMemcpy(split_seg_lo, p->split_seg_lo, b, hipMemcpyDeviceToHost));
    if (split_seg_hi) HGNN_HIP(hipMemcpy(split_seg_hi, p->split_seg_hi, b, hipMemcpyDeviceToHost));
  }
  return HGNN_OK;
}

}  // extern "C"

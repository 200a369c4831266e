// The row tasks of a plan: every row of a graph (or of its column blocks) as one or more pieces of at most S non-zeros.
// Integer work only; set-up.
//
// Why pieces of rows and not equal runs of non-zeros: a lane group that stays inside one row needs no row id per non-zero,
// no row change in its loop and no merging of pieces with its neighbours.  A wave that walked 256 consecutive non-zeros
// spent about 850 vector instructions on 32 products per lane; with a row per lane group it is about 300.  What the equal
// runs gave for free, lane groups that end together, comes from sorting the rows of a window by length.
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "ranges.h"

namespace hgnn {

// counts[q][b][window]
template <bool MIDS>
__global__ __launch_bounds__(kTaskThreads) void task_count_kernel(TaskSource q, int nwin, int* __restrict__ counts) {
  __shared__ int total[kTaskCounters];
  const int b = blockIdx.y;
  const int* rp = q.rowptr + int64_t(b) * (int64_t(q.nrows) + 1);
  if (threadIdx.x < kTaskCounters) total[threadIdx.x] = 0;
  __syncthreads();
  int n[kTaskCounters] = {0, 0, 0, 0, 0};
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const int64_t r = int64_t(blockIdx.x) * kTaskWindow + u * kTaskThreads + threadIdx.x;
    if (r >= q.nrows) break;
    task_count_row<false, MIDS>(q, rp, int(r), n);
  }
  for (int i = 0; i < kTaskCounters; ++i) {
    int v = n[i];
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off);
    if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(&total[i], v);
  }
  __syncthreads();
  if (threadIdx.x < kTaskCounters) counts[(int64_t(threadIdx.x) * q.nb + b) * nwin + blockIdx.x] = task_counter<false, MIDS>(total, threadIdx.x);
}

__global__ __launch_bounds__(kTaskThreads) void task_scan_kernel(TaskSource q, int nwin, int* __restrict__ counts, int* __restrict__ sums,
                                                                  hgnn_task_sec* __restrict__ sec, TaskTotals* out) {
  task_scan(q, nwin, counts, sums, sec, out);
}

// Without a plan: exclusive scans of the counts of the windows in place, a workgroup for every array of them (n_first of those at `first`,
// the others at `second`), and their totals.
constexpr int kFreeScanThreads = 1024;
__global__ __launch_bounds__(kFreeScanThreads) void free_scan_kernel(int nwin, int* __restrict__ first, int n_first, int* __restrict__ second,
                                                                      int* __restrict__ sums) {
  __shared__ int s_wave[kFreeScanThreads / kWave];
  const int i = blockIdx.x, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int* const v = i < n_first ? first + int64_t(i) * nwin : second + int64_t(i - n_first) * nwin;
  const int per = (nwin + kFreeScanThreads - 1) / kFreeScanThreads, j0 = min(int(threadIdx.x) * per, nwin), j1 = min(j0 + per, nwin);
  int own = 0;
  for (int j = j0; j < j1; ++j) own += v[j];
  int incl = own;
  for (int d = 1; d < kWave; d <<= 1) {
    const int t = __shfl_up(incl, d);
    if (lane >= d) incl += t;
  }
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  int at = incl - own;
  for (int w = 0; w < wave; ++w) at += s_wave[w];
  if (threadIdx.x == kFreeScanThreads - 1) sums[i] = at + own;
  for (int j = j0; j < j1; ++j) {
    const int n = v[j];
    v[j] = at;
    at += n;
  }
}

template <bool SELF, bool MIDS>
__global__ __launch_bounds__(kTaskThreads) void task_write_kernel(TaskSource q, int nwin, const int* __restrict__ counts,
                                                                   const int* __restrict__ sums, hgnn_task_sec* __restrict__ sec,
                                                                   TaskTotals* __restrict__ totals, int4* __restrict__ task,
                                                                   int* __restrict__ zrow, int4* __restrict__ split) {
  task_write<SELF, false, MIDS>(q, blockIdx.x, blockIdx.y, nwin, counts, sums, sec, totals, task, zrow, split, 0);
}

// f(MIDS) for a launch
template <class F>
static void with_mids(const TaskSource& q, F&& f) {
  if (has_mids(q)) f(std::integral_constant<bool, true>());
  else f(std::integral_constant<bool, false>());
}

// room for the counts of q, which the caller's kernels or task_count form
hgnn_status task_prepare(const TaskSource& q, TaskCounts& c) {
  c.nwin = int(ceil_div(q.nrows, kTaskWindow));
  HGNN_HIP(c.counts.alloc(sizeof(int) * size_t(kTaskAll) * size_t(q.nb) * (size_t(c.nwin) + 1)));
  const size_t nsec = size_t(q.nb) + (q.range_min != kNoRanges ? 1 : 0);
  HGNN_HIP(c.secs.alloc(sizeof(hgnn_task_sec) * nsec + sizeof(TaskTotals) + sizeof(int)));
  c.count = c.counts.as<int>();
  c.sums = c.count + size_t(kTaskAll) * size_t(q.nb) * size_t(c.nwin);
  c.sec = c.secs.as<hgnn_task_sec>();
  c.split_at = c.count + size_t(kTaskSplit) * size_t(q.nb) * size_t(c.nwin);
  c.totals = c.mail.data ? reinterpret_cast<TaskTotals*>(c.mail.data) : reinterpret_cast<TaskTotals*>(c.sec + nsec);
  c.n_range = reinterpret_cast<int*>(c.totals + 1);
  return HGNN_OK;
}

static hgnn_status task_count(const TaskSource& q, TaskCounts& c, SetupStream& s) {  // without ranges
  const hgnn_status st = task_prepare(q, c);
  if (st != HGNN_OK) return st;
  if (c.nwin > 0) task_count_kernel<false><<<dim3(unsigned(c.nwin), unsigned(q.nb)), kTaskThreads, 0, s>>>(q, c.nwin, c.count);  // (of blocks)
  task_scan_kernel<<<1, kTaskThreads, 0, s>>>(q, c.nwin, c.count, c.sums, c.sec, c.totals);
  HGNN_LAUNCH_CHECK("task_count_kernel / task_scan_kernel");
  return HGNN_OK;
}

// After a wait for the counts: the arrays of the tasks, which task_write fills in afterwards.
hgnn_status task_allocate(const TaskSource& q, TaskCounts& c, int max_F, int max_H, hgnn_row_tasks** out) {
  hgnn_row_tasks* t = new (std::nothrow) hgnn_row_tasks();
  if (!t) return fail(HGNN_ENOMEM, "hgnn_plan_create: host allocation failed");
  *out = t;  // the plan owns it from here
  TaskTotals& tot = c.got;
  if (c.mail.data) {
    tot = *c.totals;
    if (c.ranges) tot.n_range = *c.n_range;
  } else {
    HGNN_HIP(hipMemcpy(&tot, c.totals, sizeof(tot), hipMemcpyDeviceToHost));
    if (c.ranges) HGNN_HIP(hipMemcpy(&tot.n_range, c.n_range, sizeof(int), hipMemcpyDeviceToHost));
  }
  if (tot.n_range > q.nnz / kRangeLeastMean) tot.n_range = 0;
  t->nb = q.nb;
  t->nnz = q.nnz;
  t->n_split = tot.n_split;
  t->n_slots = tot.n_slots;
  t->n_rtask = tot.n_range;
  t->stage_slots = std::max(t->n_slots, t->n_rtask);
  const int nsec = q.nb + (tot.n_range > 0 ? 1 : 0);
  t->host.resize(size_t(nsec));
  t->sec = c.sec;
  c.secs.p = nullptr;
  HGNN_HIP(dev_malloc(&t->task, sizeof(int4) * size_t(tot.n_task > 0 ? tot.n_task : 1)));
  HGNN_HIP(dev_malloc(&t->zrow, sizeof(int) * size_t(tot.n_zero > 0 ? tot.n_zero : 1)));
  if (t->n_split > 0) {
    HGNN_HIP(dev_malloc(&t->split, sizeof(int4) * size_t(t->n_split) * (tot.n_range > 0 ? 2 : 1)));
    HGNN_HIP(dev_malloc(&t->staging, sizeof(hgnn_half) * 2 * size_t(t->stage_slots) * size_t(max_F)));
    HGNN_HIP(dev_malloc(&t->stage_mz, sizeof(float) * 3 * size_t(t->stage_slots) * size_t(max_H)));
  }
  if (q.nb == 1) t->host[0] = hgnn_task_sec{0, tot.n_whole, tot.n_whole, tot.n_task - tot.n_whole, 0, int32_t(tot.n_zero), 0};
  if (tot.n_range > 0) {  // (one block)
    const int whole = tot.n_whole - tot.n_long_whole, group = tot.n_task - tot.n_whole - tot.n_long_group;
    t->host[1] = hgnn_task_sec{0, whole, tot.n_whole, group, 0, int32_t(tot.n_zero), 0};
    HGNN_HIP(dev_malloc(&t->rtask, sizeof(int4) * size_t(tot.n_range)));
  }
  return HGNN_OK;
}

// the tasks of plan p's column blocks
hgnn_status build_block_tasks(hgnn_plan* p, SetupStream& s) {
  DevTemp first(s);
  std::vector<int32_t> host(size_t(p->nb));
  for (int b = 0; b < p->nb; ++b) host[size_t(b)] = int32_t(p->boff[size_t(b)]);
  HGNN_HIP(first.alloc(sizeof(int32_t) * size_t(p->nb)));
  HGNN_HIP(hipMemcpyAsync(first.p, host.data(), sizeof(int32_t) * size_t(p->nb), hipMemcpyHostToDevice, s));
  const TaskSource q{p->brp, first.as<int32_t>(), p->nrows, p->nb, p->S, kGroupMaxBlocks, p->nnz, kNoRanges};
  TaskCounts c(s);
  hgnn_status st = task_count(q, c, s);
  if (st != HGNN_OK) return st;
  HGNN_HIP(s.wait());
  st = task_allocate(q, c, p->max_F, p->max_H, &p->btasks);
  if (st != HGNN_OK) return st;
  hgnn_row_tasks* t = p->btasks;
  HGNN_HIP(hipMemcpyAsync(t->host.data(), t->sec, sizeof(hgnn_task_sec) * size_t(q.nb), hipMemcpyDeviceToHost, s));
  if (c.nwin > 0)
    task_write_kernel<false, false><<<dim3(unsigned(c.nwin), unsigned(q.nb)), kTaskThreads, 0, s>>>(q, c.nwin, c.count, c.sums, t->sec, nullptr,
                                                                                            t->task, t->zrow, t->split);
  HGNN_LAUNCH_CHECK("task_write_kernel");
  HGNN_HIP(s.wait());
  p->btasks->col16 = p->bcol16;
  p->btasks->width = p->block_width;
  return HGNN_OK;
}

// A staged row for every so many non-zeros is room enough for power-law graphs (one for 150 to 200; log-normal rows of 120 on average 143).
// What a graph could have at most, eight pieces in rows of 257, is one for 29: 31 M non-zeros x 64 388 MB of workspace instead of 96.
constexpr int kFreeRangeMean = 128;

constexpr int64_t kSumsAt = 64;  // in the 256 bytes of the totals
static_assert(sizeof(TaskTotals) <= kSumsAt && kSumsAt + sizeof(int) * (kTaskAll + kRanges + 2) <= 256, "room");

TaskScratch task_scratch_at(void* base, int64_t nrows, int64_t nnz, int S, int F, int range_min) {
  // bounds from the sizes alone: a row of more than S non-zeros has at most len / S + 1 pieces, and there are fewer than
  // nnz / S such rows
  const int64_t nwin = ceil_div(nrows, kTaskWindow), over = nnz / S + 1;
  const bool ranges = range_min != kNoRanges;
  TaskScratch t{};
  char* const p = static_cast<char*>(base);
  int64_t at = 0;
  auto take = [&](int64_t bytes) {
    char* r = p ? p + at : nullptr;
    at += (bytes + 255) / 256 * 256;
    return r;
  };
  t.rows = ranges ? std::max(over, nnz / range_min + 1) : over;
  t.cap = ranges ? nnz / kFreeRangeMean : 0;
  t.sec = reinterpret_cast<hgnn_task_sec*>(take(sizeof(hgnn_task_sec)));
  t.totals = reinterpret_cast<TaskTotals*>(take(kSumsAt + sizeof(int) * (kTaskAll + kRanges + 2)));
  t.sums = t.totals ? reinterpret_cast<int32_t*>(reinterpret_cast<char*>(t.totals) + kSumsAt) : nullptr;
  t.counts = reinterpret_cast<int32_t*>(take(nwin * (ranges ? int(kTaskAll) + 1 : int(kTaskCounters)) * 4));
  t.task = reinterpret_cast<int4*>(take((nrows + over) * 16));
  t.zrow = reinterpret_cast<int32_t*>(take(nrows * 4));
  t.split = reinterpret_cast<int4*>(take(t.rows * 16));
  t.staging = reinterpret_cast<float*>(take(std::max(2 * over, t.cap) * int64_t((F + 7) & ~7) * 4));
  if (ranges) {
    t.rtask = reinterpret_cast<int4*>(take(t.cap * 16));
    t.range_lists = reinterpret_cast<int32_t*>(take(nwin * (kRanges + 1) * 4));
    t.cuts = reinterpret_cast<int32_t*>(take(int64_t(range_cut_bytes(nrows, nnz, range_min))));
  }
  t.bytes = size_t(at);
  return t;
}

// Without a plan and with column ranges: two launches, in each of which the workgroups for the long rows come first.  The second adds up the
// pieces at column ranges and leaves the long rows in ordinary pieces where they are more than there is room for.
template <bool MIDS>
__global__ __launch_bounds__(kTaskThreads) void free_count_kernel(TaskSource q, int nwin, int* __restrict__ counts, RangeLists ranges) {
  if (int(blockIdx.x) < nwin) {
    range_cut<kTaskThreads>(ranges, int(blockIdx.x));
    return;
  }
  __shared__ int total[kTaskAll];
  const int w = int(blockIdx.x) - nwin;
  if (threadIdx.x < kTaskAll) total[threadIdx.x] = 0;
  __syncthreads();
  int n[kTaskAll] = {};
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const int64_t r = int64_t(w) * kTaskWindow + u * kTaskThreads + threadIdx.x;
    if (r >= q.nrows) break;
    task_count_row<true, MIDS>(q, q.rowptr, int(r), n);
  }
#pragma unroll
  for (int i = 0; i < kTaskAll; ++i) {
    const int v = wave_sum(n[i]);
    if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(&total[i], v);
  }
  __syncthreads();
  if (threadIdx.x < kTaskAll) counts[int64_t(threadIdx.x) * nwin + w] = task_counter<true, MIDS>(total, threadIdx.x);
}

template <bool MIDS>
__global__ __launch_bounds__(kTaskThreads) void free_write_kernel(TaskSource q, int nwin, int range_cap, const int* __restrict__ counts,
                                                                  const int* __restrict__ sums,
                                                                  hgnn_task_sec* __restrict__ sec, TaskTotals* __restrict__ totals,
                                                                  int4* __restrict__ task, int* __restrict__ zrow, int4* __restrict__ split,
                                                                  RangeLists ranges, int range_blocks, int4* __restrict__ rtask) {
  const int b = int(blockIdx.x) - range_blocks;
  if (b >= 0) {
    task_write<true, true, MIDS>(q, b, 0, nwin, counts, sums, sec, totals, task, zrow, split, range_cap);
    return;
  }
  const int w = int(blockIdx.x) * kRangeGroup;
  int all[2];
  const RangePlace place = range_place(ranges, w, sums ? sums + kTaskAll : nullptr, all);
  if (all[0] > range_cap) return;
  if (all[1] > 0) range_write(ranges, w, place, rtask, split);
  if (w == 0 && threadIdx.x == 0) {
    totals->n_range = totals->n_slots = all[0];
    totals->n_split = all[1];
  }
}

// Up to so many windows every workgroup adds up the counts of all of them, beyond a launch scans them first: the additions grow with the square of
// the rows.  us a call, added up / scanned, in pieces and at column ranges: 0.4 M rows 99.3 / 99.0, 98.5 / 98.1; 0.7 M 174 / 173, 168 / 162;
// 1.5 M 238 / 235, 232 / 222; 2.4 M 638 / 628, 587 / 569; 10 M 1268 / 1203, 1366 / 1203; 20 M 1971 / 1736, 2365 / 1781; 0.2 M 57.7 / 58.5, 57.2 / 58.0.
constexpr int kFreeScanWindows = 400;
hgnn_status task_build_in(const TaskSource& q, const TaskScratch& t, const int32_t* col, int ncols, hipStream_t s) {
  const int nwin = int(ceil_div(q.nrows, kTaskWindow));
  int* const sums = nwin > kFreeScanWindows ? t.sums : nullptr;
  if (q.range_min == kNoRanges) {
    with_mids(q, [&](auto mids) {
      constexpr bool M = decltype(mids)::value;
      task_count_kernel<M><<<dim3(unsigned(nwin), 1u), kTaskThreads, 0, s>>>(q, nwin, t.counts);
      if (sums) free_scan_kernel<<<kTaskCounters, kFreeScanThreads, 0, s>>>(nwin, t.counts, kTaskCounters, nullptr, sums);
      task_write_kernel<true, M><<<dim3(unsigned(nwin), 1u), kTaskThreads, 0, s>>>(q, nwin, t.counts, sums, t.sec, t.totals, t.task, t.zrow, t.split);
    });
    HGNN_LAUNCH_CHECK("task_count_kernel / task_write_kernel");
    return HGNN_OK;
  }
  const int range_blocks = int(ceil_div(nwin, kRangeGroup));
  const RangeLists ranges = range_lists(q, col, ncols, nwin, t.cuts, t.range_lists, t.counts + int(kTaskAll) * int64_t(nwin),
                                        t.range_lists + kRanges * int64_t(nwin));
  with_mids(q, [&](auto mids) {
    constexpr bool M = decltype(mids)::value;
    free_count_kernel<M><<<dim3(unsigned(2 * nwin)), kTaskThreads, 0, s>>>(q, nwin, t.counts, ranges);
    if (sums) free_scan_kernel<<<kTaskAll + kRanges + 2, kFreeScanThreads, 0, s>>>(nwin, t.counts, kTaskAll + 1, t.range_lists, sums);
    free_write_kernel<M><<<dim3(unsigned(range_blocks + nwin)), kTaskThreads, 0, s>>>(q, nwin, int(t.cap), t.counts, sums, t.sec, t.totals, t.task, t.zrow,
                                                                                     t.split, ranges, range_blocks, t.rtask);
  });
  HGNN_LAUNCH_CHECK("free_count_kernel / free_write_kernel");
  return HGNN_OK;
}

void destroy_tasks(hgnn_row_tasks* t, bool idle) {
  if (!t) return;
  dev_put(t->task, idle);
  dev_put(t->zrow, idle);
  dev_put(t->rtask, idle);
  dev_put(t->split, idle);
  dev_put(t->sec, idle);
  dev_put(t->staging, idle);
  dev_put(t->stage_mz, idle);
  delete t;
}

}  // namespace hgnn

// The row tasks of a plan: every row of a graph (or of its column blocks) as one or more pieces of at most S non-zeros.
// Integer work only; set-up.
//
// Why pieces of rows and not equal runs of non-zeros: a lane group that stays inside one row needs no row id per non-zero,
// no row change in its loop and no merging of pieces with its neighbours.  A wave that walked 256 consecutive non-zeros
// spent about 850 vector instructions on 32 products per lane; with a row per lane group it is about 300.  What the equal
// runs gave for free, lane groups that end together, comes from sorting the rows of a window by length.
#include <string.h>

#include "common.h"

namespace hgnn {

constexpr int kTaskThreads = 256;
constexpr int kTaskRowsPerThread = kTaskWindow / kTaskThreads;
constexpr int kMaxGroupLen = 256;
static_assert(kGroupMaxBlocks <= kMaxGroupLen, "table of lengths");
enum { kTaskW, kTaskG, kTaskZ, kTaskSplit, kTaskSlots, kTaskCounters, kTaskLong = kTaskCounters, kTaskAll };  // kTaskLong: with a plan

constexpr int kLongRow = -1, kNone = -2;  // RowCut::m of a row for ranges.hip, and of no row

struct RowCut {
  int len, part, m;  // non-zeros, non-zeros per piece, pieces
};

__device__ __forceinline__ RowCut cut_row(const TaskSource& q, const int* rp, int r) {
  RowCut c;
  c.len = rp[r + 1] - rp[r];
  if (c.len < 0) c.len = 0;  // an offset array that validation will reject
  c.part = c.len;
  c.m = c.len > 0 ? 1 : 0;
  if (c.len >= q.range_min) {
    c.m = kLongRow;
  } else if (c.len > q.S) {
    c.part = pieces_of(c.len, pieces_of(c.len, q.S));
    c.m = pieces_of(c.len, c.part);
  }
  return c;
}

// counts[q][b][window]; RANGES: long rows are counted, too, and left out of the others
template <bool RANGES>
__global__ __launch_bounds__(kTaskThreads) void task_count_kernel(TaskSource q, int nwin, int* __restrict__ counts) {
  constexpr int counters = RANGES ? kTaskAll : kTaskCounters;
  __shared__ int total[kTaskAll];
  const int b = blockIdx.y;
  if (!RANGES) q.range_min = kNoRanges;
  const int* rp = q.rowptr + int64_t(b) * (int64_t(q.nrows) + 1);
  if (threadIdx.x < kTaskAll) total[threadIdx.x] = 0;
  __syncthreads();
  int n[kTaskAll] = {0, 0, 0, 0, 0, 0};
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const int64_t r = int64_t(blockIdx.x) * kTaskWindow + u * kTaskThreads + threadIdx.x;
    if (r >= q.nrows) break;
    const RowCut c = cut_row(q, rp, int(r));
    if (c.m == kLongRow) ++n[kTaskLong];
    else if (c.m == 0) ++n[kTaskZ];
    else n[c.part > q.group_max ? kTaskW : kTaskG] += c.m;
    if (c.m > 1) {
      ++n[kTaskSplit];
      n[kTaskSlots] += c.m;
    }
  }
  for (int i = 0; i < counters; ++i) {
    int v = n[i];
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off);
    if ((threadIdx.x & (kWave - 1)) == 0 && v) atomicAdd(&total[i], v);
  }
  __syncthreads();
  if (int(threadIdx.x) < counters) counts[(int64_t(threadIdx.x) * q.nb + b) * nwin + blockIdx.x] = total[threadIdx.x];
}

// One workgroup: exclusive scans over the windows of every (counter, block), then the sections of the blocks.  A wave per
// (counter, block).
__global__ __launch_bounds__(kTaskThreads) void task_scan_kernel(TaskSource q, int nwin, int* __restrict__ counts, int* __restrict__ sums,
                                                                  hgnn_task_sec* __restrict__ sec, TaskTotals* out) {
  const int nb = q.nb;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int counters = q.range_min == kNoRanges ? kTaskCounters : kTaskAll;
  for (int i = wave; i < counters * nb; i += kTaskThreads / kWave) {
    int* c = counts + int64_t(i) * nwin;
    int carry = 0;
    for (int w0 = 0; w0 < nwin; w0 += kWave) {
      const int v = w0 + lane < nwin ? c[w0 + lane] : 0;
      int incl = v;
      for (int d = 1; d < kWave; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
      }
      if (w0 + lane < nwin) c[w0 + lane] = carry + incl - v;
      carry += __shfl(incl, kWave - 1);
    }
    if (lane == 0) sums[i] = carry;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    TaskTotals t{};
    for (int b = 0; b < nb; ++b) {
      hgnn_task_sec s;
      s.nw = sums[kTaskW * nb + b];
      s.ng = sums[kTaskG * nb + b];
      s.nz = sums[kTaskZ * nb + b];
      s.w_off = t.n_task;
      s.g_off = t.n_task + s.nw;
      s.z_off = t.n_zero;
      s.first = q.first ? q.first[b] : 0;
      t.n_task += s.nw + s.ng;
      t.n_zero += s.nz;
      t.n_whole += s.nw;
      const int split = sums[kTaskSplit * nb + b], slots = sums[kTaskSlots * nb + b];
      sums[kTaskSplit * nb + b] = t.n_split;
      sums[kTaskSlots * nb + b] = t.n_slots;
      t.n_split += split;
      t.n_slots += slots;
      sec[b] = s;
    }
    if (counters == kTaskAll) t.n_long = sums[kTaskLong * nb];
    *out = t;
  }
}

// One workgroup per window and block: counting sort of the lane-group pieces by falling length.  The order of equal
// pieces depends on the order in which the LDS counters are reached; no result does.  SELF (one block): every workgroup adds
// up the counts of the windows before it, instead of a launch that scans them; the first leaves section and totals.
template <bool SELF>
__global__ __launch_bounds__(kTaskThreads) void task_write_kernel(TaskSource q, int nwin, const int* __restrict__ counts,
                                                                   const int* __restrict__ sums, hgnn_task_sec* __restrict__ sec,
                                                                   TaskTotals* __restrict__ totals, int4* __restrict__ task,
                                                                   int* __restrict__ zrow, int4* __restrict__ split) {
  __shared__ int at[kMaxGroupLen + 1];  // pieces of each length, then where the next one goes
  __shared__ int next[kTaskCounters];
  const int b = blockIdx.y, w = blockIdx.x;
  const int* rp = q.rowptr + int64_t(b) * (int64_t(q.nrows) + 1);
  __shared__ int before[kTaskCounters], all[kTaskCounters];
  hgnn_task_sec s;
  if (SELF) {
    q.range_min = kNoRanges;
    if (threadIdx.x < kTaskCounters) before[threadIdx.x] = all[threadIdx.x] = 0;
    __syncthreads();
    int b4[kTaskCounters] = {0, 0, 0, 0, 0}, sum[kTaskCounters] = {0, 0, 0, 0, 0};
    for (int j = threadIdx.x; j < nwin; j += kTaskThreads) {
#pragma unroll
      for (int i = 0; i < kTaskCounters; ++i) {
        const int n = counts[int64_t(i) * nwin + j];
        sum[i] += n;
        b4[i] += j < w ? n : 0;
      }
    }
#pragma unroll
    for (int i = 0; i < kTaskCounters; ++i) {
      for (int off = kWave / 2; off > 0; off >>= 1) {
        b4[i] += __shfl_down(b4[i], off);
        sum[i] += __shfl_down(sum[i], off);
      }
      if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&before[i], b4[i]);
        atomicAdd(&all[i], sum[i]);
      }
    }
    __syncthreads();
    s = hgnn_task_sec{0, all[kTaskW], all[kTaskW], all[kTaskG], 0, all[kTaskZ], 0};
    if (w == 0 && threadIdx.x == 0) {
      *sec = s;
      *totals = TaskTotals{all[kTaskZ], all[kTaskW] + all[kTaskG], all[kTaskW], all[kTaskSplit], all[kTaskSlots], 0, 0};
    }
  } else {
    s = sec[b];
  }
  for (int i = threadIdx.x; i <= kMaxGroupLen; i += kTaskThreads) at[i] = 0;
  if (threadIdx.x < kTaskCounters) {
    const int i = threadIdx.x;
    const int base = i == kTaskW ? s.w_off : i == kTaskG ? s.g_off : i == kTaskZ ? 0 : (SELF ? 0 : sums[i * q.nb + b]);
    next[i] = base + (SELF ? before[i] : counts[(int64_t(i) * q.nb + b) * nwin + w]);
  }
  __syncthreads();
  RowCut cut[kTaskRowsPerThread];
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const int64_t r = int64_t(w) * kTaskWindow + u * kTaskThreads + threadIdx.x;
    cut[u] = RowCut{0, 0, kNone};
    if (r < q.nrows) cut[u] = cut_row(q, rp, int(r));
    if (cut[u].m > 0 && cut[u].part <= q.group_max) {
      const int last = cut[u].len - (cut[u].m - 1) * cut[u].part;
      if (cut[u].m > 1) atomicAdd(&at[cut[u].part], cut[u].m - 1);
      atomicAdd(&at[last], 1);
    }
  }
  __syncthreads();
  if (threadIdx.x < kWave) {  // longest first
    int carry = next[kTaskG];
    for (int i0 = kMaxGroupLen; i0 >= 0; i0 -= kWave) {
      const int i = i0 - int(threadIdx.x);
      const int n = i >= 0 ? at[i] : 0;
      int incl = n;
      for (int d = 1; d < kWave; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (int(threadIdx.x) >= d) incl += t;
      }
      if (i >= 0) at[i] = carry + incl - n;
      carry += __shfl(incl, kWave - 1);
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const RowCut c = cut[u];
    const int r = w * kTaskWindow + u * kTaskThreads + int(threadIdx.x);
    int slot = -1, pos = 0, k0 = 0;
    if (c.m == 0) zrow[s.z_off + atomicAdd(&next[kTaskZ], 1)] = r;
    if (c.m > 1) {
      slot = atomicAdd(&next[kTaskSlots], c.m);
      split[atomicAdd(&next[kTaskSplit], 1)] = make_int4(r, slot, c.m, b);
    }
    const bool whole = c.part > q.group_max;
    if (c.m > 0) {
      if (whole) pos = atomicAdd(&next[kTaskW], c.m);
      k0 = s.first + rp[r];
    }
    auto piece = [&](int j, int k, int part, int m, int len, bool wh, int at_w, int row, int sl) {
      const int n = j + 1 < m ? part : len - j * part;
      const int p = wh ? at_w + j : atomicAdd(&at[n], 1);
      task[p] = make_int4(k + j * part, n | (b << 16), row, sl < 0 ? -1 : sl + j);
    };
    constexpr int kFew = 4;
    if (c.m <= kFew)
      for (int j = 0; j < c.m; ++j) piece(j, k0, c.part, c.m, c.len, whole, pos, r, slot);
    // a row of many pieces: the whole wave writes them (its own lane took 20 us for the longest row of a power-law graph)
    for (unsigned long long many = __ballot(c.m > kFew); many; many &= many - 1) {
      const int src = __ffsll((long long)many) - 1;
      const int m = __shfl(c.m, src), k = __shfl(k0, src), part = __shfl(c.part, src), len = __shfl(c.len, src);
      const int at_w = __shfl(pos, src), row = __shfl(r, src), sl = __shfl(slot, src);
      const bool wh = part > q.group_max;
      for (int j = lane; j < m; j += kWave) piece(j, k, part, m, len, wh, at_w, row, sl);
    }
  }
}

hgnn_status task_count(const TaskSource& q, TaskCounts& c, SetupStream& s) {
  const int nwin = int(ceil_div(q.nrows, kTaskWindow));
  HGNN_HIP(c.counts.alloc(sizeof(int) * size_t(kTaskAll) * size_t(q.nb) * (size_t(nwin) + 1)));
  HGNN_HIP(c.sec.alloc(sizeof(hgnn_task_sec) * size_t(q.nb) + sizeof(TaskTotals)));
  int* counts = c.counts.as<int>();
  int* sums = counts + size_t(kTaskAll) * size_t(q.nb) * size_t(nwin);
  hgnn_task_sec* sec = c.sec.as<hgnn_task_sec>();
  c.long_at = counts + size_t(kTaskLong) * size_t(q.nb) * size_t(nwin);
  c.n_long = sums + size_t(kTaskLong) * size_t(q.nb);
  c.totals = c.mail.data ? reinterpret_cast<TaskTotals*>(c.mail.data) : reinterpret_cast<TaskTotals*>(sec + q.nb);
  const dim3 grid(unsigned(nwin), unsigned(q.nb));
  if (nwin > 0 && q.range_min == kNoRanges) task_count_kernel<false><<<grid, kTaskThreads, 0, s>>>(q, nwin, counts);
  else if (nwin > 0) task_count_kernel<true><<<grid, kTaskThreads, 0, s>>>(q, nwin, counts);
  task_scan_kernel<<<1, kTaskThreads, 0, s>>>(q, nwin, counts, sums, sec, c.totals);
  HGNN_LAUNCH_CHECK("task_count_kernel / task_scan_kernel");
  return HGNN_OK;
}

// After a wait for the stream of task_count.  The arrays are written when the stream has been waited for again.
hgnn_status task_build(const TaskSource& q, TaskCounts& c, int max_F, int max_H, hgnn_row_tasks** out, SetupStream& s) {
  const int nwin = int(ceil_div(q.nrows, kTaskWindow));
  int* counts = c.counts.as<int>();
  int* sums = counts + size_t(kTaskAll) * size_t(q.nb) * size_t(nwin);
  hgnn_row_tasks* t = new (std::nothrow) hgnn_row_tasks();
  if (!t) return fail(HGNN_ENOMEM, "task_build: host allocation failed");
  *out = t;  // the plan owns it from here
  TaskTotals tot;
  if (c.mail.data) tot = *c.totals;
  else HGNN_HIP(hipMemcpy(&tot, c.totals, sizeof(tot), hipMemcpyDeviceToHost));
  t->nb = q.nb;
  t->nnz = q.nnz;
  t->n_split = tot.n_split + tot.n_long;
  t->n_slots = tot.n_slots + tot.n_range;
  t->n_rtask = tot.n_range;
  t->host.resize(size_t(q.nb));
  t->sec = c.sec.as<hgnn_task_sec>();
  c.sec.p = nullptr;
  HGNN_HIP(dev_malloc(&t->task, sizeof(int4) * size_t(tot.n_task > 0 ? tot.n_task : 1)));
  HGNN_HIP(dev_malloc(&t->zrow, sizeof(int) * size_t(tot.n_zero > 0 ? tot.n_zero : 1)));
  if (t->n_split > 0) {
    HGNN_HIP(dev_malloc(&t->split, sizeof(int4) * size_t(t->n_split)));
    HGNN_HIP(dev_malloc(&t->staging, sizeof(hgnn_half) * 2 * size_t(t->n_slots) * size_t(max_F)));
    HGNN_HIP(dev_malloc(&t->stage_mz, sizeof(float) * 3 * size_t(t->n_slots) * size_t(max_H)));
  }
  if (q.nb == 1) t->host[0] = hgnn_task_sec{0, tot.n_whole, tot.n_whole, tot.n_task - tot.n_whole, 0, int32_t(tot.n_zero), 0};
  else HGNN_HIP(hipMemcpyAsync(t->host.data(), t->sec, sizeof(hgnn_task_sec) * size_t(q.nb), hipMemcpyDeviceToHost, s));
  if (nwin > 0)
    task_write_kernel<false><<<dim3(unsigned(nwin), unsigned(q.nb)), kTaskThreads, 0, s>>>(q, nwin, counts, sums, t->sec, nullptr,
                                                                                          t->task, t->zrow, t->split);
  HGNN_LAUNCH_CHECK("task_write_kernel");
  if (tot.n_range > 0) {
    HGNN_HIP(dev_malloc(&t->rtask, sizeof(int4) * size_t(tot.n_range)));
    return range_write(q, c, tot, t->rtask, t->split + tot.n_split, s);
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
  st = task_build(q, c, p->max_F, p->max_H, &p->btasks, s);
  if (st != HGNN_OK) return st;
  HGNN_HIP(s.wait());
  p->btasks->col16 = p->bcol16;
  p->btasks->width = p->block_width;
  return HGNN_OK;
}

TaskScratch task_scratch_at(void* base, int64_t nrows, int64_t nnz, int S, int F) {
  // bounds from the sizes alone: a row of more than S non-zeros has at most len / S + 1 pieces, and there are fewer than
  // nnz / S such rows
  const int64_t nwin = ceil_div(nrows, kTaskWindow), over = nnz / S + 1;
  TaskScratch t{};
  char* const p = static_cast<char*>(base);
  int64_t at = 0;
  auto take = [&](int64_t bytes) {
    char* r = p ? p + at : nullptr;
    at += (bytes + 255) / 256 * 256;
    return r;
  };
  t.sec = reinterpret_cast<hgnn_task_sec*>(take(sizeof(hgnn_task_sec)));
  t.totals = reinterpret_cast<TaskTotals*>(take(sizeof(TaskTotals)));
  t.counts = reinterpret_cast<int32_t*>(take(nwin * kTaskCounters * 4));
  t.task = reinterpret_cast<int4*>(take((nrows + over) * 16));
  t.zrow = reinterpret_cast<int32_t*>(take(nrows * 4));
  t.split = reinterpret_cast<int4*>(take(over * 16));
  t.staging = reinterpret_cast<float*>(take(2 * over * int64_t((F + 7) & ~7) * 4));
  t.bytes = size_t(at);
  return t;
}

hgnn_status task_build_in(const TaskSource& q, const TaskScratch& t, hipStream_t s) {
  const int nwin = int(ceil_div(q.nrows, kTaskWindow));
  task_count_kernel<false><<<dim3(unsigned(nwin), 1u), kTaskThreads, 0, s>>>(q, nwin, t.counts);
  task_write_kernel<true><<<dim3(unsigned(nwin), 1u), kTaskThreads, 0, s>>>(q, nwin, t.counts, nullptr, t.sec, t.totals, t.task, t.zrow,
                                                                            t.split);
  HGNN_LAUNCH_CHECK("task_count_kernel / task_write_kernel");
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

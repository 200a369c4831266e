// Device side of the lists of row tasks (tasks.hip, plan.hip): a workgroup of kTaskThreads per window of kTaskWindow rows.
#pragma once

#include "common.h"

namespace hgnn {

constexpr int kTaskThreads = 256;
constexpr int kTaskRowsPerThread = kTaskWindow / kTaskThreads;
constexpr int kMaxGroupLen = 256;
static_assert(kGroupMaxBlocks <= kMaxGroupLen, "table of lengths");
enum { kTaskW, kTaskG, kTaskZ, kTaskSplit, kTaskSlots, kTaskCounters, kTaskLong = kTaskCounters, kTaskAll };  // kTaskLong: with a plan

constexpr int kLongRow = -1, kNone = -2;  // RowCut::m of a row for ranges.h, and of no row

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

// what row r adds to the counters
__device__ __forceinline__ void task_count_row(const TaskSource& q, const int* rp, int r, int (&n)[kTaskAll]) {
  const RowCut c = cut_row(q, rp, r);
  if (c.m == kLongRow) ++n[kTaskLong];
  else if (c.m == 0) ++n[kTaskZ];
  else n[c.part > q.group_max ? kTaskW : kTaskG] += c.m;
  if (c.m > 1) {
    ++n[kTaskSplit];
    n[kTaskSlots] += c.m;
  }
}

// One workgroup: exclusive scans over the windows of every (counter, block), then the sections of the blocks.  A wave per
// (counter, block).
__device__ __forceinline__ void task_scan(const TaskSource& q, int nwin, int* __restrict__ counts, int* __restrict__ sums,
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
__device__ __forceinline__ void task_write(TaskSource q, int w, int b, int nwin, const int* __restrict__ counts, const int* __restrict__ sums,
                                           hgnn_task_sec* __restrict__ sec, TaskTotals* __restrict__ totals, int4* __restrict__ task,
                                           int* __restrict__ zrow, int4* __restrict__ split) {
  __shared__ int at[kMaxGroupLen + 1];  // pieces of each length, then where the next one goes
  __shared__ int next[kTaskCounters];
  const int* rp = q.rowptr + int64_t(b) * (int64_t(q.nrows) + 1);
  __shared__ int before[kTaskCounters], all[kTaskCounters];
  hgnn_task_sec s;
  if (SELF) {
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

}  // namespace hgnn

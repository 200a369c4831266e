// Device side of the lists of row tasks (tasks.hip, plan.hip): a workgroup of kTaskThreads per window of kTaskWindow rows.
#pragma once

#include "common.h"

namespace hgnn {

constexpr int kTaskThreads = 256;
constexpr int kTaskRowsPerThread = kTaskWindow / kTaskThreads;
constexpr int kMaxGroupLen = 256;
static_assert(kGroupMaxBlocks <= kMaxGroupLen, "table of lengths");
// kTaskLongW, kTaskLongG: W and G of the rows from range_min on, which have a part of the lists to themselves
enum { kTaskW, kTaskG, kTaskZ, kTaskSplit, kTaskSlots, kTaskCounters, kTaskLongW = kTaskCounters, kTaskLongG, kTaskAll };

constexpr int kNone = -1;  // RowCut::m of no row

struct RowCut {
  int len, part, m;  // non-zeros, non-zeros per piece, pieces
  bool far;          // cut at column ranges, too
};

// RANGES: there may be rows from q.range_min on
template <bool RANGES>
__device__ __forceinline__ RowCut cut_row(const TaskSource& q, const int* rp, int r) {
  RowCut c;
  c.len = rp[r + 1] - rp[r];
  if (c.len < 0) c.len = 0;  // an offset array that validation will reject
  c.part = c.len;
  c.m = c.len > 0 ? 1 : 0;
  c.far = RANGES && q.range_min != kNoRanges && c.len >= q.range_min;
  if (c.len > q.S) {
    c.part = pieces_of(c.len, pieces_of(c.len, q.S));
    c.m = pieces_of(c.len, c.part);
  }
  return c;
}

// Rows of one piece just above group_max, up to kMidLen: a window (kTaskWindow rows) leaves them to lane groups, too, where that takes most of its
// waves away.  They are counted beside its empty rows, of which there are no more than 65535.  A wave of its own is mostly overhead there, which
// counts where there are many; else it is the shorter chain.  us, waves / lane groups: uniform, 2 M non-zeros of 42 233 rows x 64, SpMM 28.0 / 20.9, SDDMM
// 33.0 / 24.5, attention forward 57.8 / 31.9, backward 57.7 / 46.6; of 62 500 rows (32 on average) 28.6 / 29.5, 32.1 / 31.1, 57.9 / 45.2, 61.8 / 58.0; of 33 333
// (60) 20.6 / 18.3, 24.1 / 21.2, 40.1 / 30.5, 41.0 / 37.7; 400 000 of 8000 7.3 / 6.4, 8.2 / 7.7, 11.2 / 10.0; of 6667 6.6 / 7.2, 7.1 / 8.3, 10.6 / 11.0; 160 000 of
// 4000 5.6 / 5.8, 6.6 / 7.3, 10.5 / 10.7, 12.6 / 13.7.  All rows up to 64 of a power law of 1.5 M of 30 000: 17.8 / 19.4, 16.7 / 19.4, 36.0 / 39.1, 36.1 / 39.7;
// log-normal, 1.7 M of 60 328: 27.3 / 28.6, 27.5 / 28.7, 45.2 / 41.7, 50.6 / 47.7.  What loses: row sums behind a map of the first 24.7 / 26.3, with four
// heads of the mean 60 22.4 / 29.8.
// In the order of the degrees other graphs have such windows, too.  With a plan they keep to waves unless the graph has kMidLeastRows of the rows
// (power law, 1.5 M of 30 000, SpMM x 16 12.6 / 14.4, SDDMM 11.1 / 13.6; log-normal, 1.7 M of 60 328, saving attention 40.2 / 33.7, SDDMM x 64 24.6 / 22.4).  Without
// one they do not ask (uniform, 400 000 of 6667 29.0 / 24.2; of what is in the order of its degrees only 1.7 M log-normal 50.9 / 57.2 and 5.5 M power law x 16
// through the map 130 / 152 are slower).
// MIDS: the graph may have them (has_mids), as a template because the smallest plan-free calls are a chain of latencies (9000 non-zeros, never / asked
// in the kernels / as a template 15.0 / 15.9 / 15.0).
constexpr int kMidLen = 64, kMidShift = 16;
constexpr int64_t kMidLeastNnz = int64_t(1) << 18, kMidLeastRows = 7000;
inline bool has_mids(const TaskSource& q) { return q.nnz >= kMidLeastNnz && q.group_max < kMidLen; }
template <bool MIDS>
__device__ __forceinline__ bool mid_row(const TaskSource& q, const RowCut& c) {
  return MIDS && c.m == 1 && c.part > q.group_max && c.part <= kMidLen && !c.far;
}
// above 0: so many rows, and pieces of lane groups and of waves beside them, take less than half the waves with the rows in lane
// groups, eight to a wave.  A sum over rows, of fewer than 2^27 (group_max is 32 up to 8 M non-zeros only).
__device__ __forceinline__ int mid_gain(int mid, int group, int whole) { return 6 * mid - group - 8 * whole; }

// About how many of a graph's rows are such: of one for every thread of the workgroup, at equal distances, in two steps (they are asked for ahead of the
// window's own).
template <bool MIDS>
struct MidSample {
  bool mid = false;
  __device__ __forceinline__ MidSample(const TaskSource& q) {
    const int64_t r = int64_t(q.nrows) * (2 * int(threadIdx.x) + 1) / (2 * kTaskThreads);
    if (MIDS && r < q.nrows) mid = mid_row<MIDS>(q, cut_row<true>(q, q.rowptr, int(r)));
  }
  __device__ __forceinline__ void add(int* sum) const {  // to a word of LDS
    if (!MIDS) return;
    const int n = __popcll(__ballot(mid));
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(sum, n);
  }
  static __device__ __forceinline__ bool many(const TaskSource& q, int sum) { return int64_t(sum) * q.nrows >= kMidLeastRows * kTaskThreads; }
};

// the counters of a window from what its rows have added to them (the same rows whether long ones are cut at column ranges or not); may: whether its
// middle rows may go to lane groups
template <bool RANGES, bool MIDS>
__device__ __forceinline__ int task_counter(const int* total, int i, bool may = true) {
  if (!MIDS) return total[i];
  const int mid = total[kTaskZ] >> kMidShift;
  if (i == kTaskZ) return total[kTaskZ] & ((1 << kMidShift) - 1);
  if (i != kTaskW && i != kTaskG) return total[i];
  const int group = total[kTaskG] + (RANGES ? total[kTaskLongG] : 0), whole = total[kTaskW] + (RANGES ? total[kTaskLongW] : 0);
  return total[i] + ((may && mid_gain(mid, group, whole) > 0) == (i == kTaskG) ? mid : 0);
}

// what row r adds to the counters
template <bool RANGES, bool MIDS, int N>
__device__ __forceinline__ void task_count_row(const TaskSource& q, const int* rp, int r, int (&n)[N]) {
  static_assert(N == (RANGES ? kTaskAll : kTaskCounters), "counters");
  const RowCut c = cut_row<RANGES>(q, rp, r);
  const bool whole = c.part > q.group_max;
  if (c.m == 0) {
    ++n[kTaskZ];
  } else if (mid_row<MIDS>(q, c)) {
    n[kTaskZ] += 1 << kMidShift;
  } else if (RANGES && c.far) {
    n[whole ? int(kTaskLongW) : int(kTaskLongG)] += c.m;
  } else {
    n[whole ? kTaskW : kTaskG] += c.m;
  }
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
      if (counters == kTaskAll) {  // (one block) the short rows alone, then all
        t.n_long_whole = sums[kTaskLongW];
        t.n_long_group = sums[kTaskLongG];
        sec[1] = hgnn_task_sec{0, s.nw, s.nw + t.n_long_whole, s.ng, 0, sums[kTaskZ], 0};
        s.nw += t.n_long_whole;
        s.ng += t.n_long_group;
      }
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
    *out = t;
  }
}

// One workgroup per window and block: counting sort of the lane-group pieces by falling length.  The order of equal
// pieces depends on the order in which the LDS counters are reached; no result does.  SELF (one block): every workgroup adds
// up the counts of the windows before it, unless a launch has scanned them (then sums are their totals); the first leaves section and totals.  Pieces of rows from
// q.range_min on follow those of the others.  With both they are left out if no more than range_cap pieces take their place, whose number
// of every window follows the counters.
template <bool SELF, bool RANGES, bool MIDS>
__device__ __forceinline__ void task_write(TaskSource q, int w, int b, int nwin, const int* __restrict__ counts, const int* __restrict__ sums,
                                           hgnn_task_sec* __restrict__ sec, TaskTotals* __restrict__ totals, int4* __restrict__ task,
                                           int* __restrict__ zrow, int4* __restrict__ split, int range_cap) {
  constexpr int kLists = RANGES ? 2 : 1, kNext = RANGES ? int(kTaskAll) : int(kTaskCounters), kAdd = kNext + (RANGES ? 1 : 0);
  __shared__ int at[kLists][kMaxGroupLen + 1];  // pieces of each length, then where the next one goes; [1]: of rows from range_min on
  __shared__ int next[kNext];
  const int* rp = q.rowptr + int64_t(b) * (int64_t(q.nrows) + 1);
  __shared__ int before[kAdd], all[kAdd];
  hgnn_task_sec s;
  bool drop = false;
  if (SELF) {
    if (threadIdx.x < kAdd) {
      before[threadIdx.x] = sums ? counts[int64_t(threadIdx.x) * nwin + w] : 0;
      all[threadIdx.x] = sums ? sums[threadIdx.x] : 0;
    }
    __syncthreads();
    if (!sums) {
      int b4[kAdd] = {}, sum[kAdd] = {};
      for (int j = threadIdx.x; j < nwin; j += kTaskThreads) {
#pragma unroll
        for (int i = 0; i < kAdd; ++i) {
          const int n = counts[int64_t(i) * nwin + j];
          sum[i] += n;
          b4[i] += j < w ? n : 0;
        }
      }
#pragma unroll
      for (int i = 0; i < kAdd; ++i) {
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
    }
    int nw = all[kTaskW], ng = all[kTaskG];
    if constexpr (RANGES) {
      drop = all[kTaskAll] <= range_cap;
      if (!drop) {
        nw += all[kTaskLongW];
        ng += all[kTaskLongG];
      }
    }
    s = hgnn_task_sec{0, nw, nw, ng, 0, all[kTaskZ], 0};
    if (w == 0 && threadIdx.x == 0) {
      *sec = s;
      totals->n_zero = all[kTaskZ];
      totals->n_task = nw + ng;
      totals->n_whole = nw;
      if (!drop) {
        totals->n_split = all[kTaskSplit];
        totals->n_slots = all[kTaskSlots];
        totals->n_range = 0;
      }
    }
  } else {
    s = sec[b];
  }
  RowCut cut[kTaskRowsPerThread];
  auto read_rows = [&] {
    for (int u = 0; u < kTaskRowsPerThread; ++u) {
      const int64_t r = int64_t(w) * kTaskWindow + u * kTaskThreads + threadIdx.x;
      cut[u] = RowCut{0, 0, kNone, false};
      if (r < q.nrows) cut[u] = cut_row<RANGES>(q, rp, int(r));
    }
  };
  // Middle rows are in lane groups where the window's count of waves says so; the rows are then read ahead of the barrier that the counters want
  // anyway.
  __shared__ int s_waves[kTaskThreads / kWave], s_counted;
  if (MIDS) {
    read_rows();
    int waves = 0;  // without middle rows and those from range_min on
    for (int u = 0; u < kTaskRowsPerThread; ++u) {
      const RowCut& c = cut[u];
      if (c.m > 0 && c.part > q.group_max && !c.far && !mid_row<MIDS>(q, c)) waves += c.m;
    }
    waves = wave_sum(waves);
    if ((threadIdx.x & (kWave - 1)) == 0) s_waves[threadIdx.x / kWave] = waves;
    if (threadIdx.x == 0) {
      const int* const c = counts + (int64_t(kTaskW) * q.nb + b) * nwin + w;
      if (SELF && !sums) s_counted = *c;
      else s_counted = (w + 1 < nwin ? c[1] : sums[kTaskW * q.nb + b]) - *c;
    }
  }
  for (int i = threadIdx.x; i < kLists * (kMaxGroupLen + 1); i += kTaskThreads) at[0][i] = 0;
  if (threadIdx.x < (RANGES && q.range_min != kNoRanges ? int(kTaskAll) : int(kTaskCounters))) {
    const int i = threadIdx.x;
    int base = i == kTaskW ? s.w_off : i == kTaskG ? s.g_off : i == kTaskZ ? 0 : (SELF ? 0 : sums[i * q.nb + b]);
    if (RANGES && i == kTaskLongW) base = s.w_off + (SELF ? all[kTaskW] : sums[kTaskW]);  // (one block)
    if (RANGES && i == kTaskLongG) base = s.g_off + (SELF ? all[kTaskG] : sums[kTaskG]);
    next[i] = base + (SELF ? before[i] : counts[(int64_t(i) * q.nb + b) * nwin + w]);
  }
  __syncthreads();
  bool grouped = false;
  if (MIDS) {
    int waves = 0;
    for (int i = 0; i < kTaskThreads / kWave; ++i) waves += s_waves[i];
    grouped = s_counted == waves;
  } else {
    read_rows();
  }
  if (RANGES && drop)
    for (int u = 0; u < kTaskRowsPerThread; ++u)
      if (cut[u].far) cut[u].m = kNone;
  auto is_whole = [&](const RowCut& c) { return c.part > q.group_max && !(MIDS && grouped && mid_row<MIDS>(q, c)); };
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    if (cut[u].m > 0 && !is_whole(cut[u])) {
      int* const a = at[RANGES && cut[u].far ? 1 : 0];
      const int last = cut[u].len - (cut[u].m - 1) * cut[u].part;
      if (cut[u].m > 1) atomicAdd(&a[cut[u].part], cut[u].m - 1);
      atomicAdd(&a[last], 1);
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  if (threadIdx.x < kLists * kWave) {  // longest first
    const int y = threadIdx.x / kWave;
    int carry = next[RANGES && y ? int(kTaskLongG) : int(kTaskG)];
    for (int i0 = kMaxGroupLen; i0 >= 0; i0 -= kWave) {
      const int i = i0 - lane;
      const int n = i >= 0 ? at[y][i] : 0;
      int incl = n;
      for (int d = 1; d < kWave; d <<= 1) {
        const int t = __shfl_up(incl, d);
        if (lane >= d) incl += t;
      }
      if (i >= 0) at[y][i] = carry + incl - n;
      carry += __shfl(incl, kWave - 1);
    }
  }
  __syncthreads();
  for (int u = 0; u < kTaskRowsPerThread; ++u) {
    const RowCut c = cut[u];
    const int r = w * kTaskWindow + u * kTaskThreads + int(threadIdx.x);
    int slot = -1, pos = 0, k0 = 0;
    if (c.m == 0) zrow[s.z_off + atomicAdd(&next[kTaskZ], 1)] = r;
    if (c.m > 1) {
      slot = atomicAdd(&next[kTaskSlots], c.m);
      split[atomicAdd(&next[kTaskSplit], 1)] = make_int4(r, slot, c.m, b);
    }
    const bool whole = is_whole(c);
    if (c.m > 0) {
      if (whole) pos = atomicAdd(&next[RANGES && c.far ? int(kTaskLongW) : int(kTaskW)], c.m);
      k0 = s.first + rp[r];
    }
    auto piece = [&](int j, int k, int part, int m, int len, bool wh, bool far, int at_w, int row, int sl) {
      const int n = j + 1 < m ? part : len - j * part;
      const int p = wh ? at_w + j : atomicAdd(&at[RANGES && far ? 1 : 0][n], 1);
      task[p] = make_int4(k + j * part, n | (b << 16), row, sl < 0 ? -1 : sl + j);
    };
    constexpr int kFew = 4;
    if (c.m <= kFew)
      for (int j = 0; j < c.m; ++j) piece(j, k0, c.part, c.m, c.len, whole, c.far, pos, r, slot);
    // a row of many pieces: the whole wave writes them (its own lane took 20 us for the longest row of a power-law graph)
    for (unsigned long long many = __ballot(c.m > kFew); many; many &= many - 1) {
      const int src = __ffsll((long long)many) - 1;
      const int m = __shfl(c.m, src), k = __shfl(k0, src), part = __shfl(c.part, src), len = __shfl(c.len, src);
      const int at_w = __shfl(pos, src), row = __shfl(r, src), sl = __shfl(slot, src);
      const bool wh = part > q.group_max, far = RANGES && __shfl(int(c.far), src);
      for (int j = lane; j < m; j += kWave) piece(j, k, part, m, len, wh, far, at_w, row, sl);
    }
  }
}

}  // namespace hgnn

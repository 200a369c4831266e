// Long rows of a graph whose feature table misses the L2s, cut at the borders of column ranges.  Integer work only; set-up.
//
// Eight L2s of 4 MB keep the popular rows of a large table eight times over when every XCD gathers from all of it.  Columns ascend
// inside a row, so a row's share of a column range is a run of its non-zeros, and a run is a piece of the row like any other (task.h):
// nothing is copied or re-ordered.  The pieces are listed range after range and an eighth of the list goes to each XCD, whose L2 then
// sees an eighth of the columns.  What it costs is a staged partial row per (row, range), so only rows that have several pieces anyway
// are cut; on a power law they hold most of the non-zeros (62 M x 128: L2 hits 31 -> 49 %, misses 11.9 -> 8.9 GB a call).
#pragma once

#include "task_build.h"

namespace hgnn {

constexpr int kRanges = 8;        // as many as there are XCDs
constexpr int kRangeGroup = 4;    // windows of kTaskWindow rows whose pieces are sorted by length together (1, 2, 4: 5.5 M non-zeros x 4
                                  // heads, attention forward 110, 103, 102 us, SDDMM 62.5, 59.8, 58.6; a plan 76, 79, 82)
constexpr int kRangePiece = 256;  // most non-zeros of a piece (also at most S)
// Fewest non-zeros of a piece on average, for the memory: two partial rows are staged for each in a plan.  Graphs with small S would
// gain below it, too: 5 M non-zeros in rows of 50, F = 128, S = 32, 6 to a piece: SpMM 172 / 152 us, staging 106 / 417 MB.
constexpr int kRangeLeastMean = 8;

// Every window of kTaskWindow rows cuts its own long rows; the pieces of a window and range are sorted by length together.
struct RangeLists {
  const int* rowptr;
  const int* col;
  int* cuts;   // [range_cut_rows][kRanges - 1] where a long row's share of the ranges from the second on begins
  int* count;  // [kRanges][nwin] pieces, then where they go
  int* slots;  // [nwin] pieces of a window's rows, then the first of them
  int* long_rows;  // [nwin] long rows of a window, or nullptr (a plan has their number from its other counts)
  int nrows, nwin, piece, min_row, width;
  int shift;  // where a row's cuts are: a place for every row (-1), or for every 2^shift <= min_row non-zeros (no two long rows share one)
  __device__ __forceinline__ int* cuts_of(int row, int beg) const { return cuts + int64_t(shift < 0 ? row : beg >> shift) * (kRanges - 1); }
};

static int range_cut_shift(int min_row) {
  int s = 0;
  while (min_row >> (s + 1)) ++s;
  return s;
}
static int64_t range_cut_rows(int64_t nrows, int64_t nnz, int min_row) {
  const int64_t places = (nnz >> range_cut_shift(min_row)) + 1;
  return nrows < places ? nrows : places;
}
static size_t range_cut_bytes(int64_t nrows, int64_t nnz, int min_row) {
  return sizeof(int) * (kRanges - 1) * size_t(range_cut_rows(nrows, nnz, min_row));
}

static RangeLists range_lists(const TaskSource& q, const int* col, int ncols, int nwin, int* cuts, int* count, int* slots, int* long_rows) {
  RangeLists a{};
  a.rowptr = q.rowptr;
  a.col = col;
  a.nrows = q.nrows;
  a.nwin = nwin;
  a.piece = q.S < kRangePiece ? q.S : kRangePiece;
  a.min_row = q.range_min;
  a.width = int(ceil_div(ncols, kRanges));
  a.shift = range_cut_rows(q.nrows, q.nnz, q.range_min) == q.nrows ? -1 : range_cut_shift(q.range_min);
  a.cuts = cuts;
  a.count = count;
  a.slots = slots;
  a.long_rows = long_rows;
  return a;
}

struct RangeShare {
  int beg, len, part, m;  // first non-zero, non-zeros, non-zeros per piece, pieces
};
__device__ __forceinline__ RangeShare range_share(int piece, int beg, int end) {
  RangeShare s{beg, end - beg, 0, 0};
  if (s.len > piece) {  // few: three divisions for everyone were 40 us of a plan of 5.5 M non-zeros
    s.part = pieces_of(s.len, pieces_of(s.len, piece));
    s.m = pieces_of(s.len, s.part);
  } else if (s.len > 0) {  // (columns that validation will reject can lead to less)
    s.part = s.len;
    s.m = 1;
  }
  return s;
}
// the share of range x of long row r, whose cuts are there
__device__ __forceinline__ RangeShare range_share_of(const RangeLists& a, int r, int x) {
  const int beg = a.rowptr[r], end = a.rowptr[r + 1];
  const int* c = a.cuts_of(r, beg);
  return range_share(a.piece, x == 0 ? beg : c[x - 1], x == kRanges - 1 ? end : c[x]);
}

// Window w by a workgroup of THREADS: a lane per (long row, range), the first non-zero of the range by binary search; its end is where
// the next lane's begins.  Columns may be in any order: searches for rising values in the same array part where a middle element is
// below one value and not the other, the former ends behind it and the latter at or before it, so the cuts ascend and every non-zero
// is in one piece whatever the array holds.
template <int THREADS>
__device__ __forceinline__ void range_cut(const RangeLists& a, int w) {
  __shared__ int s_row[kTaskWindow], s_n, s_count[kRanges];
  if (threadIdx.x == 0) s_n = 0;
  if (threadIdx.x < kRanges) s_count[threadIdx.x] = 0;
  __syncthreads();
  for (int u = 0; u < kTaskWindow; u += THREADS) {
    const int64_t r = int64_t(w) * kTaskWindow + u + threadIdx.x;
    if (r < a.nrows && a.rowptr[r + 1] - a.rowptr[r] >= a.min_row) s_row[atomicAdd(&s_n, 1)] = int(r);
  }
  __syncthreads();
  const int n = s_n, x = threadIdx.x % kRanges;
  for (int i0 = 0; i0 < n; i0 += THREADS / kRanges) {  // uniform: lanes exchange
    const int i = i0 + int(threadIdx.x) / kRanges;
    const bool ok = i < n;
    const int row = ok ? s_row[i] : 0;
    const int beg = ok ? a.rowptr[row] : 0, end = ok ? a.rowptr[row + 1] : 0;
    pos_t lo = pos_t(beg), hi = pos_t(end);
    if (x > 0) {
      const int64_t first = int64_t(x) * a.width;
      while (lo < hi) {
        const pos_t mid = (lo + hi) / 2;
        if (a.col[mid] < first) lo = mid + 1;
        else hi = mid;
      }
      if (ok) a.cuts_of(row, beg)[x - 1] = int(lo);
    }
    const int next = __shfl_down(int(lo), 1, kRanges);
    const int m = range_share(a.piece, int(lo), x == kRanges - 1 ? end : next).m;
    if (ok && m) atomicAdd(&s_count[x], m);
  }
  __syncthreads();
  if (threadIdx.x < kRanges) a.count[int(threadIdx.x) * a.nwin + w] = s_count[threadIdx.x];
  if (threadIdx.x == 0) {
    int all = 0;
    for (int j = 0; j < kRanges; ++j) all += s_count[j];
    a.slots[w] = all;
    if (a.long_rows) a.long_rows[w] = n;
  }
}

// inclusive scan over the workgroup of kTaskThreads of one value per thread; *total on all threads
__device__ __forceinline__ int range_scan(int v, int* s_wave, int* total) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int incl = v;
  for (int d = 1; d < kWave; d <<= 1) {
    const int t = __shfl_up(incl, d);
    if (lane >= d) incl += t;
  }
  __syncthreads();  // what a previous scan left has been read
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  int before = 0, all = 0;
  for (int w = 0; w < kTaskThreads / kWave; ++w) {
    if (w < wave) before += s_wave[w];
    all += s_wave[w];
  }
  *total = all;
  return before + incl;
}

// one workgroup of kTaskThreads: exclusive scans in place; all pieces
__device__ __forceinline__ int range_scan_all(const RangeLists& a) {
  __shared__ int s_wave[kTaskThreads / kWave];
  auto scan = [&](int* v, int n) {
    int carry = 0;
    for (int i0 = 0; i0 < n; i0 += kTaskThreads) {
      const int i = i0 + int(threadIdx.x), x = i < n ? v[i] : 0;
      int total;
      const int incl = range_scan(x, s_wave, &total);
      if (i < n) v[i] = carry + incl - x;
      carry += total;
    }
    return carry;
  };
  (void)scan(a.slots, a.nwin);
  return scan(a.count, kRanges * a.nwin);
}

// Where a group of windows puts its pieces and rows.
struct RangePlace {
  int task[kRanges];  // the first piece of every range
  int slot, split;    // the first staging slot and the first entry of the rows of several pieces
};

// the same without a plan: what the windows before w hold, and in *all (pieces, long rows) what all of them do.  Unless a launch has scanned
// the counts (then sums are the totals of slots, counts and long rows), the workgroup adds them up.
__device__ __forceinline__ RangePlace range_place(const RangeLists& a, int w, const int* __restrict__ sums, int* all) {
  constexpr int kSums = kRanges + 2;  // pieces of every range, pieces, long rows
  __shared__ int s_before[kSums], s_all[kSums];
  if (threadIdx.x < kSums) s_before[threadIdx.x] = s_all[threadIdx.x] = 0;
  __syncthreads();
  if (sums && threadIdx.x < kSums) {
    const int i = threadIdx.x;
    const int* v = i < kRanges ? a.count + i * a.nwin : (i == kRanges ? a.slots : a.long_rows);
    s_before[i] = v[w];
    s_all[i] = sums[i < kRanges ? i + 1 : (i == kRanges ? 0 : i)];
  }
  for (int i = sums ? -1 : kSums - 1; i >= 0; --i) {
    const int* v = i < kRanges ? a.count + i * a.nwin : (i == kRanges ? a.slots : a.long_rows);
    int before = 0, sum = 0;
#pragma unroll 4
    for (int j = threadIdx.x; j < a.nwin; j += kTaskThreads) {
      const int n = v[j];
      sum += n;
      before += j < w ? n : 0;
    }
    before = wave_sum(before);
    sum = wave_sum(sum);
    if ((threadIdx.x & (kWave - 1)) == 0) {
      atomicAdd(&s_before[i], before);
      atomicAdd(&s_all[i], sum);
    }
    if (i == kSums - 1) {
      __syncthreads();
      if (s_all[i] == 0) break;  // no long rows
    }
  }
  __syncthreads();
  RangePlace p;
  int first = 0;
#pragma unroll
  for (int x = 0; x < kRanges; ++x) {
    p.task[x] = first + s_before[x];
    first += s_all[x];
  }
  p.slot = s_before[kRanges];
  p.split = s_before[kRanges + 1];
  all[0] = s_all[kRanges];
  all[1] = s_all[kRanges + 1];
  return p;
}

// kRangeGroup windows from window w on by a workgroup of kTaskThreads, a lane per (long row, range) as in range_cut: the pieces of a range by length, so that
// the lane groups of a wave end together; the slots of a row's pieces follow each other through the ranges.
__device__ __forceinline__ void range_write(const RangeLists& a, int w, const RangePlace& place, int4* __restrict__ task, int4* __restrict__ split) {
  __shared__ int s_row[kRangeGroup * kTaskWindow], s_n, at[kRanges][kRangePiece + 1];
  __shared__ int s_wave[kTaskThreads / kWave], s_first[kRanges];
  const int t = threadIdx.x, x = t % kRanges;
  if (t == 0) s_n = 0;
#pragma unroll
  for (int y = 0; y < kRanges; ++y)
    if (t == y) s_first[y] = place.task[y];
  for (int k = t; k < kRanges * (kRangePiece + 1); k += kTaskThreads) at[0][k] = 0;
  __syncthreads();
  {
    constexpr int kRowsEach = kRangeGroup * kTaskRowsPerThread;
    int len[kRowsEach];
#pragma unroll
    for (int u = 0; u < kRowsEach; ++u) {
      const int64_t r = int64_t(w) * kTaskWindow + u * kTaskThreads + t;
      len[u] = r < a.nrows ? a.rowptr[r + 1] - a.rowptr[r] : 0;
    }
#pragma unroll
    for (int u = 0; u < kRowsEach; ++u)
      if (len[u] >= a.min_row) s_row[atomicAdd(&s_n, 1)] = w * kTaskWindow + u * kTaskThreads + t;
  }
  __syncthreads();
  const int n = s_n;
  constexpr int kRows = kTaskThreads / kRanges;
  for (int i = t / kRanges; i < n; i += kRows) {
    const RangeShare s = range_share_of(a, s_row[i], x);
    if (s.m > 1) atomicAdd(&at[x][s.part], s.m - 1);
    if (s.m > 0) atomicAdd(&at[x][s.len - (s.m - 1) * s.part], 1);
  }
  __syncthreads();
  const int lane = t & (kWave - 1);
  const bool rising = w / kRangeGroup % 2 != 0;  // in turn, so that a wave across two groups of windows takes equal lengths, too
  for (int y = t / kWave; y < kRanges; y += kTaskThreads / kWave) {
    int carry = s_first[y];
    for (int k0 = 0; k0 <= kRangePiece; k0 += kWave) {
      const int k = rising ? k0 + lane : kRangePiece - k0 - lane;
      const bool in = k >= 0 && k <= kRangePiece;
      const int c = in ? at[y][k] : 0;
      int incl = c;
      for (int d = 1; d < kWave; d <<= 1) {
        const int v = __shfl_up(incl, d);
        if (lane >= d) incl += v;
      }
      if (in) at[y][k] = carry + incl - c;
      carry += __shfl(incl, kWave - 1);
    }
  }
  int next = place.slot;
  for (int i0 = 0; i0 < n; i0 += kRows) {  // uniform: the workgroup scans
    const int i = i0 + t / kRanges;
    RangeShare s{0, 0, 0, 0};
    if (i < n) s = range_share_of(a, s_row[i], x);
    int total;
    const int incl = range_scan(s.m, s_wave, &total);  // (its barriers are behind the offsets in `at`)
    const int slot = next + incl - s.m, end = __shfl(next + incl, kRanges - 1, kRanges);
    if (i < n && x == 0) split[place.split + i] = make_int4(s_row[i], slot, end - slot, 0);
    // All pieces but the last are equally long, so they follow each other in the list.  Where there are many the whole wave writes them: a
    // row of 3 M non-zeros was a serial loop of eight lanes, a plan with S = 256 358 us instead of 154, with S = 4 19 ms instead of 1.8.
    int first = 0, last = 0;
    if (s.m > 1) first = atomicAdd(&at[x][s.part], s.m - 1);
    if (s.m > 0) last = atomicAdd(&at[x][s.len - (s.m - 1) * s.part], 1);
    const int row = i < n ? s_row[i] : 0;
    if (s.m > 0) task[last] = make_int4(s.beg + (s.m - 1) * s.part, s.len - (s.m - 1) * s.part, row, slot + s.m - 1);
    constexpr int kFew = 4;
    if (s.m <= kFew)
      for (int j = 0; j < s.m - 1; ++j) task[first + j] = make_int4(s.beg + j * s.part, s.part, row, slot + j);
    for (unsigned long long many = __ballot(s.m > kFew); many; many &= many - 1) {
      const int src = __ffsll((long long)many) - 1;
      const int m = __shfl(s.m, src), part = __shfl(s.part, src), beg = __shfl(s.beg, src), r = __shfl(row, src), sl = __shfl(slot, src);
      const int f = __shfl(first, src);
      for (int j = lane; j < m - 1; j += kWave) task[f + j] = make_int4(beg + j * part, part, r, sl + j);
    }
    next += total;
  }
}

}  // namespace hgnn

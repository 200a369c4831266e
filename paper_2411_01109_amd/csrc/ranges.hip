// Long rows of a graph whose feature table misses the L2s, cut at the borders of column ranges.  Integer work only; set-up.
//
// Eight L2s of 4 MB keep the popular rows of a large table eight times over when every XCD gathers from all of it.  Columns ascend
// inside a row, so a row's share of a column range is a run of its non-zeros, and a run is a piece of the row like any other (task.h):
// nothing is copied or re-ordered.  The pieces are listed range after range and an eighth of the list goes to each XCD, whose L2 then
// sees an eighth of the columns.  What it costs is a staged partial row per (row, range), so only rows that have several pieces anyway
// are cut; on a power law they hold most of the non-zeros (62 M x 128: L2 hits 31 -> 49 %, misses 11.9 -> 8.9 GB a call).
#include "common.h"

namespace hgnn {

constexpr int kRangeThreads = 256;
constexpr int kRangeWindow = kRangeThreads;  // long rows that are sorted by length together, one per thread
constexpr int kRangePiece = 256;             // most non-zeros of a piece (also at most S)
constexpr int kRangeWaves = kRangeThreads / kWave;

// Where rows are cut.  A segment size is the least length because such rows leave staged partial rows (fp16, as ever) in any case.
// us a call, rows in pieces of S / at column ranges (F = 64 and one head if not said; power law unless log-normal):
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
//   34 MB, 5.5 M, 4 heads                 59 / 58           123 / 114     59 / 58    105 / 99, 130 / 121
//   13 MB, 8 M                            58 / 61           106 / 101     52 / 52
//   8 MB, 8 M                             56 / 64            96 / 94      50 / 53
//   34 MB, 2.1 M, F = 128: GIN layer forward 44 / 46; 10 MB, 1.3 M: by degrees 30 / 48
// Counting and listing the pieces takes 55 us of a plan that takes 100 otherwise, so the line is what the eight L2s hold together and not
// half of it: below, a layer gains 1 to 4 %.
int range_min_row(int64_t nnz, int64_t ncols, int max_F, int S, int64_t l2) {
  constexpr int64_t kLeastNnz = int64_t(4) << 20;
  return nnz > kLeastNnz && ncols * max_F * 2 > 8 * l2 ? S + 1 : kNoRanges;
}

// The arrays are laid out for `cap` rows, as many as nnz non-zeros can make long; how many there are is read from the device, so
// that the host waits once for these numbers and all others.  Nothing has been checked when the counting kernels run.
struct RangeLists {
  const int* rowptr;
  const int* n_long;
  int* rows;   // [cap]
  int* cuts;   // [kRanges + 1][cap] where a row's share of each range begins
  int* count;  // [kRanges][nwin] pieces, then where they go
  int* slots;  // [nwin] pieces of a window's rows, then the first of them
  int cap, nwin, piece;
  int64_t nnz;
  __device__ __forceinline__ int n() const { return *n_long < cap ? *n_long : cap; }
};

static RangeLists range_lists(const TaskSource& q, const TaskCounts& c, size_t* bytes) {
  RangeLists a{};
  a.rowptr = q.rowptr;
  a.n_long = c.n_long;
  a.nnz = q.nnz;
  a.cap = int(q.nnz / q.range_min) + 1;
  a.nwin = int(ceil_div(a.cap, kRangeWindow));
  a.piece = q.S < kRangePiece ? q.S : kRangePiece;
  const size_t cap = size_t(a.cap), nwin = size_t(a.nwin);
  if (bytes) *bytes = sizeof(int) * ((kRanges + 2) * cap + (kRanges + 1) * nwin);
  a.rows = c.ranges.as<int>();
  a.cuts = a.rows + cap;
  a.count = a.cuts + (kRanges + 1) * cap;
  a.slots = a.count + kRanges * nwin;
  return a;
}

// the long rows of a window of kTaskWindow rows
__global__ __launch_bounds__(kRangeThreads) void range_list_kernel(RangeLists a, const int* __restrict__ long_at, int nrows, int range_min) {
  __shared__ int next;
  if (threadIdx.x == 0) next = long_at[blockIdx.x];
  __syncthreads();
  for (int u = 0; u < kTaskWindow; u += kRangeThreads) {
    const int64_t r = int64_t(blockIdx.x) * kTaskWindow + u + threadIdx.x;
    if (r >= nrows || a.rowptr[r + 1] - a.rowptr[r] < range_min) continue;
    const int k = atomicAdd(&next, 1);
    if (k < a.cap) a.rows[k] = int(r);
  }
}

// a thread per (row, range): the first non-zero of the range by binary search
__global__ __launch_bounds__(kRangeThreads) void range_cut_kernel(RangeLists a, const int* __restrict__ col, int width) {
  const int64_t t = int64_t(blockIdx.x) * kRangeThreads + threadIdx.x;
  const int64_t i = t / kRanges;
  const int x = int(t % kRanges);
  if (i >= a.n()) return;
  const int row = a.rows[i];
  int beg = a.rowptr[row], end = a.rowptr[row + 1];
  if (beg < 0 || end < beg || end > a.nnz) beg = end = 0;  // an offset array that validation will reject
  pos_t lo = pos_t(beg), hi = pos_t(end);
  if (x == 0) {
    a.cuts[int64_t(kRanges) * a.cap + i] = end;
  } else {
    const int64_t first = int64_t(x) * width;
    while (lo < hi) {
      const pos_t mid = (lo + hi) / 2;
      if (col[mid] < first) lo = mid + 1;
      else hi = mid;
    }
  }
  a.cuts[int64_t(x) * a.cap + i] = int(lo);
}

struct Share {
  int len, part, m;  // non-zeros, non-zeros per piece, pieces
};
__device__ __forceinline__ Share share_of(const RangeLists& a, int n, int i, int x) {
  Share s{0, 0, 0};
  if (i < n) s.len = a.cuts[int64_t(x + 1) * a.cap + i] - a.cuts[int64_t(x) * a.cap + i];
  if (s.len > 0) {
    s.part = pieces_of(s.len, pieces_of(s.len, a.piece));
    s.m = pieces_of(s.len, s.part);
  }
  return s;
}

// inclusive scan over the workgroup of one value per thread; *total on all threads
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
  for (int w = 0; w < kRangeWaves; ++w) {
    if (w < wave) before += s_wave[w];
    all += s_wave[w];
  }
  *total = all;
  return before + incl;
}

// a workgroup per window, a thread per row
__global__ __launch_bounds__(kRangeThreads) void range_count_kernel(RangeLists a) {
  __shared__ int s_wave[kRangeWaves];
  const int n = a.n(), i = blockIdx.x * kRangeWindow + threadIdx.x;
  int all = 0;
  for (int x = 0; x < kRanges; ++x) {
    int total;
    (void)range_scan(share_of(a, n, i, x).m, s_wave, &total);
    if (threadIdx.x == 0) a.count[x * a.nwin + blockIdx.x] = total;
    all += total;
  }
  if (threadIdx.x == 0) a.slots[blockIdx.x] = all;
}

// one workgroup: exclusive scans in place, and all pieces to the host
__global__ __launch_bounds__(kRangeThreads) void range_scan_kernel(RangeLists a, TaskTotals* out) {
  __shared__ int s_wave[kRangeWaves];
  auto scan = [&](int* v, int n) {
    int carry = 0;
    for (int i0 = 0; i0 < n; i0 += kRangeThreads) {
      const int i = i0 + int(threadIdx.x), x = i < n ? v[i] : 0;
      int total;
      const int incl = range_scan(x, s_wave, &total);
      if (i < n) v[i] = carry + incl - x;
      carry += total;
    }
    return carry;
  };
  const int all = scan(a.count, kRanges * a.nwin);
  (void)scan(a.slots, a.nwin);
  if (threadIdx.x == 0) out->n_range = all;
}

// a workgroup per window: the pieces of a range by falling length, so that the lane groups of a wave end together.  The slots
// of a row's pieces follow each other through the ranges.
__global__ __launch_bounds__(kRangeThreads) void range_write_kernel(RangeLists a, int first_slot, int4* __restrict__ task,
                                                                   int4* __restrict__ split) {
  __shared__ int at[kRangePiece + 1];
  __shared__ int s_wave[kRangeWaves];
  const int n = a.n(), t = threadIdx.x, i = blockIdx.x * kRangeWindow + t;
  int m = 0, total;
  for (int x = 0; x < kRanges; ++x) m += share_of(a, n, i, x).m;
  int slot = first_slot + a.slots[blockIdx.x] + range_scan(m, s_wave, &total) - m;
  int row = 0;
  if (i < n) {
    row = a.rows[i];
    split[i] = make_int4(row, slot, m, 0);
  }
  for (int x = 0; x < kRanges; ++x) {
    __syncthreads();
    for (int k = t; k <= kRangePiece; k += kRangeThreads) at[k] = 0;
    __syncthreads();
    const Share s = share_of(a, n, i, x);
    if (s.m > 0) {
      if (s.m > 1) atomicAdd(&at[s.part], s.m - 1);
      atomicAdd(&at[s.len - (s.m - 1) * s.part], 1);
    }
    __syncthreads();
    if (t < kWave) {  // longest first
      int carry = a.count[x * a.nwin + blockIdx.x];
      for (int k0 = kRangePiece; k0 >= 0; k0 -= kWave) {
        const int k = k0 - t;
        const int c = k >= 0 ? at[k] : 0;
        int incl = c;
        for (int d = 1; d < kWave; d <<= 1) {
          const int u = __shfl_up(incl, d);
          if (t >= d) incl += u;
        }
        if (k >= 0) at[k] = carry + incl - c;
        carry += __shfl(incl, kWave - 1);
      }
    }
    __syncthreads();
    if (s.m > 0) {
      const int beg = a.cuts[int64_t(x) * a.cap + i];
      for (int j = 0; j < s.m; ++j) {
        const int len = j + 1 < s.m ? s.part : s.len - j * s.part;
        task[atomicAdd(&at[len], 1)] = make_int4(beg + j * s.part, len, row, slot + j);
      }
      slot += s.m;
    }
  }
}

// after the counts of the row tasks: the long rows and their pieces, counted; the number of pieces is in c.totals with the others
hgnn_status range_count(const TaskSource& q, const int32_t* col, int ncols, TaskCounts& c, SetupStream& s) {
  size_t bytes = 0;
  (void)range_lists(q, c, &bytes);
  HGNN_HIP(c.ranges.alloc(bytes));
  const RangeLists a = range_lists(q, c, nullptr);
  const int width = int(ceil_div(ncols, kRanges));
  if (q.nrows > 0) range_list_kernel<<<dim3(unsigned(ceil_div(q.nrows, kTaskWindow))), kRangeThreads, 0, s>>>(a, c.long_at, q.nrows, q.range_min);
  range_cut_kernel<<<dim3(unsigned(ceil_div(int64_t(a.cap) * kRanges, kRangeThreads))), kRangeThreads, 0, s>>>(a, col, width);
  range_count_kernel<<<dim3(unsigned(a.nwin)), kRangeThreads, 0, s>>>(a);
  range_scan_kernel<<<1, kRangeThreads, 0, s>>>(a, c.totals);
  HGNN_LAUNCH_CHECK("range_list_kernel / range_cut_kernel / range_count_kernel / range_scan_kernel");
  return HGNN_OK;
}

// the c.got.n_range pieces and, behind the other rows of several pieces, the c.got.n_long rows they belong to
hgnn_status range_write(const TaskSource& q, const TaskCounts& c, hgnn_row_tasks* t, SetupStream& s) {
  const RangeLists a = range_lists(q, c, nullptr);
  range_write_kernel<<<dim3(unsigned(ceil_div(c.got.n_long, kRangeWindow))), kRangeThreads, 0, s>>>(a, c.got.n_slots, t->rtask, t->split + c.got.n_split);
  HGNN_LAUNCH_CHECK("range_write_kernel");
  return HGNN_OK;
}

}  // namespace hgnn

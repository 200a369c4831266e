// CSR of the transposed graph plus the edge-id map, for the backward SpMM dX <- A_w^T dY
// (paper section 2.1.2), and CSR from a COO edge list (section 2.1.1).  One-off set-up: a stable radix sort of
// the non-zeros by column id, or by (row id, column id), as words that carry everything (sort.h); where the fields do not fit 64 bits,
// keys and positions go through rocPRIM's device radix sort.
#include <string.h>

#include <rocprim/device/device_radix_sort.hpp>

#include "common.h"
#include "sort.h"

namespace hgnn {

// rowptr_T[j] = number of sorted keys whose leading field (key >> shift) is < j
template <class Key>
__global__ void offsets_kernel(const Key* __restrict__ sorted, int shift, int64_t nnz, int ncols, int* __restrict__ rowptr_T) {
  int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (j > ncols) return;
  int64_t lo = 0, hi = nnz;
  while (lo < hi) {
    int64_t mid = (lo + hi) >> 1;
    if (int64_t(sorted[mid] >> shift) < j) lo = mid + 1;
    else hi = mid;
  }
  rowptr_T[j] = int(lo);
}

// COO -> CSR: a word is (row, col, list position) (position_bits = 0: without it), so that one stable sort of the leading fields
// orders the edges by row, then column, then position in the list; bad receives 1 when an id is out of range (which then counts as 0)
struct CooWords {
  const int *row, *col;
  int nrows, ncols, col_bits, position_bits;
  int* bad;
  template <int PER>
  __device__ __forceinline__ void prepare(int64_t, int, int*) const {}
  __device__ __forceinline__ uint64_t word(int r, int c, int64_t k, bool& ok) const {
    const bool rok = uint32_t(r) < uint32_t(nrows), cok = uint32_t(c) < uint32_t(ncols);
    ok = ok && rok && cok;
    const uint64_t rc = (uint64_t(uint32_t(rok ? r : 0)) << col_bits) | uint64_t(uint32_t(cok ? c : 0));
    return position_bits ? (rc << position_bits) | uint64_t(k) : rc;
  }
  template <int PER>
  __device__ __forceinline__ void load(int64_t first, int n, int mine, const int*, uint64_t (&w)[PER]) const {
    int r[PER], c[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t k = first + min(mine + j * kWave, n - 1);
      r[j] = row[k];
      c[j] = col[k];
    }
    bool ok = true;
#pragma unroll
    for (int j = 0; j < PER; ++j) w[j] = word(r[j], c[j], first + min(mine + j * kWave, n - 1), ok);
    if (!ok) *bad = 1;
  }
  __device__ __forceinline__ uint64_t count(const SortPass& p, int64_t k) const {  // (the rows only where the digit reaches into them)
    bool ok = true;
    return word(p.shift + p.bits > position_bits + col_bits ? row[k] : 0, col[k], k, ok);
  }
};

// the same in two arrays where the three fields do not fit 64 bits
__global__ void coo_keys_kernel(CooWords w, int64_t nnz, uint64_t* __restrict__ keys, int* __restrict__ ids) {
  int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= nnz) return;
  bool ok = true;
  keys[k] = w.word(w.row[k], w.col[k], k, ok);
  if (!ok) *w.bad = 1;
  ids[k] = int(k);
}

// by a whole wave, 64 places looked at in each step: how many of n places come before the first where before() does not hold; every place is
// looked at inside [0, n) whatever before() says
template <class Before>
__device__ __forceinline__ int64_t wave_partition(int64_t n, Before&& before) {
  const int lane = threadIdx.x & (kWave - 1);
  int64_t lo = 0, hi = n;  // the answer is in [lo, hi]
  while (lo < hi) {
    const int64_t step = (hi - lo + kWave - 1) / kWave, at = lo + lane * step;
    const int held = __popcll(__ballot(at < hi && before(at)));
    // of a sorted array those lanes are the first ones
    if (held == 0) {
      hi = lo;
    } else {
      const int64_t last = lo + (held - 1) * step;  // holds there
      hi = last + step < hi ? last + step : hi;
      lo = last + 1;
    }
  }
  return lo;
}

// row_of_edge by a whole wave
__device__ __forceinline__ int wave_row_of_edge(const int* __restrict__ rowptr, int nrows, int64_t k) {
  return int(wave_partition(int64_t(nrows) + 1, [&](int64_t r) { return int64_t(rowptr[r]) <= k; })) - 1;
}

// Sorted words taken apart: the low `position_bits` to pos (may be null), the next `id_bits` to id, and offset[r] = number of words
// whose leading `lead_bits` are < r, for r = 0 .. nlead.  The workgroup that holds the first word of a row writes that row's offset and
// those of the empty rows before it, long stretches of them with all its threads.  Bound by memory: 17.2 us for 5.5 M words (5.1 TB/s).
// FORM kSplitGaps: a workgroup takes some 75 us for a stretch of a million (33 M vertices with all edges at one: 1.2 of 1.8 ms), so windows of
// kSplitWindow offsets that are equal throughout are left to workgroups of their own, the first `windows`; 1.3 us at 5.5 M words.
// kSplitSearch: those workgroups write all offsets, by searches among the words of those rows.  With few words most stretches are long enough
// to be written one after the other: 1000 words over 100 000 rows 70 / 47 us a list, 131 072 over 300 000 103 / 107.
enum SplitForm { kSplitFill, kSplitGaps, kSplitSearch };
constexpr int kSplitWindow = 1024, kStagedWords = 4096;
template <SplitForm FORM>
__global__ __launch_bounds__(kBlock) void split_words_kernel(const uint64_t* __restrict__ words, int64_t nnz, int position_bits, int id_bits,
                                                            int lead_bits, int nlead, int windows, int* __restrict__ id, int* __restrict__ pos,
                                                            int* __restrict__ offset) {
  constexpr int kAlone = 16;
  __shared__ int s_n, s_gap[(FORM == kSplitGaps ? 2 : 1) * (kBlock + 1)][3];
  auto lead_of = [&](uint64_t w) { return int(min(uint64_t(nlead), (w >> (position_bits + id_bits)) & ((uint64_t(1) << lead_bits) - 1))); };
  if (FORM != kSplitFill && int(blockIdx.x) < windows) {
    const int64_t a = int64_t(blockIdx.x) * kSplitWindow, b = a + kSplitWindow - 1 < nlead ? a + kSplitWindow - 1 : nlead;
    const int w = threadIdx.x / kWave;
    if (w < 2) {
      const int64_t n = wave_partition(nnz, [&](int64_t i) { return lead_of(words[i]) < (w == 0 ? a : b); });
      if ((threadIdx.x & (kWave - 1)) == 0) s_gap[0][w] = int(n);
    }
    __syncthreads();
    const int from = s_gap[0][0], n = s_gap[0][1] - from;
    if (FORM == kSplitGaps) {
      if (n == 0)
        for (int64_t r = a + threadIdx.x; r <= b; r += kBlock) offset[r] = from;
      return;
    }
    __shared__ int s_lead[FORM == kSplitSearch ? kStagedWords : 1];
    if (n <= kStagedWords) {
      for (int i = threadIdx.x; i < n; i += kBlock) s_lead[i] = lead_of(words[from + i]);
      __syncthreads();
    }
    constexpr int kEach = kSplitWindow / kBlock;
    int at[kEach] = {};  // words below, searched for side by side
    for (int step = n > 0 ? 1 << (31 - __clz(n)) : 0; step > 0; step >>= 1)
#pragma unroll
      for (int j = 0; j < kEach; ++j) {
        const int i = at[j] + step;
        if (i <= n) {
          const int lead = n <= kStagedWords ? s_lead[i - 1] : lead_of(words[from + i - 1]);
          if (lead < a + j * kBlock + int(threadIdx.x)) at[j] = i;
        }
      }
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int64_t r = a + j * kBlock + threadIdx.x;
      if (r <= b) offset[r] = from + at[j];
    }
    return;
  }
  if (FORM != kSplitSearch) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
  }
  const int64_t k = (int64_t(blockIdx.x) - (FORM != kSplitFill ? windows : 0)) * kBlock + threadIdx.x;
  auto fill_part = [&](int from, int to, int64_t v) {
    if (to - from < kAlone) {
      for (int r = from; r <= to; ++r) offset[r] = int(v);
    } else {
      const int i = atomicAdd(&s_n, 1);
      s_gap[i][0] = from;
      s_gap[i][1] = to;
      s_gap[i][2] = int(v);
    }
  };
  auto fill = [&](int from, int to, int64_t v) {  // offset[from .. to] = v
    if (FORM == kSplitGaps) {  // but for the windows inside: [a, b) are those (the last one may be shorter)
      const int64_t a = (int64_t(from) + kSplitWindow - 1) / kSplitWindow * kSplitWindow;
      const int64_t b = to == nlead ? int64_t(nlead) + 1 : (int64_t(to) + 1) / kSplitWindow * kSplitWindow;
      if (a < b) {
        if (from < a) fill_part(from, int(a) - 1, v);
        if (b <= to) fill_part(int(b), to, v);
        return;
      }
    }
    fill_part(from, to, v);
  };
  if (k < nnz) {
    const uint64_t w = words[k];
    id[k] = int(uint32_t(w >> position_bits) & ((uint32_t(1) << id_bits) - 1u));
    if (pos) pos[k] = int(uint32_t(w) & ((uint32_t(1) << position_bits) - 1u));
    if (FORM != kSplitSearch) {
      const int r = lead_of(w), q = k > 0 ? lead_of(words[k - 1]) : -1;
      if (r > q) fill(q + 1, r, k);
      if (k == nnz - 1 && r < nlead) fill(r + 1, nlead, nnz);
    }
  }
  if (FORM == kSplitSearch) return;
  __syncthreads();
  for (int i = 0; i < s_n; ++i)
    for (int r = s_gap[i][0] + int(threadIdx.x); r <= s_gap[i][1]; r += kBlock) offset[r] = s_gap[i][2];
}

static void launch_split_words(const uint64_t* words, int64_t nnz, int position_bits, int id_bits, int lead_bits, int nlead, int* id, int* pos,
                               int* offset, hipStream_t s) {
  // (with sixteen words for every offset the sort takes ten times as long as the longest stretch that there can be)
  const SplitForm form = nnz < nlead / 8 ? kSplitSearch : (nlead > 65536 && nnz < 16 * int64_t(nlead) ? kSplitGaps : kSplitFill);
  const int64_t edges = ceil_div(nnz, kBlock), windows = form == kSplitFill ? 0 : ceil_div(int64_t(nlead) + 1, kSplitWindow);
  const auto kernel = form == kSplitFill ? split_words_kernel<kSplitFill> : (form == kSplitGaps ? split_words_kernel<kSplitGaps> : split_words_kernel<kSplitSearch>);
  kernel<<<dim3(unsigned(edges + windows)), kBlock, 0, s>>>(words, nnz, position_bits, id_bits, lead_bits, nlead, int(windows), id, pos, offset);
}

// The row of every non-zero, handed to put(k, row): a workgroup takes kExpand consecutive positions, its rows mark the slot
// of their first non-zero in LDS and a running maximum spreads the ids (a search of the offset array per non-zero took
// 196 us at 5.5 M non-zeros).  A graph may come here before anything has looked at its offset array: whatever that holds, reads
// stay inside its nrows + 1 entries and marks inside the tile (the rows are then wrong, as the array is).
constexpr int kExpandPerThread = 8;
constexpr int kExpand = kBlock * kExpandPerThread;

// s_row[i] = row of position e0 + i, i < n <= PER THREADS; the workgroup has been waited for at the end
template <int THREADS, int PER>
__device__ __forceinline__ void expand_tile(const int* __restrict__ rowptr, int nrows, int64_t e0, int n, int* s_row) {
  __shared__ int s_max[THREADS / kWave], s_lim[2];
  if (threadIdx.x < 2 * kWave) {
    const int w = threadIdx.x / kWave, r = wave_row_of_edge(rowptr, nrows, w == 0 ? e0 : e0 + n - 1);
    if ((threadIdx.x & (kWave - 1)) == 0) s_lim[w] = r;
  }
  for (int i = threadIdx.x; i < THREADS * PER; i += THREADS) s_row[i] = -1;
  __syncthreads();
  const int lo = max(s_lim[0], 0), hi = min(s_lim[1], nrows - 1);
  if (hi - lo > 16 * n) {  // few positions among many rows: the row of each by search (8192 over 1 M rows, a transpose 329 -> 86 us)
    int r[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) r[j] = lo;
    for (int step = 1 << (31 - __clz(hi - lo)); step > 0; step >>= 1)
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (hi - r[j] >= step && int64_t(rowptr[r[j] + step]) <= e0 + j * THREADS + int(threadIdx.x)) r[j] += step;
#pragma unroll
    for (int j = 0; j < PER; ++j) s_row[j * THREADS + threadIdx.x] = r[j];
    __syncthreads();
    return;
  }
  for (int r = lo + 1 + int(threadIdx.x); r <= hi; r += THREADS) {
    const int p = rowptr[r];
    const int64_t at = int64_t(p) - e0;
    if (rowptr[r + 1] > p && at >= 0 && at < n) s_row[at] = r;
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int v[PER], run = lo;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    run = max(run, s_row[threadIdx.x * PER + j]);
    v[j] = run;
  }
  int incl = run;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int t = __shfl_up(incl, d);
    if (lane >= d) incl = max(incl, t);
  }
  if (lane == kWave - 1) s_max[wave] = incl;
  int excl = __shfl_up(incl, 1);
  if (lane == 0) excl = lo;
  __syncthreads();
  for (int w = 0; w < wave; ++w) excl = max(excl, s_max[w]);
#pragma unroll
  for (int j = 0; j < PER; ++j) s_row[threadIdx.x * PER + j] = max(v[j], excl);
  __syncthreads();
}

template <class Put>
__device__ __forceinline__ void expand_rows(const int* __restrict__ rowptr, int nrows, int64_t nnz, Put&& put) {
  __shared__ int s_row[kExpand];
  const int64_t e0 = int64_t(blockIdx.x) * kExpand;
  const int n = int(nnz - e0 < kExpand ? nnz - e0 : kExpand);
  expand_tile<kBlock, kExpandPerThread>(rowptr, nrows, e0, n, s_row);
  for (int i = threadIdx.x; i < n; i += kBlock) put(e0 + i, s_row[i]);
}

// transposition: a word is (column, row, position); sorting the columns' bits brings everything along
struct TransposeWords {
  const int *rowptr, *col;
  int nrows, row_bits, position_bits;
  template <int PER>
  __device__ __forceinline__ void prepare(int64_t first, int n, int* s_row) const { expand_tile<kSortThreads, PER>(rowptr, nrows, first, n, s_row); }
  template <int PER>
  __device__ __forceinline__ void load(int64_t first, int n, int mine, const int* s_row, uint64_t (&w)[PER]) const {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int i = min(mine + j * kWave, n - 1);
      w[j] = (((uint64_t(uint32_t(col[first + i])) << row_bits) | uint64_t(uint32_t(s_row[i]))) << position_bits) | uint64_t(first + i);
    }
  }
  __device__ __forceinline__ uint64_t count(const SortPass&, int64_t k) const { return uint64_t(uint32_t(col[k])) << (row_bits + position_bits); }
};

// the same in two arrays where the three fields do not fit 64 bits: column keys with positions; rows of all positions
__global__ __launch_bounds__(kBlock) void transpose_rows_kernel(const int* __restrict__ rowptr, const int* __restrict__ col, int nrows,
                                                                int64_t nnz, int* __restrict__ rows, uint32_t* __restrict__ keys,
                                                                int* __restrict__ ids) {
  expand_rows(rowptr, nrows, nnz, [&](int64_t k, int r) {
    rows[k] = r;
    keys[k] = uint32_t(col[k]);
    ids[k] = int(k);
  });
}

__global__ void source_rows_kernel(const int* __restrict__ rows, const int* __restrict__ order, int64_t nnz, int* __restrict__ col_T,
                                   int* __restrict__ eid_T) {
  int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= nnz) return;
  const int e = order[k];
  eid_T[k] = e;
  col_T[k] = rows[e];
}

static int bits_for(int64_t n) {  // bits that hold 0 .. n - 1
  int b = 1;
  while ((int64_t(1) << b) < n) ++b;
  return b;
}

// out[i, f] = fp16(scale[i] * X[i, f]), 8 halves per thread
__global__ void scale_rows_kernel(int64_t n, int F8, const half_t* __restrict__ X, int64_t ldx, const float* __restrict__ scale,
                                  half_t* __restrict__ out, int64_t ldo) {
  const int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (j >= n * F8) return;
  const int64_t i = j / F8;
  const int f0 = int(j - i * F8) * 8;
  const float sc = scale[i];
  const half8_t x = *reinterpret_cast<const half8_t*>(X + i * ldx + f0);
  half8_t y;
#pragma unroll
  for (int q = 0; q < 8; ++q) y[q] = half_t(sc * float(x[q]));
  *reinterpret_cast<half8_t*>(out + i * ldo + f0) = y;
}

// out[k*H + h] = in[eid[k]*H + h]: an edge tensor brought into the edge order of the transposed graph
__global__ void edge_gather_kernel(const int* __restrict__ eid, int64_t total, int H, const half_t* __restrict__ in,
                                   half_t* __restrict__ out) {
  const int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (j >= total) return;
  const int64_t k = j / H;
  out[j] = in[int64_t(eid[k]) * H + (j - k * H)];
}

}  // namespace hgnn

using namespace hgnn;

extern "C" hgnn_status hgnn_transpose(const hgnn_csr* g, int32_t* rowptr_T, int32_t* col_T, int32_t* eid_T,
                                      void* stream) {
  clear_error();
  hgnn_status st = check_csr_args(g, "hgnn_transpose");
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EINVAL, "hgnn_transpose: the input graph must not carry an edge-id map");
  HGNN_REQUIRE(rowptr_T != nullptr, HGNN_EINVAL, "hgnn_transpose: rowptr_T is NULL");
  HGNN_REQUIRE(g->nnz == 0 || (col_T && eid_T), HGNN_EINVAL, "hgnn_transpose: col_T or eid_T is NULL");
  SetupStream s(stream);
  const int64_t E = g->nnz;
  if (E == 0) {
    HGNN_HIP(hipMemsetAsync(rowptr_T, 0, sizeof(int) * (size_t(g->ncols) + 1), s));
    HGNN_HIP(s.wait());
    return HGNN_OK;
  }
  const int col_bits = bits_for(g->ncols), row_bits = bits_for(g->nrows), pos_bits = bits_for(E);
  const dim3 per_edge(unsigned(ceil_div(E, kBlock))), per_tile(unsigned(ceil_div(E, kExpand)));
  const dim3 per_col(unsigned(ceil_div(int64_t(g->ncols) + 1, kBlock)));
  DevTemp buf[2] = {DevTemp(s), DevTemp(s)}, ids[2] = {DevTemp(s), DevTemp(s)}, rows(s), tmp(s);
  size_t tmp_bytes = 0;
  hipError_t e = hipSuccess;
  if (col_bits + row_bits + pos_bits <= 64) {
    // one word per non-zero carries its row and position through a sort of the columns alone: no gather afterwards
    for (int i = 0; i < 2 && e == hipSuccess; ++i) e = buf[i].alloc(8 * size_t(E));
    if (e == hipSuccess) e = tmp.alloc(sort_scratch_bytes(E));
    if (e == hipSuccess) {
      const int first = row_bits + pos_bits;
      const uint64_t* words = sort_words(TransposeWords{g->rowptr, g->col, g->nrows, row_bits, pos_bits}, E, first, first + col_bits,
                                         buf[0].as<uint64_t>(), buf[1].as<uint64_t>(), tmp.p, s);
      launch_split_words(words, E, pos_bits, row_bits, col_bits, g->ncols, col_T, eid_T, rowptr_T, s);
      e = hipGetLastError();
    }
  } else {
    for (int i = 0; i < 2 && e == hipSuccess; ++i) e = buf[i].alloc(4 * size_t(E));
    for (int i = 0; i < 2 && e == hipSuccess; ++i) e = ids[i].alloc(4 * size_t(E));
    if (e == hipSuccess) e = rows.alloc(4 * size_t(E));
    rocprim::double_buffer<uint32_t> keys(buf[0].as<uint32_t>(), buf[1].as<uint32_t>());
    rocprim::double_buffer<int> order(ids[0].as<int>(), ids[1].as<int>());
    if (e == hipSuccess) e = rocprim::radix_sort_pairs(nullptr, tmp_bytes, keys, order, unsigned(E), 0u, unsigned(col_bits), s);
    if (e == hipSuccess) e = tmp.alloc(tmp_bytes);
    if (e == hipSuccess) {
      transpose_rows_kernel<<<per_tile, kBlock, 0, s>>>(g->rowptr, g->col, g->nrows, E, rows.as<int>(), keys.current(), order.current());
      e = rocprim::radix_sort_pairs(tmp.p, tmp_bytes, keys, order, unsigned(E), 0u, unsigned(col_bits), s);
    }
    if (e == hipSuccess) {
      source_rows_kernel<<<per_edge, kBlock, 0, s>>>(rows.as<int>(), order.current(), E, col_T, eid_T);
      offsets_kernel<uint32_t><<<per_col, kBlock, 0, s>>>(keys.current(), 0, E, g->ncols, rowptr_T);
      e = hipGetLastError();
    }
  }
  if (e == hipSuccess) e = s.wait();
  if (e != hipSuccess)
    return fail(e == hipErrorOutOfMemory ? HGNN_ENOMEM : HGNN_EHIP, "hgnn_transpose: %s", hipGetErrorString(e));
  return HGNN_OK;
}

extern "C" hgnn_status hgnn_coo_to_csr(int32_t nrows, int32_t ncols, int64_t nnz, const int32_t* row, const int32_t* col,
                                       int32_t* rowptr, int32_t* col_out, int32_t* eid, void* stream) {
  clear_error();
  const char* who = "hgnn_coo_to_csr";
  HGNN_REQUIRE(nrows >= 0 && ncols >= 0 && nnz >= 0, HGNN_EINVAL, "%s: negative size", who);
  HGNN_REQUIRE(nnz < (int64_t(1) << 31), HGNN_EINVAL, "%s: nnz = %lld does not fit int32", who, (long long)nnz);
  HGNN_REQUIRE(rowptr != nullptr, HGNN_EINVAL, "%s: rowptr is NULL", who);
  HGNN_REQUIRE(nnz == 0 || (row && col && col_out), HGNN_EINVAL, "%s: row, col or col_out is NULL", who);
  HGNN_REQUIRE(nnz == 0 || (nrows > 0 && ncols > 0), HGNN_EINVAL, "%s: edges in a graph without rows or columns", who);
  SetupStream s(stream);
  if (nnz == 0) {
    HGNN_HIP(hipMemsetAsync(rowptr, 0, sizeof(int) * (size_t(nrows) + 1), s));
    HGNN_HIP(s.wait());
    return HGNN_OK;
  }
  const int row_bits = bits_for(nrows), col_bits = bits_for(ncols), pos_bits = bits_for(nnz);
  const dim3 per_edge(unsigned(ceil_div(nnz, kBlock)));
  const size_t E = size_t(nnz);
  DevTemp buf[2] = {DevTemp(s), DevTemp(s)}, ids[2] = {DevTemp(s), DevTemp(s)}, bad(s), tmp(s);
  HostMail mail(s);
  size_t tmp_bytes = 0;
  int hbad = 0;
  // the list position rides in the key where it fits (or is not asked for), else beside it
  const bool packed = !eid || row_bits + col_bits + pos_bits <= 64;
  const int in_key = packed && eid ? pos_bits : 0;
  const unsigned first = unsigned(in_key), last = first + unsigned(row_bits + col_bits);
  // the flag is host memory where there is a slot: one copy and one fill less
  int* flag = reinterpret_cast<int*>(mail.data);
  hipError_t e = hipSuccess;
  if (flag) *flag = 0;
  else e = bad.alloc(4);
  for (int i = 0; i < 2 && e == hipSuccess; ++i) e = buf[i].alloc(8 * E);
  for (int i = 0; i < 2 && e == hipSuccess && !packed; ++i) e = ids[i].alloc(4 * E);
  rocprim::double_buffer<uint64_t> keys(buf[0].as<uint64_t>(), buf[1].as<uint64_t>());
  rocprim::double_buffer<int> order(ids[0].as<int>(), ids[1].as<int>());
  auto sort_pairs = [&](void* t) { return rocprim::radix_sort_pairs(t, tmp_bytes, keys, order, unsigned(E), first, last, s); };
  if (packed) tmp_bytes = sort_scratch_bytes(nnz);
  else if (e == hipSuccess) e = sort_pairs(nullptr);
  if (e == hipSuccess) e = tmp.alloc(tmp_bytes);
  if (e == hipSuccess && !flag) e = hipMemsetAsync(bad.p, 0, 4, s);
  if (e == hipSuccess) {
    const CooWords src{row, col, nrows, ncols, col_bits, in_key, flag ? flag : bad.as<int>()};
    const uint64_t* words = nullptr;
    if (packed) {
      words = sort_words(src, nnz, int(first), int(last), buf[0].as<uint64_t>(), buf[1].as<uint64_t>(), tmp.p, s);
    } else {
      coo_keys_kernel<<<per_edge, kBlock, 0, s>>>(src, nnz, keys.current(), order.current());
      e = sort_pairs(tmp.p);
      words = keys.current();
    }
    if (e == hipSuccess) {
      launch_split_words(words, nnz, in_key, col_bits, row_bits, nrows, col_out, packed ? eid : nullptr, rowptr, s);
      e = hipGetLastError();
    }
  }
  if (e == hipSuccess && !packed) e = hipMemcpyAsync(eid, order.current(), 4 * E, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && !flag) e = hipMemcpyAsync(&hbad, bad.p, 4, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = s.wait();
  if (e != hipSuccess) return fail(e == hipErrorOutOfMemory ? HGNN_ENOMEM : HGNN_EHIP, "%s: %s", who, hipGetErrorString(e));
  if (flag) hbad = *static_cast<volatile const int*>(flag);
  if (hbad) return fail(HGNN_EINVAL, "%s: a row id outside [0, nrows) or a column id outside [0, ncols)", who);
  return HGNN_OK;
}

extern "C" hgnn_status hgnn_edge_to_transposed(const hgnn_csr* gt, int32_t H, const hgnn_half* t, hgnn_half* t_T,
                                               void* stream) {
  clear_error();
  const char* who = "hgnn_edge_to_transposed";
  hgnn_status st = check_csr_args(gt, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(gt->eid != nullptr, HGNN_EINVAL, "%s: the graph carries no edge-id map", who);
  HGNN_REQUIRE(H >= 1, HGNN_EINVAL, "%s: H = %d must be positive", who, H);
  if (gt->nnz == 0) return HGNN_OK;
  HGNN_REQUIRE(t != nullptr && t_T != nullptr, HGNN_EINVAL, "%s: t or t_T is NULL", who);
  HGNN_REQUIRE(t != t_T, HGNN_EINVAL, "%s: the permutation cannot run in place", who);
  const int64_t total = gt->nnz * H;
  edge_gather_kernel<<<dim3(unsigned(ceil_div(total, kBlock))), kBlock, 0, static_cast<hipStream_t>(stream)>>>(
      gt->eid, total, H, reinterpret_cast<const half_t*>(t), reinterpret_cast<half_t*>(t_T));
  HGNN_LAUNCH_CHECK("edge_gather_kernel");
  return HGNN_OK;
}

extern "C" hgnn_status hgnn_scale_rows(int64_t n, int32_t F, const hgnn_half* X, int64_t ldx, const float* scale,
                                       hgnn_half* out, int64_t ldo, void* stream) {
  clear_error();
  const char* who = "hgnn_scale_rows";
  HGNN_REQUIRE(n >= 0 && F > 0, HGNN_EINVAL, "%s: n = %lld, F = %d", who, static_cast<long long>(n), F);
  HGNN_REQUIRE(ldx >= F && ldo >= F, HGNN_EINVAL, "%s: leading dimension smaller than F", who);
  if (n == 0) return HGNN_OK;
  HGNN_REQUIRE(X && scale && out, HGNN_EINVAL, "%s: NULL argument", who);
  HGNN_REQUIRE(ldx % 8 == 0 && ldo % 8 == 0 && aligned16(X) && aligned16(out), HGNN_EUNSUPPORTED,
               "%s: needs ld %% 8 == 0 and 16-byte aligned X, out (rows are moved in 16-byte pieces up to the pitch)", who);
  const int F8 = (F + 7) / 8;
  scale_rows_kernel<<<dim3(unsigned(ceil_div(n * F8, kBlock))), kBlock, 0, static_cast<hipStream_t>(stream)>>>(
      n, F8, reinterpret_cast<const half_t*>(X), ldx, scale, reinterpret_cast<half_t*>(out), ldo);
  HGNN_LAUNCH_CHECK("scale_rows_kernel");
  return HGNN_OK;
}

// CSR of the transposed graph plus the edge-id map, for the backward SpMM dX <- A_w^T dY
// (paper section 2.1.2), and CSR from a COO edge list (section 2.1.1).  One-off set-up: a stable radix sort of
// the non-zeros by column id, or by (row id, column id) (rocPRIM's device radix sort is the library step), then
// offsets by binary search.
#include <string.h>

#include <rocprim/device/device_radix_sort.hpp>

#include "common.h"

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

// COO -> CSR: key = (row, col, list position) packed into one 64-bit word (position_bits = 0: without it), so that one
// stable sort of the leading fields orders the edges by row, then column, then position in the list; bad receives 1 when
// an id is out of range (such an edge gets row and column 0)
__global__ void coo_keys_kernel(const int* __restrict__ row, const int* __restrict__ col, int64_t nnz, int nrows, int ncols, int col_bits,
                                int position_bits, uint64_t* __restrict__ keys, int* __restrict__ ids, int* __restrict__ bad) {
  int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= nnz) return;
  const int r = row[k], c = col[k];
  const bool ok = r >= 0 && r < nrows && c >= 0 && c < ncols;
  if (!ok) atomicOr(bad, 1);
  const uint64_t rc = ok ? (uint64_t(uint32_t(r)) << col_bits) | uint64_t(uint32_t(c)) : 0;
  keys[k] = position_bits ? (rc << position_bits) | uint64_t(k) : rc;
  if (ids) ids[k] = int(k);
}

__global__ void coo_split_kernel(const uint64_t* __restrict__ keys, int64_t nnz, int col_bits, int position_bits,
                                 int* __restrict__ col_out, int* __restrict__ eid) {
  int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= nnz) return;
  const uint64_t key = keys[k];
  col_out[k] = int(uint32_t(key >> position_bits) & ((uint32_t(1) << col_bits) - 1u));
  if (eid) eid[k] = int(uint32_t(key) & ((uint32_t(1) << position_bits) - 1u));
}

// The row of every non-zero, handed to put(k, row): a workgroup takes kExpand consecutive positions, its rows mark the slot
// of their first non-zero in LDS and a running maximum spreads the ids (a search of the offset array per non-zero took
// 196 us at 5.5 M non-zeros).  A graph may come here before anything has looked at its offset array: whatever that holds, reads
// stay inside its nrows + 1 entries and marks inside the tile (the rows are then wrong, as the array is).
constexpr int kExpandPerThread = 8;
constexpr int kExpand = kBlock * kExpandPerThread;

template <class Put>
__device__ __forceinline__ void expand_rows(const int* __restrict__ rowptr, int nrows, int64_t nnz, Put&& put) {
  __shared__ int s_row[kExpand];
  __shared__ int s_max[kBlock / kWave], s_lim[2];
  const int64_t e0 = int64_t(blockIdx.x) * kExpand;
  const int n = int(nnz - e0 < kExpand ? nnz - e0 : kExpand);
  if (threadIdx.x < 2) s_lim[threadIdx.x] = row_of_edge(rowptr, nrows, threadIdx.x == 0 ? e0 : e0 + n - 1);
  for (int i = threadIdx.x; i < kExpand; i += kBlock) s_row[i] = -1;
  __syncthreads();
  const int lo = max(s_lim[0], 0), hi = min(s_lim[1], nrows - 1);
  for (int r = lo + 1 + int(threadIdx.x); r <= hi; r += kBlock) {
    const int p = rowptr[r];
    const int64_t at = int64_t(p) - e0;
    if (rowptr[r + 1] > p && at >= 0 && at < n) s_row[at] = r;
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  int v[kExpandPerThread], run = lo;
#pragma unroll
  for (int j = 0; j < kExpandPerThread; ++j) {
    run = max(run, s_row[threadIdx.x * kExpandPerThread + j]);
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
  for (int j = 0; j < kExpandPerThread; ++j) s_row[threadIdx.x * kExpandPerThread + j] = max(v[j], excl);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kBlock) put(e0 + i, s_row[i]);
}

// transposition keys: (column, row, position) packed into one word; sorting the columns' bits brings everything along
__global__ __launch_bounds__(kBlock) void transpose_keys_kernel(const int* __restrict__ rowptr, const int* __restrict__ col, int nrows,
                                                                int64_t nnz, int row_bits, int position_bits,
                                                                uint64_t* __restrict__ keys) {
  expand_rows(rowptr, nrows, nnz, [&](int64_t k, int r) {
    keys[k] = (((uint64_t(uint32_t(col[k])) << row_bits) | uint64_t(uint32_t(r))) << position_bits) | uint64_t(k);
  });
}

__global__ void transpose_split_kernel(const uint64_t* __restrict__ keys, int64_t nnz, int row_bits, int position_bits,
                                       int* __restrict__ col_T, int* __restrict__ eid_T) {
  int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= nnz) return;
  const uint64_t key = keys[k];
  eid_T[k] = int(uint32_t(key) & ((uint32_t(1) << position_bits) - 1u));
  col_T[k] = int(uint32_t(key >> position_bits) & ((uint32_t(1) << row_bits) - 1u));
}

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

// Sort of 64-bit words by the bits [first, last), workgroups of 1024 lanes with eight words each.  A pass moves every word
// once however many bits it takes (43 us for 5.5 M words), so digits of nine bits where they save a pass over digits of
// eight: 36 bits in four passes instead of five, 18 in two instead of three (5.5 M edges: list to CSR 330 -> 280 us,
// transpose 235 -> 183).
// Below 200 000 words a sort by merging is faster where a list takes four passes (us, merging / digits: list to CSR 0.05 M 88 / 121,
// 0.13 M 102 / 125, 0.2 M 114 / 129, 0.4 M 167 / 136; transpose, two passes, 82 / 92, 101 / 90, 109 / 89, 165 / 95).
static hipError_t sort_words(void* tmp, size_t& tmp_bytes, rocprim::double_buffer<uint64_t>& keys, unsigned n, unsigned first,
                             unsigned last, hipStream_t s) {
  using rocprim::default_config;
  using rocprim::kernel_config;
  constexpr auto rank = rocprim::block_radix_rank_algorithm::match;
  using Eight = rocprim::radix_sort_onesweep_config<kernel_config<512, 12>, kernel_config<1024, 8>, 8, rank>;
  using Nine = rocprim::radix_sort_onesweep_config<kernel_config<512, 12>, kernel_config<1024, 8>, 9, rank>;
  constexpr size_t merge_below = 200000;
  const unsigned bits = last - first;
  if ((bits + 8) / 9 < (bits + 7) / 8)
    return rocprim::radix_sort_keys<rocprim::radix_sort_config<default_config, default_config, Nine, merge_below>>(tmp, tmp_bytes, keys, n, first, last, s);
  return rocprim::radix_sort_keys<rocprim::radix_sort_config<default_config, default_config, Eight, merge_below>>(tmp, tmp_bytes, keys, n, first, last, s);
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
    rocprim::double_buffer<uint64_t> keys(buf[0].as<uint64_t>(), buf[1].as<uint64_t>());
    const unsigned first = unsigned(row_bits + pos_bits), last = first + unsigned(col_bits);
    if (e == hipSuccess) e = sort_words(nullptr, tmp_bytes, keys, unsigned(E), first, last, s);
    if (e == hipSuccess) e = tmp.alloc(tmp_bytes);
    if (e == hipSuccess) {
      transpose_keys_kernel<<<per_tile, kBlock, 0, s>>>(g->rowptr, g->col, g->nrows, E, row_bits, pos_bits, keys.current());
      e = sort_words(tmp.p, tmp_bytes, keys, unsigned(E), first, last, s);
    }
    if (e == hipSuccess) {
      transpose_split_kernel<<<per_edge, kBlock, 0, s>>>(keys.current(), E, row_bits, pos_bits, col_T, eid_T);
      offsets_kernel<uint64_t><<<per_col, kBlock, 0, s>>>(keys.current(), int(first), E, g->ncols, rowptr_T);
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
  const dim3 per_edge(unsigned(ceil_div(nnz, kBlock))), per_row(unsigned(ceil_div(int64_t(nrows) + 1, kBlock)));
  const size_t E = size_t(nnz);
  DevTemp buf[2] = {DevTemp(s), DevTemp(s)}, ids[2] = {DevTemp(s), DevTemp(s)}, bad(s), tmp(s);
  HostMail mail(s);
  size_t tmp_bytes = 0;
  int hbad = 0;
  // the list position rides in the key where it fits (or is not asked for), else beside it
  const bool packed = !eid || row_bits + col_bits + pos_bits <= 64;
  const int in_key = packed && eid ? pos_bits : 0;
  const unsigned first = unsigned(in_key), last = first + unsigned(row_bits + col_bits);
  hipError_t e = bad.alloc(4);
  for (int i = 0; i < 2 && e == hipSuccess; ++i) e = buf[i].alloc(8 * E);
  for (int i = 0; i < 2 && e == hipSuccess && !packed; ++i) e = ids[i].alloc(4 * E);
  rocprim::double_buffer<uint64_t> keys(buf[0].as<uint64_t>(), buf[1].as<uint64_t>());
  rocprim::double_buffer<int> order(ids[0].as<int>(), ids[1].as<int>());
  auto sort = [&](void* t) {
    return packed ? sort_words(t, tmp_bytes, keys, unsigned(E), first, last, s)
                  : rocprim::radix_sort_pairs(t, tmp_bytes, keys, order, unsigned(E), first, last, s);
  };
  if (e == hipSuccess) e = sort(nullptr);
  if (e == hipSuccess) e = tmp.alloc(tmp_bytes);
  if (e == hipSuccess) e = hipMemsetAsync(bad.p, 0, 4, s);
  if (e == hipSuccess) {
    coo_keys_kernel<<<per_edge, kBlock, 0, s>>>(row, col, nnz, nrows, ncols, col_bits, in_key, keys.current(),
                                                packed ? nullptr : order.current(), bad.as<int>());
    e = sort(tmp.p);
  }
  if (e == hipSuccess) {
    coo_split_kernel<<<per_edge, kBlock, 0, s>>>(keys.current(), nnz, col_bits, in_key, col_out, packed ? eid : nullptr);
    offsets_kernel<uint64_t><<<per_row, kBlock, 0, s>>>(keys.current(), in_key + col_bits, nnz, nrows, rowptr);
    e = hipGetLastError();
  }
  if (e == hipSuccess && !packed) e = hipMemcpyAsync(eid, order.current(), 4 * E, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = hipMemcpyAsync(mail.data ? static_cast<void*>(mail.data) : &hbad, bad.p, 4, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = s.wait();
  if (e != hipSuccess) return fail(e == hipErrorOutOfMemory ? HGNN_ENOMEM : HGNN_EHIP, "%s: %s", who, hipGetErrorString(e));
  if (mail.data) hbad = *reinterpret_cast<const int*>(mail.data);
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

// Column blocking of the SpMM for feature tables that miss an XCD's L2 but fit the Infinity Cache.
//
// The gather of neighbour rows is what bounds the SpMM (paper section 6.2: "not compute-bound");
// on MI355X each XCD has a private 4 MB L2, so a table of tens of MB is re-fetched over the fabric
// for almost every non-zero.  The plan therefore may cut the columns into nb blocks: block b keeps,
// as a CSR of its own, the non-zeros whose column lies in [b*width, (b+1)*width).  Because columns
// ascend inside a row, a block's share of a row is a contiguous piece of that row.  The SpMM then
// runs block after block -- all compute units gather from the same slice of the table at the same
// time, which the L2s can hold -- over the row tasks of every block into a per-block partial output,
// and one pass adds the nb partials of every row (no atomics).
// One-off set-up code; rocPRIM's device scan is the library step.
#include <string.h>

#include <algorithm>

#include <rocprim/device/device_scan.hpp>

#include "common.h"

namespace hgnn {

// cut[r*(nb+1) + b] = first CSR position of row r whose column is >= b*width (b = nb: end of the row)
__global__ void block_cuts_kernel(const int* __restrict__ rowptr, const int* __restrict__ col, int nrows, int nb, int width,
                                  int* __restrict__ cut) {
  const int64_t idx = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (idx >= int64_t(nrows) * (nb + 1)) return;
  const int r = int(idx / (nb + 1)), b = int(idx % (nb + 1));
  int lo = rowptr[r], hi = rowptr[r + 1];
  if (b < nb) {
    const int64_t key = int64_t(b) * width;
    while (lo < hi) {
      const int mid = lo + ((hi - lo) >> 1);
      if (col[mid] < key) lo = mid + 1;
      else hi = mid;
    }
  } else {
    lo = hi;
  }
  cut[idx] = lo;
}

// cnt[b*nrows + r] = number of non-zeros of row r in block b
__global__ void block_counts_kernel(const int* __restrict__ cut, int nrows, int nb, int* __restrict__ cnt) {
  const int64_t idx = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (idx >= int64_t(nrows) * nb) return;
  const int b = int(idx / nrows), r = int(idx % nrows);
  cnt[idx] = cut[int64_t(r) * (nb + 1) + b + 1] - cut[int64_t(r) * (nb + 1) + b];
}

// goff = exclusive scan of cnt (block-major); brp[b][r] = goff[b*nrows + r] - goff[b*nrows]
__global__ void block_rowptr_kernel(const int* __restrict__ goff, int nrows, int nb, int64_t nnz, int* __restrict__ brp) {
  const int64_t idx = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (idx >= int64_t(nb) * (nrows + 1)) return;
  const int b = int(idx / (nrows + 1)), r = int(idx % (nrows + 1));
  const int64_t base = goff[int64_t(b) * nrows];
  const int64_t here = r < nrows ? goff[int64_t(b) * nrows + r] : (b + 1 < nb ? goff[int64_t(b + 1) * nrows] : nnz);
  brp[idx] = int(here - base);
}

// delta[b*nrows + r] = (first CSR position of row r's piece in block b) - (its position inside block b), so that
// the original position of a blocked non-zero is its block position + delta of its row
__global__ void block_delta_kernel(const int* __restrict__ cut, const int* __restrict__ goff, int nrows, int nb,
                                   int* __restrict__ delta) {
  const int64_t idx = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (idx >= int64_t(nrows) * nb) return;
  const int b = int(idx / nrows), r = int(idx % nrows);
  delta[idx] = cut[int64_t(r) * (nb + 1) + b] - (goff[idx] - goff[int64_t(b) * nrows]);
}

// every non-zero k of the graph goes to its block, keeping its place inside the row piece
__global__ void block_fill_kernel(hgnn_csr g, const int* __restrict__ cut, const int* __restrict__ goff, int nb, int width,
                                  int* __restrict__ bcol, uint16_t* __restrict__ bcol16, int* __restrict__ beid) {
  const int64_t k = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (k >= g.nnz) return;
  const int r = row_of_edge(g.rowptr, g.nrows, k);
  const int c = g.col[k];
  const int b = c / width;
  const int64_t dest = int64_t(goff[int64_t(b) * g.nrows + r]) + (k - cut[int64_t(r) * (nb + 1) + b]);
  if (bcol16) bcol16[dest] = uint16_t(c - b * width);
  else bcol[dest] = c;
  if (beid) beid[dest] = g.eid[k];
}

hgnn_status build_col_blocks(hgnn_plan* p, const hgnn_csr* g, int nb, SetupStream& s) {
  const int V = g->nrows;
  const int64_t E = g->nnz;
  const int width = int(ceil_div(g->ncols, nb));
  p->nb = nb;
  p->block_width = width;
  p->block_eid = g->eid != nullptr;
  DevTemp cut_buf(s), cnt_buf(s), goff_buf(s), tmp(s);
  size_t tmp_bytes = 0;
  const size_t n_flat = size_t(nb) * size_t(V);
  hipError_t e = cut_buf.alloc(sizeof(int) * size_t(V) * size_t(nb + 1));
  if (e == hipSuccess) e = cnt_buf.alloc(sizeof(int) * n_flat);
  if (e == hipSuccess) e = goff_buf.alloc(sizeof(int) * n_flat);
  int *const cut = cut_buf.as<int>(), *const cnt = cnt_buf.as<int>(), *const goff = goff_buf.as<int>();
  if (e == hipSuccess) e = dev_malloc(&p->brp, sizeof(int) * size_t(nb) * (size_t(V) + 1));
  if (e == hipSuccess) e = width <= 65536 ? dev_malloc(&p->bcol16, sizeof(uint16_t) * size_t(E)) : dev_malloc(&p->bcol, sizeof(int) * size_t(E));
  if (e == hipSuccess && g->eid) e = dev_malloc(&p->beid, sizeof(int) * size_t(E));
  // partial rows twice over and three scalars per row and head: the fused GAT pass that saves for its backward
  // leaves two vectors and (max, sum, masked sum) per block; row sums of edge tensors use one scalar
  if (e == hipSuccess) e = dev_malloc(&p->bstage, sizeof(hgnn_half) * 2 * n_flat * size_t(p->max_F));
  if (e == hipSuccess) e = dev_malloc(&p->bsum, sizeof(float) * 3 * n_flat * size_t(p->max_H));
  if (e == hipSuccess) e = dev_malloc(&p->bdelta, sizeof(int) * n_flat);
  if (e == hipSuccess) {
    block_cuts_kernel<<<dim3(unsigned(ceil_div(int64_t(V) * (nb + 1), kBlock))), kBlock, 0, s>>>(g->rowptr, g->col, V, nb,
                                                                                                 width, cut);
    block_counts_kernel<<<dim3(unsigned(ceil_div(int64_t(n_flat), kBlock))), kBlock, 0, s>>>(cut, V, nb, cnt);
    e = rocprim::exclusive_scan(nullptr, tmp_bytes, cnt, goff, 0, n_flat, rocprim::plus<int>(), s);
  }
  if (e == hipSuccess) e = tmp.alloc(tmp_bytes);
  if (e == hipSuccess) e = rocprim::exclusive_scan(tmp.p, tmp_bytes, cnt, goff, 0, n_flat, rocprim::plus<int>(), s);
  if (e == hipSuccess) {
    block_rowptr_kernel<<<dim3(unsigned(ceil_div(int64_t(nb) * (V + 1), kBlock))), kBlock, 0, s>>>(goff, V, nb, E, p->brp);
    block_fill_kernel<<<dim3(unsigned(ceil_div(E, kBlock))), kBlock, 0, s>>>(*g, cut, goff, nb, width, p->bcol, p->bcol16, p->beid);
    block_delta_kernel<<<dim3(unsigned(ceil_div(int64_t(n_flat), kBlock))), kBlock, 0, s>>>(cut, goff, V, nb, p->bdelta);
    e = hipGetLastError();
  }
  p->boff.assign(size_t(nb) + 1, 0);
  for (int b = 0; b < nb && e == hipSuccess; ++b) {
    int v = 0;
    e = hipMemcpyAsync(&v, goff + size_t(b) * V, sizeof(int), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = s.wait();
    p->boff[size_t(b)] = v;
  }
  p->boff[size_t(nb)] = E;
  if (e == hipSuccess) e = s.wait();
  if (e != hipSuccess)
    return fail(e == hipErrorOutOfMemory ? HGNN_ENOMEM : HGNN_EHIP, "build_col_blocks: %s", hipGetErrorString(e));
  return HGNN_OK;
}

namespace {

// the cut of a plan whose arrays are there, on the host, block by block
struct HostBlock {
  std::vector<int32_t> rowptr, col, slot;
};

hipError_t fetch_block(const hgnn_plan* c, int b, HostBlock& h) {
  const int64_t off = c->boff[size_t(b)];
  const size_t n = size_t(c->boff[size_t(b) + 1] - off), V = size_t(c->nrows);
  std::vector<int32_t> delta(V);
  std::vector<uint16_t> narrow;
  h.rowptr.resize(V + 1);
  h.col.resize(n);
  h.slot.resize(n);
  auto get = [](void* dst, const void* src, size_t bytes) { return bytes ? hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost) : hipSuccess; };
  hipError_t e = get(h.rowptr.data(), c->brp + size_t(b) * (V + 1), 4 * (V + 1));
  if (c->bcol16) narrow.resize(n);
  if (e == hipSuccess) e = c->bcol16 ? get(narrow.data(), c->bcol16 + off, 2 * n) : get(h.col.data(), c->bcol + off, 4 * n);
  if (e == hipSuccess) e = c->beid ? get(h.slot.data(), c->beid + off, 4 * n) : get(delta.data(), c->bdelta + size_t(b) * V, 4 * V);
  if (e != hipSuccess) return e;
  for (size_t k = 0; k < narrow.size(); ++k) h.col[k] = b * c->block_width + int32_t(narrow[k]);
  if (!c->beid)
    for (size_t r = 0; r < V; ++r)
      for (int32_t k = h.rowptr[r]; k < h.rowptr[r + 1]; ++k) h.slot[size_t(k)] = k + delta[r];
  return hipSuccess;
}

}  // namespace

}  // namespace hgnn

using namespace hgnn;

// A row's piece of block b is put together from the blocks of the cut that the plan holds: its own, or the finer one, whose
// blocks need not end where this one does.
extern "C" hgnn_status hgnn_plan_block_export(const hgnn_plan* p, int32_t b, int64_t* nnz_b, int32_t* rowptr_b, int32_t* col_b,
                                              int32_t* eid_b, int32_t* seg_row_lo, int32_t* seg_row_hi) {
  clear_error();
  const char* who = "hgnn_plan_block_export";
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nb > 1 && b >= 0 && b < p->nb, HGNN_EINVAL, "%s: block %d of %d", who, b, p->nb);
  HGNN_HIP(hipDeviceSynchronize());
  const hgnn_plan* c = p->brp ? p : p->fine;
  const int64_t lo = int64_t(b) * p->block_width, hi = std::min<int64_t>(lo + p->block_width, p->ncols);
  const size_t V = size_t(p->nrows);
  std::vector<HostBlock> parts;
  for (int f = int(lo / c->block_width); f < c->nb && int64_t(f) * c->block_width < hi; ++f) {
    parts.emplace_back();
    HGNN_HIP(fetch_block(c, f, parts.back()));
  }
  HostBlock out;
  out.rowptr.assign(V + 1, 0);
  for (size_t r = 0; r < V; ++r) {
    for (const HostBlock& h : parts)
      for (int32_t k = h.rowptr[r]; k < h.rowptr[r + 1]; ++k)
        if (h.col[size_t(k)] >= lo && h.col[size_t(k)] < hi) {
          out.col.push_back(h.col[size_t(k)]);
          out.slot.push_back(h.slot[size_t(k)]);
        }
    out.rowptr[r + 1] = int32_t(out.col.size());
  }
  const int64_t n = int64_t(out.col.size());
  if (nnz_b) *nnz_b = n;
  if (rowptr_b) std::copy(out.rowptr.begin(), out.rowptr.end(), rowptr_b);
  if (col_b) std::copy(out.col.begin(), out.col.end(), col_b);
  if (eid_b) std::copy(out.slot.begin(), out.slot.end(), eid_b);
  for (int64_t k = 0; k * p->S < n; ++k) {
    if (seg_row_lo) seg_row_lo[k] = row_of_edge(out.rowptr.data(), p->nrows, k * p->S);
    if (seg_row_hi) seg_row_hi[k] = row_of_edge(out.rowptr.data(), p->nrows, std::min<int64_t>((k + 1) * p->S, n) - 1);
  }
  return HGNN_OK;
}

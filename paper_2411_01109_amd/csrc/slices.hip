// Column slices: per-edge passes whose only random access is a per-vertex scalar of the column side.
//
// Two steps of the GAT path read or update one scalar per non-zero at the non-zero's column: the factorised
// score e = LeakyReLU(el[row] + er[col]) (paper section 3.1.2, the SDDMM variant of GAT) gathers er[col], and the
// column sums of the score gradient d(e_r)[j] = sum over the non-zeros of column j (section 2.1.2: the backward
// pass needs the transposed direction) scatter into out[col].  Served by the L2s, either costs one cache request
// per non-zero, and the request rate of the L2s then bounds the pass at a fraction of what streaming the edge
// arrays would take.  On gfx950 a workgroup may hold 160 KB of LDS, enough for the scalars of 16 K columns, so
// the plan can cut the columns into slices of that width: a workgroup loads (or zeroes) the table of one slice
// in LDS and walks the pieces of one chunk of the non-zeros that fall into the slice -- a contiguous piece of
// every row, because columns ascend inside a row -- gathering from / adding into LDS.  What is left in
// memory traffic is the stream of column ids and edge values.
//
// Column sums are accumulated as 64-bit fixed-point integers (an fp16 value is an integer multiple of 2^-24 below
// 2^16 in magnitude, so the conversion is exact), with LDS atomic adds: integer addition is associative, so the
// result does not depend on the order in which the waves arrive (no run-to-run variation), and it is the exact sum,
// rounded once on output.  Every workgroup leaves its slice's partial sums in the plan; a second kernel adds the
// chunks' partials per column.  Non-finite inputs (never produced by the path itself) go through a separate
// fp32 side array so that they still poison their column's sum.
#include "common.h"

#include <algorithm>

namespace hgnn {

constexpr int kSliceThreads = 1024;
constexpr int kSliceWaves = kSliceThreads / kWave;
constexpr int kSliceUnroll = 8;  // row pieces whose loads a wave has in flight together

struct SliceArgs {
  const int* scut;       // [ns+1][nrows]: first CSR position of row r whose column is >= s*W (s = ns: end of the row)
  const int2* share;     // [nch * kSliceWaves + 1] row and position where every wave's share begins
  const int* col;
  int nrows, ncols, ns, nch, W;
  // score (and alpha from lse)
  const float* el;   // [nrows]
  const float* er;   // [ncols]
  const float* lse;  // [nrows] or nullptr
  half_t* out;       // [nnz]
  float slope;
  // column sums
  const half_t* t;            // [nnz]
  unsigned long long* part;   // [nch][ncols]
  float* poison;              // [ncols]
};

// fp16 bit pattern -> value * 2^24 as a 64-bit integer (exact); finite inputs only
__device__ __forceinline__ long long half_bits_to_fixed(unsigned bits) {
  const unsigned ex = (bits >> 10) & 31u, man = bits & 1023u;
  const unsigned long long m = ex ? (man | 1024u) : man;
  const long long v = (long long)(m << (ex ? ex - 1u : 0u));
  return (bits & 0x8000u) ? -v : v;
}

// LDS of a workgroup: the slice's table (W scalars of 4 or 8 bytes), then per wave the bookkeeping of the 64 rows
// it is working on: a bit for each slot of a round, and of every row with a piece its first position less its first slot and, for the
// score, its el and lse
__host__ __device__ inline int slice_wave_bytes(bool colsum) { return 2 * kSliceUnroll * 4 + 64 * (colsum ? 4 : 12); }
__host__ __device__ inline size_t slice_lds_bytes(int W, bool colsum) {
  return size_t(W) * (colsum ? 8 : 4) + size_t(kSliceWaves) * slice_wave_bytes(colsum);
}

template <bool COLSUM>
__global__ __launch_bounds__(kSliceThreads) void edge_slice_kernel(SliceArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* s_er = reinterpret_cast<float*>(smem);
  unsigned long long* s_acc = reinterpret_cast<unsigned long long*>(smem);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  // (W is a multiple of 64)
  unsigned* s_begins = reinterpret_cast<unsigned*>(smem + size_t(a.W) * (COLSUM ? 8 : 4) + size_t(wave) * slice_wave_bytes(COLSUM));
  int* s_row = reinterpret_cast<int*>(s_begins + 2 * kSliceUnroll);  // [64], or pairs of it and el
  float* s_lse = reinterpret_cast<float*>(s_row + 128);
  // workgroup id = slice * nch + chunk, nch a multiple of 8: the slices of one row chunk run on one XCD (workgroups
  // are dealt out to the XCDs in turn), so the cache lines that neighbouring pieces of a row share meet in one L2
  const int s = int(blockIdx.x) / a.nch, c = int(blockIdx.x) % a.nch;
  const int col0 = s * a.W;
  const int wcols = a.ncols - col0 < a.W ? a.ncols - col0 : a.W;
  for (int i = tid; i < wcols; i += kSliceThreads) {
    if (COLSUM) s_acc[i] = 0ull;
    else s_er[i] = a.er[col0 + i];
  }
  __syncthreads();
  // A wave's share may begin and end inside a row: with whole rows, a power law's longest were a wave's work for most of the time (3.5 M
  // non-zeros of 13 292 vertices, score 287 -> 16, column sums 371 -> 28 us; 24 M of 100 000, log-normal, 61 -> 57 and 71 -> 65).  How it is
  // measured: share_begins_kernel.
  const int2 from = a.share[c * kSliceWaves + wave], to = a.share[c * kSliceWaves + wave + 1];
  const int p0 = from.y, p1 = to.y, r0 = from.x, r1 = min(to.x + 1, a.nrows);
  const int* __restrict__ lo = a.scut + size_t(s) * size_t(a.nrows);
  const int* __restrict__ hi = lo + a.nrows;
  const unsigned short* __restrict__ tbits = reinterpret_cast<const unsigned short*>(a.t);

  // A wave takes 64 rows at a time.  The non-zeros of their pieces of this slice are numbered through and dealt out to the lanes in
  // turn, so that every load instruction moves 64 non-zeros whatever the lengths of the pieces.  The loads run one round ahead of the work: while the
  // non-zeros of a round (8 x 64 slots) are scored or added, the column ids and values of the next round are on their way; the row bounds of the next
  // 64 rows are requested when a batch begins.
  // Slots beyond the batch's total repeat its last slot (a valid position): for the score that stores the same value
  // twice, for the sums the repeated value is replaced by zero.  The row of a slot, among those that have a piece, is the number of pieces that
  // begin behind the first slot and not behind this one: their first slots, less one, are set as bits, which a lane counts below its own.  A binary
  // search over the prefix values, six LDS reads in turn and some 24 vector instructions per slot, was half of the kernel.  us, score; column sums,
  // with it / now, on one machine: 114 M log-normal 236; 241 / 224; 209, 24 M of 100 000 log-normal 56; 64 / 42; 52, 20 M power law of 100 000 118; 142 / 88; 114, 8 M of
  // 30 000 uniform 23.3; 29.6 / 18.9; 26.4.  The largest are bound by the memory's lines now, of which neighbouring pieces share many (3.2 and 3.3 TB/s; on another machine 218; 203).
  auto plan_round = [&](pos_t qb, pos_t total, pos_t begin, bool has, unsigned& before, int (&kk)[kSliceUnroll], int (&jj)[kSliceUnroll]) {
    if (lane < 2 * kSliceUnroll) s_begins[lane] = 0u;
    wave_sync();
    const pos_t at = begin - 1 - qb;  // (the first piece of a batch begins at slot 0 and is not counted)
    if (has && at < pos_t(kWave * kSliceUnroll)) atomicOr(s_begins + (at >> 5), 1u << (at & 31u));
    wave_sync();
#pragma unroll
    for (int u = 0; u < kSliceUnroll; ++u) {
      const uint2 m = *reinterpret_cast<const uint2*>(s_begins + 2 * u);
      jj[u] = int(__builtin_amdgcn_mbcnt_hi(m.y, __builtin_amdgcn_mbcnt_lo(m.x, before)));
      before += unsigned(__popc(m.x) + __popc(m.y));
    }
#pragma unroll
    for (int u = 0; u < kSliceUnroll; ++u) {
      const pos_t q = qb + pos_t(u * kWave + lane);
      kk[u] = int(q < total ? q : total - 1);
    }
  };
  // position = slot + (first position - first slot) of the row; the score takes the row's el (as bits) along
  auto issue = [&](int (&kk)[kSliceUnroll], const int (&jj)[kSliceUnroll], int (&cc)[kSliceUnroll], unsigned (&tt)[kSliceUnroll]) {
#pragma unroll
    for (int u = 0; u < kSliceUnroll; ++u) {
      if (COLSUM) {
        kk[u] += s_row[jj[u]];
      } else {
        const uint2 r = reinterpret_cast<const uint2*>(s_row)[jj[u]];
        kk[u] += int(r.x);
        tt[u] = r.y;
      }
    }
#pragma unroll
    for (int u = 0; u < kSliceUnroll; ++u) {
      cc[u] = a.col[kk[u]];  // ordinary loads: the lines that pieces share are met again in the L1 and the L2
      if (COLSUM) tt[u] = tbits[kk[u]];
    }
  };
  auto work = [&](pos_t q0, pos_t total, const int (&kk)[kSliceUnroll], const int (&jj)[kSliceUnroll], const int (&cc)[kSliceUnroll],
                  const unsigned (&tt)[kSliceUnroll]) {
#pragma unroll
    for (int u = 0; u < kSliceUnroll; ++u) {
      const int cidx = cc[u] - col0;
      if (COLSUM) {
        const unsigned tb = q0 + u * kWave < total ? tt[u] : 0u;
        if (((tb >> 10) & 31u) == 31u) {  // inf / nan: through the side array
          atomicAdd(a.poison + col0 + cidx, float(a.t[kk[u]]));
        } else if (tb & 0x7fffu) {
          atomicAdd(s_acc + cidx, (unsigned long long)half_bits_to_fixed(tb));
        }
      } else {
        float v = __uint_as_float(tt[u]) + s_er[cidx];
        v = v > 0.f ? v : a.slope * v;
        if (a.lse) v = __expf(v - s_lse[jj[u]]);
        a.out[kk[u]] = half_t(v);
      }
    }
  };
  auto bounds = [&](int base, int& b, int& e, float& elv, float& lsev) {
    const int r = base + lane;
    const bool in = r < r1;
    b = in ? max(lo[r], p0) : 0;
    e = in ? max(min(hi[r], p1), b) : 0;
    elv = lsev = 0.f;
    if (!COLSUM && in) {
      elv = a.el[r];
      if (a.lse) lsev = a.lse[r];
    }
  };
  int nb_ = 0, ne_ = 0;
  float nel = 0.f, nlse = 0.f;
  bounds(r0, nb_, ne_, nel, nlse);
  for (int base = r0; base < r1; base += kWave) {
    const int b = nb_, e = ne_;
    const float elv = nel, lsev = nlse;
    if (base + kWave < r1) bounds(base + kWave, nb_, ne_, nel, nlse);  // for the next batch
    int inc = e - b;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int t = __shfl_up(inc, d);
      if (lane >= d) inc += t;
    }
    const pos_t total = pos_t(__shfl(inc, kWave - 1));
    const pos_t begin = pos_t(inc - (e - b));
    const bool has = e > b;
    const unsigned long long pieces = __ballot(has);
    const int rank = int(__builtin_amdgcn_mbcnt_hi(unsigned(pieces >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(pieces), 0u)));
    if (has) {
      if (COLSUM) {
        s_row[rank] = b - int(begin);
      } else {
        reinterpret_cast<int2*>(s_row)[rank] = make_int2(b - int(begin), __float_as_int(elv));
        if (a.lse) s_lse[rank] = lsev;
      }
    }
    unsigned before = 0;
    wave_sync();
    int kA[kSliceUnroll], jA[kSliceUnroll], cA[kSliceUnroll], kB[kSliceUnroll], jB[kSliceUnroll], cB[kSliceUnroll];
    unsigned tA[kSliceUnroll], tB[kSliceUnroll];
    if (total > 0) {
      plan_round(0, total, begin, has, before, kA, jA);
      issue(kA, jA, cA, tA);
    }
    for (pos_t qb = 0; qb < total; qb += kWave * kSliceUnroll) {
      const bool more = qb + kWave * kSliceUnroll < total;
      if (more) {
        plan_round(qb + kWave * kSliceUnroll, total, begin, has, before, kB, jB);
        issue(kB, jB, cB, tB);
      }
      work(lane + qb, total, kA, jA, cA, tA);
      if (more) {
#pragma unroll
        for (int u = 0; u < kSliceUnroll; ++u) {
          kA[u] = kB[u];
          jA[u] = jB[u];
          cA[u] = cB[u];
          tA[u] = tB[u];
        }
      }
    }
    wave_sync();  // the wave's bookkeeping is rewritten for the next 64 rows
  }
  if (COLSUM) {
    __syncthreads();
    unsigned long long* dst = a.part + size_t(c) * size_t(a.ncols) + col0;
    for (int i = tid; i < wcols; i += kSliceThreads) dst[i] = s_acc[i];
  }
}

// out[j] = fp16(sum over the chunks of their partial sums of column j); the side array of non-finite inputs is
// added and cleared.  64 columns a workgroup, whose waves take a share of the chunks each: bound by the latency of a wave's loads
// (16 chunks of 233 k columns, 4 / 16 waves: 8.2 / 12.0 us).
__global__ __launch_bounds__(kSliceThreads) void colsum_reduce_kernel(const unsigned long long* __restrict__ part, int nch, int ncols,
                                                                      float* __restrict__ poison, half_t* __restrict__ out) {
  __shared__ unsigned long long sums[kSliceWaves][kWave];
  const int x = threadIdx.x & (kWave - 1), y = threadIdx.x / kWave, waves = blockDim.x / kWave, j = blockIdx.x * kWave + x;
  unsigned long long mine = 0;
  if (j < ncols) {
#pragma unroll 8
    for (int c = y; c < nch; c += waves) mine += part[size_t(c) * size_t(ncols) + j];
  }
  sums[y][x] = mine;
  __syncthreads();
  if (y > 0 || j >= ncols) return;
  mine = 0;
  for (int w = 0; w < waves; ++w) mine += sums[w][x];
  double v = double((long long)mine) * (1.0 / 16777216.0);
  const float p = poison ? poison[j] : 0.f;
  if (p != 0.f) {  // also true for nan
    v += double(p);
    poison[j] = 0.f;
  }
  out[j] = half_t(float(v));
}

// scut[s*nrows + r] = first CSR position of row r whose column is >= s*W (s = ns: end of the row)
__global__ void slice_cuts_kernel(const int* __restrict__ rowptr, const int* __restrict__ col, int nrows, int ns, int W,
                                  int* __restrict__ scut) {
  const int64_t idx = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (idx >= int64_t(nrows) * (ns + 1)) return;
  const int s = int(idx / nrows), r = int(idx % nrows);
  int lo = rowptr[r], hi = rowptr[r + 1];
  if (s < ns) {
    const int64_t key = int64_t(s) * W;
    while (lo < hi) {
      const int mid = lo + ((hi - lo) >> 1);
      if (col[mid] < key) lo = mid + 1;
      else hi = mid;
    }
  } else {
    lo = hi;
  }
  scut[idx] = lo;
}

// A share is as much as every other, a row counted as kRowCost non-zeros, which its bounds cost whether it has any or not: of non-zeros alone, a
// wave walked a long stretch of empty rows by itself: 16 M non-zeros, half of 1 M rows empty one after the other, score 4654 -> 39, column sums 4395 ->
// 47 us; the same without those rows 36.8 -> 33.6 and 45.2 -> 42.5, 24 M of 100 000, log-normal, 56.0 -> 54.2 and 66.6 -> 65.4.
constexpr int64_t kRowCost = 4;
inline __host__ __device__ int64_t slice_cost(int64_t nrows, int64_t nnz) { return nnz + kRowCost * nrows; }

__global__ void share_begins_kernel(const int* __restrict__ rowptr, int nrows, int64_t nnz, int shares, int2* __restrict__ begin) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c > shares) return;
  const int64_t target = slice_cost(nrows, nnz) * c / shares;
  int lo = 0, hi = nrows;  // rows that begin at or before it
  while (lo < hi) {
    const int mid = lo + ((hi - lo) >> 1);
    if (slice_cost(mid, rowptr[mid]) <= target) lo = mid + 1;
    else hi = mid;
  }
  const int r = max(lo - 1, 0);
  begin[c] = make_int2(r, int(min(target - kRowCost * r, int64_t(rowptr[r + 1]))));
}

hgnn_status build_col_slices(hgnn_plan* p, const hgnn_csr* g, int W, bool asked, SetupStream& s) {
  // slices of an earlier call may still be in use by calls on the plan, on whatever stream
  const bool idle = p->scut == nullptr || device_idle(p->device);
  dev_put(p->scut, idle);
  dev_put(p->slice_share, idle);
  dev_put(p->col_part, idle);
  dev_put(p->col_poison, idle);
  p->scut = nullptr;
  p->slice_share = nullptr;
  p->col_part = nullptr;
  p->col_poison = nullptr;
  p->ns = 0;
  if (g->nrows == 0 || g->ncols == 0) return HGNN_OK;
  int dev = 0, cus = 256;
  HGNN_HIP(hipGetDevice(&dev));
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8) cus = 256;
  const int ns = int(ceil_div(g->ncols, W));
  W = int(ceil_div(ceil_div(g->ncols, ns), 64) * 64);  // the same number of slices, of equal width (a short last slice would idle its compute units)
  // one workgroup per compute unit at a time (its LDS table fills most of the 160 KB): as many chunks as give
  // every compute unit one (slice, chunk) pair, a multiple of 8 so that a chunk's slices share an XCD, and not so
  // many that a wave has less than a round of a slice's non-zeros or rows
  int nch = 8 * std::max(1, (cus / 8) / ns);
  const int64_t by_work = 8 * std::max<int64_t>(1, slice_cost(g->nrows, g->nnz) / (int64_t(8) * kSliceThreads * kSliceUnroll * ns));
  if (nch > by_work) nch = int(by_work);
  const int shares = nch * kSliceWaves;
  HGNN_HIP(dev_malloc(&p->scut, sizeof(int) * size_t(ns + 1) * size_t(g->nrows)));
  HGNN_HIP(dev_malloc(&p->slice_share, sizeof(int2) * (size_t(shares) + 1)));
  HGNN_HIP(dev_malloc(&p->col_part, sizeof(unsigned long long) * size_t(nch) * size_t(g->ncols)));
  HGNN_HIP(dev_malloc(&p->col_poison, sizeof(float) * size_t(g->ncols)));
  HGNN_HIP(hipMemsetAsync(p->col_poison, 0, sizeof(float) * size_t(g->ncols), s));
  slice_cuts_kernel<<<dim3(unsigned(ceil_div(int64_t(g->nrows) * (ns + 1), kBlock))), kBlock, 0, s>>>(g->rowptr, g->col, g->nrows,
                                                                                                    ns, W, p->scut);
  share_begins_kernel<<<dim3(unsigned(ceil_div(shares + 1, kBlock))), kBlock, 0, s>>>(g->rowptr, g->nrows, g->nnz, shares, p->slice_share);
  HGNN_LAUNCH_CHECK("slice_cuts_kernel / share_begins_kernel");
  HGNN_HIP(s.wait());
  // Scores gather through the caches just as well where there are few: us, segments / slices, 1 M non-zeros of 13 292 vertices 8.4 / 14.0, 1.2 M of
  // 4000 8.3 / 11.8, 3 M of 30 000 17.4 / 16.3, 3.5 M of 13 292 14.0 / 16.0, 5.4 M of 20 000 22.0 / 22.2, 6 M of 60 000 32.6 / 23.0 (power law 26.0 / 34.3), 8 M
  // of 30 000 33.8 / 27.9, 20 M of 16 000 53.4 / 39.7, 24 M of 100 000 103 / 57 (slices by a binary search per non-zero; now 6 M power law 27.5, 8 M of
  // 30 000 18.9, 24 M of 100 000 42, 1 M of 13 292 10.2).  Column sums have no other way.
  constexpr int64_t kScoreNnz = int64_t(4) << 20;
  p->slice_scores = asked || g->nnz > kScoreNnz;
  p->ns = ns;
  p->slice_w = W;
  p->nch = nch;
  return HGNN_OK;
}

static SliceArgs slice_args(const hgnn_plan* p, const hgnn_csr* g) {
  SliceArgs a{};
  a.scut = p->scut;
  a.share = p->slice_share;
  a.col = g->col;
  a.nrows = g->nrows;
  a.ncols = g->ncols;
  a.ns = p->ns;
  a.nch = p->nch;
  a.W = p->slice_w;
  return a;
}

template <bool COLSUM>
static hgnn_status launch_slices(const hgnn_plan* p, const SliceArgs& a, hipStream_t s) {
  const size_t lds = slice_lds_bytes(a.W, COLSUM);
  // beyond 64 KB of dynamic LDS the runtime wants to be told, once per kernel and device
  static bool told[64][2] = {};
  int dev = 0;
  HGNN_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64 || !told[dev][COLSUM ? 1 : 0]) {
    HGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&edge_slice_kernel<COLSUM>),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(slice_lds_bytes(kSliceMaxCols, true))));
    if (dev >= 0 && dev < 64) told[dev][COLSUM ? 1 : 0] = true;
  }
  edge_slice_kernel<COLSUM><<<dim3(unsigned(p->ns) * unsigned(p->nch)), kSliceThreads, lds, s>>>(a);
  HGNN_LAUNCH_CHECK("edge_slice_kernel");
  return HGNN_OK;
}

// e[k] = LeakyReLU(el[row k] + er[col k]) (one head), or alpha = exp(e - lse[row]) when lse is given, over the plan's
// column slices
hgnn_status slice_edge_score(const hgnn_plan* p, const hgnn_csr* g, const float* el, const float* er, const float* lse,
                             float slope, hgnn_half* out, hipStream_t s) {
  SliceArgs a = slice_args(p, g);
  a.el = el;
  a.er = er;
  a.lse = lse;
  a.slope = slope;
  a.out = reinterpret_cast<half_t*>(out);
  return launch_slices<false>(p, a, s);
}

}  // namespace hgnn

using namespace hgnn;

extern "C" {

hgnn_status hgnn_plan_add_slices(hgnn_plan* p, const hgnn_csr* g, int32_t slice_cols, void* stream) {
  clear_error();
  const char* who = "hgnn_plan_add_slices";
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(slice_cols == 0 || (slice_cols >= 64 && slice_cols <= kSliceMaxCols), HGNN_EINVAL,
               "%s: slice_cols = %d outside [64, %d] (0 = default)", who, slice_cols, kSliceMaxCols);
  SetupStream s(stream);
  return build_col_slices(p, g, slice_cols == 0 ? kSliceMaxCols : slice_cols, true, s);
}

int32_t hgnn_plan_num_slices(const hgnn_plan* p) { return p ? p->ns : 0; }

hgnn_status hgnn_edge_colsum(const hgnn_csr* g, const hgnn_plan* p, int32_t H, const hgnn_half* t, hgnn_half* out,
                             void* stream) {
  clear_error();
  const char* who = "hgnn_edge_colsum";
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(H >= 1, HGNN_EINVAL, "%s: H = %d must be positive", who, H);
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EUNSUPPORTED, "%s: an edge-id map is not supported here", who);
  HGNN_REQUIRE(H == 1, HGNN_EUNSUPPORTED, "%s: one head only (use hgnn_edge_rowsum on the transposed graph)", who);
  HGNN_REQUIRE(p->ns > 0 || g->ncols == 0 || g->nrows == 0, HGNN_EINVAL,
               "%s: the plan holds no column slices (hgnn_plan_add_slices)", who);
  if (g->ncols == 0) return HGNN_OK;
  HGNN_REQUIRE(out != nullptr && (g->nnz == 0 || t != nullptr), HGNN_EINVAL, "%s: t or out is NULL", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (g->nrows == 0) {  // no rows, hence no slices: every column sum is zero
    colsum_reduce_kernel<<<dim3(unsigned(ceil_div(g->ncols, kWave))), kWave, 0, s>>>(nullptr, 0, g->ncols, nullptr,
                                                                                       reinterpret_cast<half_t*>(out));
    HGNN_LAUNCH_CHECK("colsum_reduce_kernel");
    return HGNN_OK;
  }
  SliceArgs a = slice_args(p, g);
  a.t = reinterpret_cast<const half_t*>(t);
  a.part = p->col_part;
  a.poison = p->col_poison;
  st = launch_slices<true>(p, a, s);
  if (st != HGNN_OK) return st;
  colsum_reduce_kernel<<<dim3(unsigned(ceil_div(g->ncols, kWave))), p->nch <= 64 ? kBlock : kSliceThreads, 0, s>>>(p->col_part, p->nch, g->ncols, p->col_poison,
                                                                                     reinterpret_cast<half_t*>(out));
  HGNN_LAUNCH_CHECK("colsum_reduce_kernel");
  return HGNN_OK;
}

}  // extern "C"

// fp16 CSR SpMM for gfx950 (wave64): the vertex-parallel kernel behind hgnn_spmm and the
// edge-parallel discretized-reduction kernels behind hgnn_spmm_discretized
// (paper sections 2.1.2, 4.1, 5.2).
//
// Lane mapping (the wave64 form of the paper's sub-warps, section 4.1): a feature row of F
// halves is covered by L = pow2 >= F/8 lanes that load 16 bytes (8 halves) each, so a wave
// holds G = 64/L such groups and touches G different neighbour rows per load instruction.
// Products are formed and accumulated in fp32 (v_fma_mix), fp16 only when a value is stored.
#include "task.h"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace hgnn {

struct SpmmArgs {
  const int* rowptr;
  const int* deg_rowptr;  // offset array that defines deg(i) for MEAN (the whole graph's, also when a column block runs)
  const int* col;
  const int* eid;
  const int* delta;  // column blocks of a graph without edge-id map: slot of non-zero k of row r = k + delta[r]
  const half_t* w;  // [nnz][H] or nullptr
  const half_t* X;
  half_t* Y;
  const float* row_scale;
  int64_t ldx, ldy;
  int64_t nnz;
  int nrows;
  int F, H, D;
  uint32_t per_d;  // 2^32 / D, rounded up: f * per_d >> 32 is the head of feature f < 512
  int reduce;
  float one;  // 1.0f
  int rows_per_wave;  // spmm_row_kernel: rows a wave owns, 1 or 64/L
  int long_row;       // plan-free kernels: rows longer than this go to the chunked hub kernels
  // fused scaling and epilogue (discretized kernels): Y = self_coef*self + sum of partials, every partial
  // = agg_coef * s_i * sum_batch w * col_scale[j] * x_j
  const float* col_scale;  // [ncols] or nullptr
  const half_t* self;      // [nrows][ld_self] or nullptr
  int64_t ld_self;
  float self_coef, agg_coef;
  // discretized kernels
  half_t* staging;  // [slots][stage_ld] pieces of the rows that have several
  int stage_ld;
  int stage32;   // 1: the pieces are staged in fp32 (staging is an array of floats)
  int atomic_y;  // 1: conflicting pieces are added to Y with packed fp16 atomics instead of being staged (comparison variant)
  // all column blocks of a plan in one launch: waves are numbered block after block (they are dispatched in that order, so
  // the compute units still gather from one slice of X at a time, without a drain between the blocks)
  int64_t block_y_stride;  // halves between the blocks' partial outputs
};

__device__ __forceinline__ float scale_of(const SpmmArgs& a, int r) {
  float s = 1.f;
  if (a.reduce == HGNN_MEAN) {
    int d = a.deg_rowptr[r + 1] - a.deg_rowptr[r];
    s = 1.f / float(d > 1 ? d : 1);
  }
  if (a.row_scale) s *= a.row_scale[r];
  return s * a.agg_coef;
}

__device__ __forceinline__ void store8(half_t* p, const float (&v)[8], float s) {
  half8_t h;
#pragma unroll
  for (int i = 0; i < 8; ++i) h[i] = half_t(v[i] * s);
  *reinterpret_cast<half8_t*>(p) = h;
}

// Y[row, f0..f0+7] = self_coef * self[row] + s * v  (the self term only when the call carries one)
__device__ __forceinline__ void store_row(const SpmmArgs& a, int64_t row, int f0, const float (&v)[8], float s) {
  half8_t h;
  if (a.self) {
    const half8_t sv = *reinterpret_cast<const half8_t*>(a.self + row * a.ld_self + f0);
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = half_t(fmaf(a.self_coef, float(sv[i]), v[i] * s));
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = half_t(v[i] * s);
  }
  half_t* y = a.Y + row * a.ldy + f0;
  if (f0 + 8 <= a.F) {
    __builtin_nontemporal_store(h, reinterpret_cast<half8_t*>(y));
  } else {  // F is not a multiple of 8: the last lane of a row owns fewer than 8 features
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (f0 + i < a.F) y[i] = h[i];
  }
}

__device__ __forceinline__ void fma8(float (&acc)[8], float w, const half8_t& x) {
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = fmaf(w, float(x[i]), acc[i]);
}

// p[0..7] += v with four packed fp16 atomic adds (the conflict-write scheme the paper removes, section 5.2.3)
__device__ __forceinline__ void atomic_add8(half_t* p, const float (&v)[8], int nvalid) {
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (2 * q >= nvalid) break;  // F is even, so a pair is valid as a whole
    half2_t h;
    h[0] = half_t(v[2 * q]);
    h[1] = half_t(v[2 * q + 1]);
    (void)__builtin_amdgcn_flat_atomic_fadd_v2f16(reinterpret_cast<half2_t*>(p) + q, h);
  }
}

// ---------------------------------------------------------------------------------------------------
// Vertex-parallel SpMM (no plan).  A wave owns G = 64/L consecutive rows.  Rows of at most kShortRow
// non-zeros are reduced by one lane group each, all G of them at once and with no exchange between
// lanes; every longer row is reduced by the whole wave, the groups striding over its non-zeros
// and their fp32 partial vectors added across groups with lane shuffles.  Rows longer than
// the hub threshold (SpmmArgs::long_row) are hubs: they are left to the chunked kernels further down.
// ---------------------------------------------------------------------------------------------------
constexpr int kShortRow = 32;
constexpr int kLongRowMin = 256, kLongRowMax = 1024;  // the hub threshold is 8 * mean row length within these, see hgnn_spmm

// acc += sum over the non-zeros k = first, first + STRIDE, ... < end of w_k * X[col_k, f0..f0+7],
// U of them in flight at a time; the column ids of the next U are fetched while the rows of
// the current U are on their way, so one trip through the loop costs one memory latency, not two
template <int STRIDE, bool HAS_W, int U>
__device__ __forceinline__ void edges_accumulate(const SpmmArgs& a, pos_t first, pos_t end, int f0c, int head,
                                                 float (&acc)[8]) {
  int c[U];
#pragma unroll
  for (int u = 0; u < U; ++u) c[u] = first + u * STRIDE < end ? a.col[first + u * STRIDE] : 0;
  for (pos_t k = first; k < end; k += STRIDE * U) {
    half8_t x[U];
    float wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const pos_t kk = k + u * STRIDE;
      x[u] = half8_t(0);
      wv[u] = 0.f;
      if (kk < end) {
        x[u] = *reinterpret_cast<const half8_t*>(a.X + int64_t(c[u]) * a.ldx + f0c);
        if (HAS_W) {
          const int64_t slot = a.eid ? int64_t(a.eid[kk]) : int64_t(kk);
          wv[u] = float(a.w[slot * a.H + head]);
        } else {
          wv[u] = a.one;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const pos_t kn = k + (U + u) * STRIDE;
      c[u] = kn < end ? a.col[kn] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) fma8(acc, wv[u], x[u]);
  }
}

// every lane ends up with the sum of its feature slice over the wave's G groups
template <int L>
__device__ __forceinline__ void groups_reduce(float (&acc)[8]) {
#pragma unroll
  for (int off = L; off < kWave; off <<= 1) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += __shfl_xor(acc[i], off);
  }
}

// the rows of workgroup `wg` (of blockDim.x / 64 waves)
template <int L, bool HAS_W>
__device__ __forceinline__ void spmm_row_body(const SpmmArgs& a, int64_t wg) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int rw = a.rows_per_wave;  // 1 or G
  const int64_t r0 = (wg * (int(blockDim.x) / kWave) + wave) * rw;
  if (r0 >= a.nrows) return;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int head = f0c / a.D;
  // the group's own row
  const int64_t rg = r0 + g;
  const bool has_row = g < rw && rg < a.nrows;
  int beg_g = 0, end_g = 0;
  if (has_row) {
    beg_g = a.rowptr[rg];
    end_g = a.rowptr[rg + 1];
  }
  if (has_row && end_g - beg_g <= kShortRow) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    edges_accumulate<1, HAS_W, 4>(a, beg_g, end_g, f0c, head, acc);
    if (active) store_row(a, rg, f0, acc, scale_of(a, int(rg)));
  }
  // the wave's mid-length rows, one after the other
  for (int j = 0; j < rw; ++j) {
    const int beg = __shfl(beg_g, j * L), end = __shfl(end_g, j * L);
    if (end - beg <= kShortRow || end - beg > a.long_row) continue;  // done above / a hub
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    edges_accumulate<G, HAS_W, 4>(a, beg + g, end, f0c, head, acc);
    groups_reduce<L>(acc);
    if (g == 0 && active) store_row(a, r0 + j, f0, acc, scale_of(a, int(r0 + j)));
  }
}

template <int L, bool HAS_W>
__global__ __launch_bounds__(kBlock) void spmm_row_kernel(SpmmArgs a) {
  spmm_row_body<L, HAS_W>(a, blockIdx.x);
}

// Hubs.  A row longer than the hub threshold is cut into chunks of kHubChunk non-zeros, one wave per chunk,
// so that a hub of 10^5 edges keeps dozens of compute units busy instead of one.  Three
// launches: hub_scan_kernel lists the hubs and hands every one a run of consecutive chunk slots
// (the slot numbers depend on the order in which the atomic counter is reached, the values
// computed do not); spmm_hub_kernel reduces one chunk per wave into an fp32 partial row in
// scratch memory; spmm_hub_sum_kernel adds a hub's partial rows in chunk order and stores the row.
// No atomics touch feature data and the summation order is fixed.
constexpr int kHubChunk = 512;
constexpr int kHubGrid = 131072;  // single-wave workgroups walking the chunk list with a grid stride (with 16384 of them the
                                  // plain SpMM of a 62 M-edge power-law graph took 5 % longer; an idle launch costs 25 us)

struct HubLists {
  int* count;      // [0] chunks handed out, [1] hubs listed
  int* chunk_row;  // [max_chunks] the hub a chunk slot belongs to
  int* chunk_no;   // [max_chunks] its number within the hub
  int* hub_row;    // [max_hubs]
  int* hub_base;   // [max_hubs] first chunk slot of the hub
  float* part;     // [max_chunks][F rounded up to a multiple of 8]
  int max_chunks, max_hubs;
};

__global__ __launch_bounds__(kBlock) void hub_zero_kernel(HubLists h) {
  if (threadIdx.x < 2) h.count[threadIdx.x] = 0;
}

constexpr int kScanRows = 16;  // rows per thread in hub_scan_kernel

// A workgroup looks at kBlock * kScanRows rows, adds up what its hubs need in LDS and reserves it with one
// pair of atomic adds (thousands of single adds on one address would take longer than the SpMM of a small graph).
__global__ __launch_bounds__(kBlock) void hub_scan_kernel(SpmmArgs a, HubLists h) {
  __shared__ int s_chunks[kBlock], s_hubs[kBlock];
  __shared__ int s_base[2];
  const int64_t r0 = int64_t(blockIdx.x) * (kBlock * kScanRows);
  int my_chunks = 0, my_hubs = 0;
  for (int u = 0; u < kScanRows; ++u) {
    const int64_t r = r0 + u * kBlock + threadIdx.x;
    if (r >= a.nrows) break;
    const int deg = a.rowptr[r + 1] - a.rowptr[r];
    if (deg > a.long_row) {
      my_chunks += pieces_of(deg, kHubChunk);
      ++my_hubs;
    }
  }
  s_chunks[threadIdx.x] = my_chunks;
  s_hubs[threadIdx.x] = my_hubs;
  __syncthreads();
  // inclusive scan over the workgroup (Hillis-Steele; kBlock is small)
  for (int off = 1; off < kBlock; off <<= 1) {
    const int c = int(threadIdx.x) >= off ? s_chunks[threadIdx.x - off] : 0;
    const int n = int(threadIdx.x) >= off ? s_hubs[threadIdx.x - off] : 0;
    __syncthreads();
    s_chunks[threadIdx.x] += c;
    s_hubs[threadIdx.x] += n;
    __syncthreads();
  }
  if (threadIdx.x == kBlock - 1) {
    s_base[0] = s_chunks[kBlock - 1] > 0 ? atomicAdd(&h.count[0], s_chunks[kBlock - 1]) : 0;
    s_base[1] = s_hubs[kBlock - 1] > 0 ? atomicAdd(&h.count[1], s_hubs[kBlock - 1]) : 0;
  }
  __syncthreads();
  if (my_hubs == 0) return;
  int base = s_base[0] + s_chunks[threadIdx.x] - my_chunks;
  int i = s_base[1] + s_hubs[threadIdx.x] - my_hubs;
  for (int u = 0; u < kScanRows; ++u) {
    const int64_t r = r0 + u * kBlock + threadIdx.x;
    if (r >= a.nrows) break;
    const int deg = a.rowptr[r + 1] - a.rowptr[r];
    if (deg <= a.long_row) continue;
    const int nch = pieces_of(deg, kHubChunk);
    if (base + nch <= h.max_chunks && i < h.max_hubs) {  // always true for a valid rowptr
      h.hub_row[i] = int(r);
      h.hub_base[i] = base;
      for (int c = 0; c < nch; ++c) {
        h.chunk_row[base + c] = int(r);
        h.chunk_no[base + c] = c;
      }
    }
    base += nch;
    ++i;
  }
}

// one wave per chunk, single-wave workgroups walking the chunk list with a grid stride
// the chunks first, first + stride, ... of the list, one wave
template <int L, bool HAS_W>
__device__ __forceinline__ void spmm_hub_body(const SpmmArgs& a, const HubLists& h, int64_t first, int64_t stride) {
  constexpr int G = kWave / L;
  const int nchunks = h.count[0] < h.max_chunks ? h.count[0] : h.max_chunks;
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int pitch = (a.F + 7) & ~7;
  for (int64_t c = first; c < nchunks; c += stride) {
    const int row = h.chunk_row[c];
    const int row_end = a.rowptr[row + 1];
    const int b = a.rowptr[row] + h.chunk_no[c] * kHubChunk;
    const int e = row_end - b > kHubChunk ? b + kHubChunk : row_end;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    edges_accumulate<G, HAS_W, 4>(a, b + g, e, f0c, f0c / a.D, acc);
    groups_reduce<L>(acc);
    if (g == 0 && active) {
      float* out = h.part + c * pitch + f0;
#pragma unroll
      for (int i = 0; i < 8; ++i) out[i] = acc[i];
    }
  }
}

template <int L, bool HAS_W>
__global__ __launch_bounds__(kWave) void spmm_hub_kernel(SpmmArgs a, HubLists h) {
  spmm_hub_body<L, HAS_W>(a, h, blockIdx.x, gridDim.x);
}

// Rows and hub chunks in one launch of single-wave workgroups: the row workgroups first, then hub_wgs workgroups that
// walk the chunk list.  Neither kind of work depends on the other (the lists are there when the launch begins), so
// the chunks start while the last rows are still being reduced instead of waiting for the row kernel to drain:
// 1 % on a 62 M-edge power-law graph, 9-14 % on graphs of 2-5 M edges.  The order matters on the large graph:
// chunks first, or chunk walkers spread among the row workgroups, were 8 % slower than rows first.
template <int L, bool HAS_W>
__global__ __launch_bounds__(kWave) void spmm_row_hub_kernel(SpmmArgs a, HubLists h, int hub_wgs) {
  const int64_t bid = blockIdx.x;
  const int64_t row_wgs = int64_t(gridDim.x) - hub_wgs;
  if (bid < row_wgs) spmm_row_body<L, HAS_W>(a, bid);
  else spmm_hub_body<L, HAS_W>(a, h, bid - row_wgs, hub_wgs);
}

// one wave per hub; its groups stride over the hub's partial rows
template <int L>
__global__ __launch_bounds__(kBlock) void spmm_hub_sum_kernel(SpmmArgs a, HubLists h) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int nhubs = h.count[1] < h.max_hubs ? h.count[1] : h.max_hubs;
  const int i = int(blockIdx.x) * kWavesPerBlock + wave;
  if (i >= nhubs) return;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int row = h.hub_row[i];
  const int nch = pieces_of(a.rowptr[row + 1] - a.rowptr[row], kHubChunk);
  const int pitch = (a.F + 7) & ~7;
  const float* part = h.part + int64_t(h.hub_base[i]) * pitch + f0c;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int c = g; c < nch; c += G) {
    const float4 lo = *reinterpret_cast<const float4*>(part + int64_t(c) * pitch);
    const float4 hi = *reinterpret_cast<const float4*>(part + int64_t(c) * pitch + 4);
    acc[0] += lo.x, acc[1] += lo.y, acc[2] += lo.z, acc[3] += lo.w;
    acc[4] += hi.x, acc[5] += hi.y, acc[6] += hi.z, acc[7] += hi.w;
  }
  groups_reduce<L>(acc);
  if (g == 0 && active) store_row(a, row, f0, acc, scale_of(a, row));
}

// ---------------------------------------------------------------------------------------------------
// Column passes of the plan-free SpMM.  Where the feature table misses the L2s but rows are long (hundreds of
// non-zeros), waves that each sweep their own row from its first column to its last are spread all over the table at
// any moment and share little in the L2s.  The passes align them: the columns are cut into npass equal ranges and
// the launch walks pass after pass (workgroups are numbered pass-major and dispatched in that order), a wave reducing
// the piece of its row that falls into the pass's range -- contiguous, because columns ascend inside a row -- into an
// fp32 partial row in the caller's workspace; one more kernel adds a row's npass partials in pass order, scales and
// rounds once.  Same arithmetic as one sweep (fp32 sums, one rounding), fixed summation order, no atomics.
// ---------------------------------------------------------------------------------------------------
constexpr int kPassLongRow = 16384;  // rows beyond this still go to the hub kernels

// First position p of [lo, hi) with col[p] >= key (hi if there is none), found by all 64 lanes of a wave together; every
// lane passes the same arguments and receives the same answer: 64 evenly spaced samples narrow the range 64-fold per
// step.  Reads stay inside [lo, hi) whatever the entries hold (an unsorted row gives a wrong cut, never a position
// outside the row).
__device__ __forceinline__ int wave_lower_bound(const int* __restrict__ col, int lo, int hi, int64_t key, int lane) {
  while (hi - lo > kWave) {
    const int n = hi - lo;
    const int v = col[lo + int((int64_t(lane) * n) >> 6)];
    const int cnt = __popcll(__ballot(int64_t(v) < key));
    if (cnt == 0) return lo;
    const int nlo = lo + int((int64_t(cnt - 1) * n) >> 6) + 1;
    const int nhi = cnt == kWave ? hi : lo + int((int64_t(cnt) * n) >> 6);
    lo = nlo;
    hi = nhi;
  }
  const int v = lane < hi - lo ? col[lo + lane] : INT_MAX;
  return lo + __popcll(__ballot(int64_t(v) < key));
}

constexpr int kMaxPasses = 16;

// cuts[r*(npass+1) + b] = first CSR position of row r whose column is >= b*width (b = npass: end of the row).
// One wave per row.  Every border is first looked for in a window of 64 entries around the place that an even spread
// of the columns over the row would give it; the windows of all borders are loaded together, so a row whose borders
// lie inside them costs one memory latency after its offsets.  A border outside its window is searched in the part
// of the row that the window rules in.
__global__ __launch_bounds__(kBlock) void row_cuts_kernel(const int* __restrict__ rowptr, const int* __restrict__ col,
                                                           int nrows, int ncols, int npass, int width, int long_row,
                                                           int* __restrict__ cuts) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t r = int64_t(blockIdx.x) * kWavesPerBlock + wave;
  if (r >= nrows) return;
  const int beg = rowptr[r], end = rowptr[r + 1];
  const int n = end - beg;
  int* out = cuts + r * (npass + 1);
  if (n == 0 || n > long_row) {  // nothing to cut / a hub: its passes are empty
    if (lane <= npass) out[lane] = lane == npass && n <= long_row ? end : beg;
    return;
  }
  int wlo[kMaxPasses], v[kMaxPasses];
#pragma unroll
  for (int b = 1; b < kMaxPasses; ++b) {
    wlo[b] = beg;
    v[b] = INT_MAX;
    if (b < npass) {
      int w = beg + int(int64_t(n) * b * width / ncols) - kWave / 2;
      if (w > end - kWave) w = end - kWave;
      if (w < beg) w = beg;
      wlo[b] = w;
      if (lane < end - w) v[b] = col[w + lane];
    }
  }
  int cut = lane == 0 ? beg : end;
#pragma unroll
  for (int b = 1; b < kMaxPasses; ++b) {
    if (b < npass) {
      const int64_t key = int64_t(b) * width;
      const int whi = end - wlo[b] > kWave ? wlo[b] + kWave : end;
      const int cnt = __popcll(__ballot(int64_t(v[b]) < key));
      int c;
      if (cnt > 0 && cnt < whi - wlo[b]) c = wlo[b] + cnt;                          // inside the window
      else if (cnt == 0) c = wlo[b] == beg ? beg : wave_lower_bound(col, beg, wlo[b], key, lane);  // before it
      else c = whi == end ? end : wave_lower_bound(col, whi, end, key, lane);       // after it
      if (lane == b) cut = c;
    }
  }
  if (lane <= npass) out[lane] = cut;
}

// one single-wave workgroup per (pass, row), pass-major
template <int L, bool HAS_W>
__global__ __launch_bounds__(kWave) void spmm_row_pass_kernel(SpmmArgs a, const int* __restrict__ cuts,
                                                              float* __restrict__ part, int npass) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int b = int(blockIdx.x / unsigned(a.nrows));
  const int64_t r = blockIdx.x % unsigned(a.nrows);
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int beg = cuts[r * (npass + 1) + b], end = cuts[r * (npass + 1) + b + 1];
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  edges_accumulate<G, HAS_W, 4>(a, beg + g, end, f0c, f0c / a.D, acc);
  groups_reduce<L>(acc);
  if (g == 0 && active) {
    const int pitch = (a.F + 7) & ~7;
    float* out = part + (int64_t(b) * a.nrows + r) * pitch + f0;
    *reinterpret_cast<float4*>(out) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    *reinterpret_cast<float4*>(out + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
  }
}

// a lane group per row: adds the row's partials in pass order and stores the row (hubs are left to spmm_hub_sum_kernel)
template <int L>
__global__ __launch_bounds__(kBlock) void spmm_pass_sum_kernel(SpmmArgs a, const float* __restrict__ part, int npass) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int64_t r = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  const int f0 = 8 * l;
  if (r >= a.nrows || f0 >= a.F) return;
  if (a.rowptr[r + 1] - a.rowptr[r] > a.long_row) return;
  const int pitch = (a.F + 7) & ~7;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int b = 0; b < npass; ++b) {
    const float* p = part + (int64_t(b) * a.nrows + r) * pitch + f0;
    const float4 lo = *reinterpret_cast<const float4*>(p);
    const float4 hi = *reinterpret_cast<const float4*>(p + 4);
    acc[0] += lo.x, acc[1] += lo.y, acc[2] += lo.z, acc[3] += lo.w;
    acc[4] += hi.x, acc[5] += hi.y, acc[6] += hi.z, acc[7] += hi.w;
  }
  store_row(a, r, f0, acc, scale_of(a, int(r)));
}

// Scalar path for shapes the 16-byte path cannot take: one thread per (row, feature).
__global__ __launch_bounds__(kBlock) void spmm_scalar_kernel(SpmmArgs a) {
  const int64_t idx = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= int64_t(a.nrows) * a.F) return;
  const int row = int(idx / a.F), f = int(idx % a.F);
  const int head = f / a.D;
  float acc = 0.f;
  for (int k = a.rowptr[row]; k < a.rowptr[row + 1]; ++k) {
    float wv = 1.f;
    if (a.w) {
      const int64_t slot = a.eid ? a.eid[k] : k;
      wv = float(a.w[slot * a.H + head]);
    }
    acc = fmaf(wv, float(a.X[int64_t(a.col[k]) * a.ldx + f]), acc);
  }
  a.Y[int64_t(row) * a.ldy + f] = half_t(acc * scale_of(a, row));
}

constexpr int kFinishShort = 8;  // rows of at most this many pieces are summed by one lane group, longer ones by a wave

// acc += staging rows k = first, first + STRIDE, ... <= last, U of them in flight at a time
template <int STRIDE, int U = 4>
__device__ __forceinline__ void pieces_accumulate(const SpmmArgs& a, int64_t first, int64_t last, int f0,
                                                  float (&acc)[8]) {
  for (int64_t k = first; k <= last; k += STRIDE * U) {
    half8_t t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t kk = k + u * STRIDE;
      t[u] = half8_t(0);
      if (kk <= last) t[u] = *reinterpret_cast<const half8_t*>(a.staging + kk * a.stage_ld + f0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += float(t[u][i]);
  }
}

// ---------------------------------------------------------------------------------------------------
// Discretized-reduction SpMM over row tasks: pass 1.  A wave takes one long piece of a row, or as many short pieces as it
// has lane groups, or a share of the empty rows.  A lane group stays inside its row, so its loop is eight gathers, the
// broadcast of the eight columns (and factors) held by its lanes, and 64 products; nothing is parked, nothing merged but
// the groups of a long piece.  Pieces of a row that has several go to staging slots as fp16 (each covers at most S
// non-zeros, so it cannot overflow where S * max|w x| fits fp16) and spmm_task_finish_kernel adds them; every row of Y has
// exactly one writer.
//
// Bound: the gathers, 64 bytes per clock and compute unit while the table sits in the L2s, the traffic behind the L2s
// beyond that (62 M non-zeros x 128: 8.9 GB of L2 misses per call at 7.0 TB/s, 11.9 at 7.4 where no row is cut at column ranges).  A call
// against the walk over equal runs of non-zeros with row ids in LDS: R-MAT 5.5 M non-zeros x 64, four heads of edge values 88 -> 59
// us, behind a map 131 -> 123; 2.1 M x 128 with the GIN terms 62 -> 43 us; 37 k x 64 19 -> 6 us; 114 M non-zeros x 64 in blocks of
// 3.7 MB 1.09 -> 0.83 ms (18 TB/s of rows); 62 M x 128 with edge values 1.73 -> 1.29,
// through a map 2.76 -> 2.04.
// WM: 0 = no factor per non-zero, 1 = edge values, 2 = edge values (if any) times a column scale.  MAPPED: edge values
// behind an edge-id map.
// ---------------------------------------------------------------------------------------------------
// HV: heads of the edge values where they are read as one vector (1, 2, 4 or 8; aligned to it), 0 = any number.
template <int L, int WM, int HV, int MOST>
struct TaskLds {
  typedef Round<L, MOST> Rd;
  static constexpr int G = kWave / L;
  static constexpr int kHandles = G * Rd::PITCH * 4;
  typedef typename std::conditional<WM == 2 || HV == 0, float, half_t>::type factor_t;
  // factors of a group: [R][H] and one 16-byte step to the next group's banks
  static __host__ __device__ int pitch(int H) { return Rd::R * H + 16 / int(sizeof(factor_t)); }
  static size_t bytes(int H) { return size_t(kHandles) + (WM == 0 ? 0 : size_t(G) * size_t(pitch(H)) * sizeof(factor_t)); }
};

// Which form the walk takes: what is left is cheaper where a run is asked of several arrays, positions where it is the ids alone (by
// position / by what is left, us: 5.5 M non-zeros x 4 heads of edge values 60.9 / 59.0; a GIN layer without edge values, 42 M x 16
// features, whose ids come from HBM, 463 / 480).
template <bool BY_POSITION>
__device__ __forceinline__ auto run_of(pos_t i0, pos_t end, int left) {
  if constexpr (BY_POSITION) return RunEnd{i0, end};
  else return RunLeft{left};
}

template <int L, int WM, bool NEAR, bool MAPPED, int HV, int MOST, class Enter>
__device__ __forceinline__ void spmm_task(SpmmArgs a, const TaskView& v, int ncols, Enter&& enter) {
  constexpr int G = kWave / L;
  typedef Round<L, MOST> Rd;
  typedef TaskLds<L, WM, HV, MOST> Lds;
  typedef typename Lds::factor_t factor_t;
  constexpr int NV = HV > 0 ? HV : 1;
  constexpr int E = Rd::E;
  typedef _Float16 hv_t __attribute__((ext_vector_type(NV)));
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;  // idle lanes of a group load a valid address and drop the result
  const TaskWave w = enter(g);
  a.Y += int64_t(w.block) * a.block_y_stride;
  if (w.z1 > w.z0) {
    const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (pos_t i = w.z0 + g; i < w.z1; i += G)
      if (active) store_row(a, w.zrow[i], f0, zero, 0.f);
    return;
  }
  const int H = HV > 0 ? HV : a.H;
  const int head = HV == 1 ? 0 : int(__umulhi(uint32_t(f0c), a.per_d));
  int* const s_hnd = reinterpret_cast<int*>(smem) + g * Rd::PITCH;
  factor_t* const s_val = reinterpret_cast<factor_t*>(smem + Lds::kHandles) + g * Lds::pitch(H);
  const RowTable<NEAR> table(a.X, ncols, a.ldx, f0c);
  const int row = w.row >= 0 ? w.row : 0;
  const float sc = scale_of(a, row);  // requested here, used at the end
  int shift = 0;  // slot in the edge tensors = position + shift
  if (WM != 0 && !MAPPED && a.delta) shift = a.delta[int64_t(w.block) * a.nrows + row] - w.first;
  const int own = (lane & (Rd::LC - 1)) * E;
  const bool nt = MAPPED && v.nb == 1 && stream_nontemporal(a.nnz);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (pos_t k = w.beg; k < w.end; k += w.step) {
    const pos_t end = k + w.span < w.end ? k + w.span : w.end;
    const int n = int(end - k);
    const pos_t i0 = k + own;
    const auto run = run_of<WM == 0>(i0, end, n - own);  // this lane's run
    wave_sync();  // the previous round has been read
    {
      int c[E], e[E];
      hv_t wv[E];
      float cs[E];
      load_cols<E>(v, a.col, nt, w.block, k, own, run, c);
      if (MAPPED) {
        if (nt) load_run<E, true>(a.eid, i0, run, e);
        else load_run<E, false>(a.eid, i0, run, e);
      }
      // slot 0 (load_run) where there is no non-zero: behind branches the gathers waited for one another (5.5 M non-zeros x 4 heads 111 -> 108 us,
      // 31 M without a plan 658 -> 654)
      if (MAPPED && HV > 0 && (WM == 1 || a.w)) {
        hv_t t[E];
#pragma unroll
        for (int m = 0; m < E; ++m) t[m] = *reinterpret_cast<const hv_t*>(a.w + int64_t(pos_t(e[m])) * NV);
#pragma unroll
        for (int m = 0; m < E; ++m) wv[m] = run.has(m) ? t[m] : hv_t(half_t(0));
      } else if (WM != 0 && HV > 0) {
        if (!MAPPED && (WM == 1 || a.w) && run.template all<E>()) {
          __builtin_memcpy(wv, a.w + int64_t(i0 + shift) * NV, sizeof(wv));
        } else {
#pragma unroll
          for (int m = 0; m < E; ++m) {
            wv[m] = hv_t(half_t(0));
            if (run.has(m)) {
              if (WM == 1 || a.w) wv[m] = *reinterpret_cast<const hv_t*>(a.w + int64_t(MAPPED ? pos_t(e[m]) : i0 + m + shift) * NV);
              else wv[m] = hv_t(half_t(1));
            }
          }
        }
      }
      // (also without branches, 2.1 M x 128 47.5 -> 46.4 us; without factors 37: a line more a non-zero.  The factor of column 0 may be infinite)
      if (WM == 2) {
        float t[E];
#pragma unroll
        for (int m = 0; m < E; ++m) t[m] = a.col_scale[run.has(m) ? c[m] : 0];
#pragma unroll
        for (int m = 0; m < E; ++m) cs[m] = run.has(m) ? t[m] : 0.f;
      }
#pragma unroll
      for (int m = 0; m < E; ++m) c[m] = table.handle(c[m], run.has(m));
#pragma unroll
      for (int m = 0; m < E; m += 4) *reinterpret_cast<int4_t*>(s_hnd + own + m) = int4_t{c[m], c[m + 1], c[m + 2], c[m + 3]};
      if (WM == 1 && HV > 0) {
        __builtin_memcpy(__builtin_assume_aligned(s_val + own * NV, 8), wv, sizeof(wv));
      } else if (WM != 0) {
        for (int m = 0; m < E; ++m)
          for (int h = 0; h < H; ++h) {
            float x = 0.f;
            if (HV > 0) x = float(wv[m][h < NV ? h : 0]) * (WM == 2 ? cs[m] : 1.f);
            else if (run.has(m)) x = (a.w ? float(a.w[int64_t(MAPPED ? pos_t(e[m]) : i0 + m + shift) * H + h]) : 1.f) * (WM == 2 ? cs[m] : 1.f);
            s_val[(own + m) * H + h] = factor_t(x);
          }
      }
    }
    wave_sync();
    for (int q = 0; WM == 0 ? k + pos_t(q) < end : q < n; q += 8) {
      int h8[8];
      const int4_t ha = *reinterpret_cast<const int4_t*>(s_hnd + q), hb = *reinterpret_cast<const int4_t*>(s_hnd + q + 4);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        h8[u] = ha[u];
        h8[4 + u] = hb[u];
      }
      half8_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = table.row(h8[u]);
      if (WM == 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) fma8(acc, a.one, x[u]);  // 1.0 the compiler cannot fold: keeps convert+add in one v_fma_mix
      } else {
        factor_t f[8];
        if (HV == 1) {
          __builtin_memcpy(f, __builtin_assume_aligned(s_val + q, 16), sizeof(f));
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) f[u] = s_val[(q + u) * H + head];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) fma8(acc, float(f[u]), x[u]);
      }
    }
  }
  if (w.whole) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = across_groups_sum<L>(acc[i]);
    if (g) return;
  }
  if (!active || w.row < 0) return;
  if (w.slot < 0) {
    store_row(a, row, f0, acc, sc);
  } else if (WM < 2 && a.atomic_y) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= sc;
    atomic_add8(a.Y + int64_t(row) * a.ldy + f0, acc, a.F - f0);
  } else if (WM < 2 && a.stage32) {
    float* out = reinterpret_cast<float*>(a.staging) + int64_t(w.slot) * a.stage_ld + f0;
    *reinterpret_cast<float4*>(out) = make_float4(acc[0] * sc, acc[1] * sc, acc[2] * sc, acc[3] * sc);
    *reinterpret_cast<float4*>(out + 4) = make_float4(acc[4] * sc, acc[5] * sc, acc[6] * sc, acc[7] * sc);
  } else {
    store8(a.staging + int64_t(w.slot) * a.stage_ld + f0, acc, sc);
  }
}

// LOOP: 1 = the number of tasks is only known on the device, a wave takes several (the loop costs registers: not with a plan); 2 = also
// pieces at column ranges (their branch costs the others 1 to 2 %)
template <int L, int WM, bool NEAR, bool MAPPED, int HV, int LOOP, int MOST>
__global__ __launch_bounds__(kWave, L < 8 ? 5 : (LOOP ? 6 : (WM == 0 ? 8 : 7))) void spmm_task_kernel(SpmmArgs a, TaskView v, int ncols) {
  constexpr int R = Round<L, MOST>::R;
  if (LOOP) {
    const RangeWaves ranges = LOOP == 2 ? range_waves<kWave / L>(v) : RangeWaves{0, 0, 0};
    const int n = ranges.waves + task_waves<kWave / L>(v);
    for (int wid = blockIdx.x; wid < n; wid += gridDim.x)
      spmm_task<L, WM, NEAR, MAPPED, HV, MOST>(a, v, ncols, [&](int g) { return task_enter<L, R, LOOP>(v, wid, g, ranges); });
  } else {
    spmm_task<L, WM, NEAR, MAPPED, HV, MOST>(a, v, ncols, [&](int g) { return task_enter<L, R>(v, blockIdx.x, g); });
  }
}

// Pass 2 (section 5.2.3): adds the staged fp16 pieces of every row that has several (fp32, in order) and stores the row
// once.  A wave owns one row, or G: then rows of at most kFinishShort pieces are summed by their own lane group, longer ones
// by the whole wave (finish_rows_per_wave).
template <int STRIDE, int U = 4>
__device__ __forceinline__ void pieces_accumulate32(const SpmmArgs& a, int64_t first, int64_t last, int f0, float (&acc)[8]) {
  const float* p = reinterpret_cast<const float*>(a.staging) + f0;
  for (int64_t k = first; k <= last; k += STRIDE * U) {
    float4 lo[U], hi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t kk = k + u * STRIDE;
      lo[u] = hi[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (kk <= last) {
        lo[u] = *reinterpret_cast<const float4*>(p + kk * a.stage_ld);
        hi[u] = *reinterpret_cast<const float4*>(p + kk * a.stage_ld + 4);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[0] += lo[u].x, acc[1] += lo[u].y, acc[2] += lo[u].z, acc[3] += lo[u].w;
      acc[4] += hi[u].x, acc[5] += hi[u].y, acc[6] += hi[u].z, acc[7] += hi[u].w;
    }
  }
}

// F32: pieces staged in fp32, n_split is a bound and the number is in *totals
template <int L, bool F32, bool MANY>
__global__ __launch_bounds__(kBlock) void spmm_task_finish_kernel(SpmmArgs a, const int4_t* __restrict__ split, int n_split, int per_wave,
                                                                  const TaskTotals* __restrict__ totals) {
  constexpr int G = kWave / L, kMany = kManyPieces * G;
  if (F32) {
    n_split = totals->n_split;
    per_wave = finish_rows_per_wave(n_split, totals->n_slots, G);
  }
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int64_t i0 = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * per_wave;
  if ((MANY ? int64_t(blockIdx.x) * kWavesPerBlock * per_wave : i0) >= n_split) return;  // MANY: the whole workgroup
  __shared__ int4_t s_row[kWavesPerBlock * G];
  __shared__ float s_sum[kWavesPerBlock][L][8];
  __shared__ int s_n;
  if (MANY) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
  }
  int4_t q = {0, 0, 0, 0};
  if (g < per_wave && i0 + g < n_split) q = split[i0 + g];
  const int alone = per_wave > 1 ? kFinishShort : 0;
  half_t* const Y = a.Y;
  if (MANY && q[2] > kMany && l == 0) s_row[atomicAdd(&s_n, 1)] = q;
  if (q[2] > 0 && q[2] <= alone) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (F32) pieces_accumulate32<1>(a, q[1], int64_t(q[1]) + q[2] - 1, f0c, acc);
    else pieces_accumulate<1>(a, q[1], int64_t(q[1]) + q[2] - 1, f0c, acc);
    a.Y = Y + int64_t(q[3]) * a.block_y_stride;
    if (active) store_row(a, q[0], f0, acc, 1.f);
  }
  for (int j = 0; j < per_wave; ++j) {
    const int n = __shfl(q[2], j * L);
    if (n <= alone || (MANY && n > kMany)) continue;
    const int r = __shfl(q[0], j * L), first = __shfl(q[1], j * L), b = __shfl(q[3], j * L);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (F32) pieces_accumulate32<G>(a, int64_t(first) + g, int64_t(first) + n - 1, f0c, acc);
    else pieces_accumulate<G>(a, int64_t(first) + g, int64_t(first) + n - 1, f0c, acc);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = across_groups_sum<L>(acc[i]);
    a.Y = Y + int64_t(b) * a.block_y_stride;
    if (g == 0 && active) store_row(a, r, f0, acc, 1.f);
  }
  if (!MANY) return;
  __syncthreads();
  for (int j = 0; j < s_n; ++j) {  // the rows of many pieces, one after the other (in whatever order)
    const int4_t m = s_row[j];
    const int64_t first = m[1] + wave * G + g, last = int64_t(m[1]) + m[2] - 1;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (F32) pieces_accumulate32<kWavesPerBlock * G>(a, first, last, f0c, acc);
    else pieces_accumulate<kWavesPerBlock * G, 8>(a, first, last, f0c, acc);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = across_groups_sum<L>(acc[i]);
      if (g == 0) s_sum[wave][l][i] = acc[i];
    }
    __syncthreads();
    if (wave == j % kWavesPerBlock && g == 0 && active) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        acc[i] = 0.f;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) acc[i] += s_sum[w][l][i];
      }
      a.Y = Y + int64_t(m[3]) * a.block_y_stride;
      store_row(a, m[0], f0, acc, 1.f);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------------
// Vertex-parallel variant of the discretized SpMM (section 5.4): a wave reduces one neighbour group,
// at most ng non-zeros of a single row, so there is no row change inside a wave and no merge; what
// is left of the conflict is between the waves that share a long row.  A row with one group is
// stored directly; the groups of a longer row store their scaled fp16 partials in staging slots of
// their own and spmm_vgroup_finish_kernel adds them.  Edge values of a group start at an arbitrary
// position of the edge tensor: with one value per edge they are fetched as aligned pairs, starting
// one position early when the group starts at an odd position, and the pair is taken apart while it
// is copied to LDS.
// ---------------------------------------------------------------------------------------------------
struct VGroupArgs {
  const int* grp_row;
  const int* goff;
  const int* moff;
  int64_t n_groups;
  int ng;
  int pair_loads;  // edge values: one per edge, no edge-id map, 4-byte aligned base
  int acc16;       // products and sums of a lane's chunk in packed fp16 (the paper's arithmetic, section 4.2)
};

__host__ __device__ inline int align16i(int v) { return (v + 15) & ~15; }

__host__ __device__ inline int vgroup_lds_bytes(int ng, int H, bool has_w) {
  const int spad = kWave * 4 * ((ng + 255) / 256);
  return spad * 4 + (has_w ? align16i(spad * H * 2) : 0);
}

// VW = halves per lane and load: 8 (16 bytes), 4 or 2 -- the narrower forms exist for the vector-width
// study (section 6.3.1 carried over to SpMM); a row of F halves then takes L = pow2 >= F/VW lanes.
template <int L, int VW, bool HAS_W, bool OFF32>
__global__ __launch_bounds__(kBlock) void spmm_vgroup_kernel(SpmmArgs a, VGroupArgs v) {
  constexpr int G = kWave / L;
  typedef _Float16 hv_t __attribute__((ext_vector_type(VW)));
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = VW * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int head = f0c / a.D;
  const int spad = kWave * 4 * ((v.ng + 255) / 256);
  unsigned char* base = smem + size_t(wave) * vgroup_lds_bytes(v.ng, a.H, HAS_W);
  int* s_col = reinterpret_cast<int*>(base);
  half_t* s_w = reinterpret_cast<half_t*>(base + spad * 4);

  const int64_t j = int64_t(blockIdx.x) * (int(blockDim.x) / kWave) + wave;
  const bool valid = j < v.n_groups;
  int row = 0, idx = 0, cnt = 1, k0 = 0, n = 0;
  if (valid) {
    row = v.grp_row[j];
    idx = int(j - v.goff[row]);
    cnt = v.goff[row + 1] - v.goff[row];
    k0 = a.rowptr[row] + idx * v.ng;
    const int left = a.rowptr[row + 1] - k0;
    n = left < v.ng ? left : v.ng;
  }

  // ---- phase 1: coalesced stage of column ids (as byte offsets) and edge values
  const bool pairs = HAS_W && v.pair_loads;
  for (int i = lane; i < spad; i += kWave) {
    const bool in = i < n;
    const int c = in ? a.col[k0 + i] : 0;
    s_col[i] = OFF32 ? int(uint32_t(c) * uint32_t(a.ldx) * 2u) : c;
    if (HAS_W) {
      if (!pairs) {
        const int64_t slot = in ? (a.eid ? int64_t(a.eid[k0 + i]) : int64_t(k0 + i)) : 0;
        for (int h = 0; h < a.H; ++h) s_w[i * a.H + h] = in ? a.w[slot * a.H + h] : half_t(0);
      } else if (!in) {
        s_w[i] = half_t(0);
      }
    }
  }
  if (pairs) {
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    const int odd = k0 & 1;
    const int64_t b = int64_t(k0) - odd;  // even position at or just before the group's first value
    for (int i = lane; 2 * i < n + odd; i += kWave) {
      half2_t pr;
      if (b + 2 * i + 1 < a.nnz) {
        pr = *reinterpret_cast<const half2_t*>(a.w + b + 2 * i);
      } else {
        pr[0] = a.w[b + 2 * i];
        pr[1] = half_t(0);
      }
      const int i0 = 2 * i - odd;
      if (i0 >= 0 && i0 < n) s_w[i0] = pr[0];
      if (i0 + 1 < n) s_w[i0 + 1] = pr[1];
    }
  }
  wave_sync();

  // ---- phase 2: the groups of lanes take consecutive chunks of the neighbour group
  const int C = 4 * ((v.ng + 4 * G - 1) / (4 * G));
  const int c0 = g * C < n ? g * C : n;
  const int c1 = c0 + C < n ? c0 + C : n;
  float acc[VW];
#pragma unroll
  for (int q = 0; q < VW; ++q) acc[q] = 0.f;
  half2_t acc2[VW / 2 > 0 ? VW / 2 : 1];
#pragma unroll
  for (int q = 0; q < VW / 2; ++q) acc2[q] = half2_t{half_t(0), half_t(0)};
  auto gather = [&](int c) -> hv_t {
    if (OFF32) {
      const uint32_t boff = uint32_t(c) + uint32_t(f0c) * 2u;
      return *reinterpret_cast<const hv_t*>(reinterpret_cast<const char*>(a.X) + boff);
    }
    return *reinterpret_cast<const hv_t*>(a.X + int64_t(c) * a.ldx + f0c);
  };
  for (int i = c0; i < c1; i += 4) {
    const int4_t cols = *reinterpret_cast<const int4_t*>(s_col + i);
    hv_t x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = gather(cols[u]);  // padding holds offset 0, a valid row
    float wv[4] = {a.one, a.one, a.one, a.one};
    if (HAS_W) {
      if (a.H == 1) {
        const half4_t w4 = *reinterpret_cast<const half4_t*>(s_w + i);
#pragma unroll
        for (int u = 0; u < 4; ++u) wv[u] = float(w4[u]);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) wv[u] = float(s_w[(i + u) * a.H + head]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (i + 4 <= c1 || i + u < c1) {
        if (VW == 8 && v.acc16) {
          // section 4.2: the edge value mirrored into both halves of a pair multiplies two features per
          // instruction (v_pk_fma_f16); the sum of this lane's chunk stays in fp16
          const half2_t w2 = {half_t(wv[u]), half_t(wv[u])};
#pragma unroll
          for (int q = 0; q < VW / 2; ++q) {
            const half2_t x2 = {x[u][2 * q], x[u][2 * q + 1]};
            acc2[q] = x2 * w2 + acc2[q];
          }
        } else {
#pragma unroll
          for (int q = 0; q < VW; ++q) acc[q] = fmaf(wv[u], float(x[u][q]), acc[q]);
        }
      }
    }
  }
  if (VW == 8 && v.acc16) {
#pragma unroll
    for (int q = 0; q < VW / 2; ++q) {
      acc[2 * q] = float(acc2[q][0]);
      acc[2 * q + 1] = float(acc2[q][1]);
    }
  }
#pragma unroll
  for (int off = L; off < kWave; off <<= 1) {
#pragma unroll
    for (int q = 0; q < VW; ++q) acc[q] += __shfl_xor(acc[q], off);
  }
  if (valid && g == 0 && active) {
    const float sc = scale_of(a, row);
    hv_t h;
#pragma unroll
    for (int q = 0; q < VW; ++q) h[q] = half_t(acc[q] * sc);
    half_t* dst = cnt == 1 ? a.Y + int64_t(row) * a.ldy + f0 : a.staging + (int64_t(v.moff[row]) + idx) * a.stage_ld + f0;
    if (cnt != 1 || f0 + VW <= a.F) {  // staging rows are padded to a multiple of 8
      *reinterpret_cast<hv_t*>(dst) = h;
    } else {
#pragma unroll
      for (int q = 0; q < VW; ++q)
        if (f0 + q < a.F) dst[q] = h[q];
    }
  }
}

// Follow-up kernel of the vertex-parallel variant; it also writes the empty rows.  A wave looks at G
// rows: rows with up to kFinishShort groups are summed by their own lane group, longer ones by the wave.
template <int L>
__global__ __launch_bounds__(kBlock) void spmm_vgroup_finish_kernel(SpmmArgs a, VGroupArgs v) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int64_t r0 = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G;
  if (r0 >= a.nrows) return;
  const int64_t r = r0 + g;
  int cnt = 1, first = 0;  // cnt = 1: nothing to do
  if (r < a.nrows) {
    cnt = v.goff[r + 1] - v.goff[r];
    first = v.moff[r];
  }
  if (cnt == 0 && active) {
    const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    store_row(a, r, f0, zero, 0.f);
  }
  if (cnt > 1 && cnt <= kFinishShort) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    pieces_accumulate<1>(a, first, int64_t(first) + cnt - 1, f0c, acc);
    if (active) store_row(a, r, f0, acc, 1.f);
  }
  for (int j = 0; j < G; ++j) {
    const int cj = __shfl(cnt, j * L), fj = __shfl(first, j * L);
    if (cj <= kFinishShort) continue;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    pieces_accumulate<G>(a, int64_t(fj) + g, int64_t(fj) + cj - 1, f0c, acc);
    groups_reduce<L>(acc);
    if (g == 0 && active) store_row(a, r0 + j, f0, acc, 1.f);
  }
}

// zero the rows whose pieces the atomic comparison variant adds into Y
template <int L>
__global__ __launch_bounds__(kBlock) void zero_split_rows_kernel(SpmmArgs a, const int4_t* __restrict__ split, int n_split) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int64_t idx = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  if (idx >= n_split || 8 * l >= a.F) return;
  const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  SpmmArgs b = a;
  b.self = nullptr;
  store_row(b, split[idx][0], 8 * l, zero, 0.f);
}

// ---------------------------------------------------------------------------------------------------
hgnn_status check_spmm_args(const char* who, const hgnn_csr* g, const hgnn_half* w, int H, const hgnn_half* X,
                                   int64_t ldx, hgnn_half* Y, int64_t ldy, int F, hgnn_reduce op) {
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(F > 0, HGNN_EINVAL, "%s: F = %d must be positive", who, F);
  HGNN_REQUIRE(F % 2 == 0, HGNN_EINVAL, "%s: F = %d is odd; pad the feature length to the next even number", who, F);
  HGNN_REQUIRE(H >= 1 && F % H == 0, HGNN_EINVAL, "%s: H = %d does not divide F = %d", who, H, F);
  HGNN_REQUIRE(ldx >= F && ldy >= F, HGNN_EINVAL, "%s: leading dimension smaller than F", who);
  HGNN_REQUIRE(ldx % 2 == 0 && ldy % 2 == 0, HGNN_EINVAL, "%s: odd leading dimension", who);
  HGNN_REQUIRE(op == HGNN_SUM || op == HGNN_MEAN, HGNN_EINVAL, "%s: unknown reduce op %d", who, int(op));
  HGNN_REQUIRE(g->nrows == 0 || Y != nullptr, HGNN_EINVAL, "%s: Y is NULL", who);
  HGNN_REQUIRE(g->nnz == 0 || X != nullptr, HGNN_EINVAL, "%s: X is NULL", who);
  (void)w;
  return HGNN_OK;
}

static bool vector_path_ok(const hgnn_half* w, int H, const hgnn_half* X, int64_t ldx, const hgnn_half* Y, int64_t ldy,
                           int F) {
  // F itself need not be a multiple of 8: rows are read in 16-byte pieces up to the padded pitch and the
  // last piece is stored by element
  if (F > 512 || ldx % 8 != 0 || ldy % 8 != 0) return false;
  if (!aligned16(X) || !aligned16(Y)) return false;
  if (w && H > 1 && (F / H) % 8 != 0) return false;
  return true;
}

static SpmmArgs make_args(const hgnn_csr* g, const hgnn_half* w, int H, const hgnn_half* X, int64_t ldx, hgnn_half* Y,
                          int64_t ldy, int F, hgnn_reduce op, const float* row_scale) {
  SpmmArgs a{};
  a.rowptr = g->rowptr;
  a.deg_rowptr = g->rowptr;
  a.col = g->col;
  a.eid = g->eid;
  a.w = reinterpret_cast<const half_t*>(w);
  a.X = reinterpret_cast<const half_t*>(X);
  a.Y = reinterpret_cast<half_t*>(Y);
  a.row_scale = row_scale;
  a.ldx = ldx;
  a.ldy = ldy;
  a.nnz = g->nnz;
  a.nrows = g->nrows;
  a.F = F;
  a.H = w ? H : 1;  // without edge values the head structure is irrelevant
  a.D = F / a.H;
  a.per_d = a.D > 1 ? uint32_t(((uint64_t(1) << 32) + uint32_t(a.D) - 1) / uint32_t(a.D)) : 0;  // (rows of tasks have D = F or a multiple of 8)
  a.reduce = int(op);
  a.one = 1.0f;
  a.agg_coef = 1.0f;
  a.self_coef = 0.0f;
  return a;
}

template <int L, bool HAS_W>
static void launch_row_set(dim3 grid, hipStream_t s, const SpmmArgs& a, const HubLists* h) {
  if (!h) {
    spmm_row_kernel<L, HAS_W><<<grid, kWave, 0, s>>>(a);  // its waves never meet: single-wave workgroups
    return;
  }
  const int64_t hub_wgs = h->max_chunks < kHubGrid ? h->max_chunks : kHubGrid;
  const int64_t row_wgs = grid.x;
  if (row_wgs + hub_wgs >= (int64_t(1) << 31)) {
    spmm_row_kernel<L, HAS_W><<<grid, kWave, 0, s>>>(a);
    spmm_hub_kernel<L, HAS_W><<<dim3(unsigned(hub_wgs)), kWave, 0, s>>>(a, *h);
  } else {
    spmm_row_hub_kernel<L, HAS_W><<<dim3(unsigned(row_wgs + hub_wgs)), kWave, 0, s>>>(a, *h, int(hub_wgs));
  }
  spmm_hub_sum_kernel<L><<<dim3(unsigned(ceil_div(h->max_hubs, kWavesPerBlock))), kBlock, 0, s>>>(a, *h);
}

template <int L, bool HAS_W>
static void launch_pass_set(hipStream_t s, const SpmmArgs& a, const HubLists* h, const int* cuts, float* part, int npass) {
  constexpr int G = kWave / L;
  spmm_row_pass_kernel<L, HAS_W><<<dim3(unsigned(int64_t(npass) * a.nrows)), kWave, 0, s>>>(a, cuts, part, npass);
  spmm_pass_sum_kernel<L><<<dim3(unsigned(ceil_div(a.nrows, int64_t(kWavesPerBlock) * G))), kBlock, 0, s>>>(a, part, npass);
  if (h) {
    // only rows beyond kPassLongRow are left to the chunks here: a small grid walks the list
    constexpr int kGrid = 8192;
    spmm_hub_kernel<L, HAS_W><<<dim3(unsigned(h->max_chunks < kGrid ? h->max_chunks : kGrid)), kWave, 0, s>>>(a, *h);
    const int64_t max_hubs = std::min<int64_t>(h->max_hubs, a.nnz / kPassLongRow + 1);
    spmm_hub_sum_kernel<L><<<dim3(unsigned(ceil_div(max_hubs, kWavesPerBlock))), kBlock, 0, s>>>(a, *h);
  }
}

template <bool HAS_W>
static void launch_pass(int L, hipStream_t s, const SpmmArgs& a, const HubLists* h, const int* cuts, float* part, int npass) {
  switch (L) {
    case 1: launch_pass_set<1, HAS_W>(s, a, h, cuts, part, npass); break;
    case 2: launch_pass_set<2, HAS_W>(s, a, h, cuts, part, npass); break;
    case 4: launch_pass_set<4, HAS_W>(s, a, h, cuts, part, npass); break;
    case 8: launch_pass_set<8, HAS_W>(s, a, h, cuts, part, npass); break;
    case 16: launch_pass_set<16, HAS_W>(s, a, h, cuts, part, npass); break;
    case 32: launch_pass_set<32, HAS_W>(s, a, h, cuts, part, npass); break;
    default: launch_pass_set<64, HAS_W>(s, a, h, cuts, part, npass); break;
  }
}

template <bool HAS_W>
static void launch_row(int L, dim3 grid, hipStream_t s, const SpmmArgs& a, const HubLists* h) {
  switch (L) {
    case 1: launch_row_set<1, HAS_W>(grid, s, a, h); break;
    case 2: launch_row_set<2, HAS_W>(grid, s, a, h); break;
    case 4: launch_row_set<4, HAS_W>(grid, s, a, h); break;
    case 8: launch_row_set<8, HAS_W>(grid, s, a, h); break;
    case 16: launch_row_set<16, HAS_W>(grid, s, a, h); break;
    case 32: launch_row_set<32, HAS_W>(grid, s, a, h); break;
    default: launch_row_set<64, HAS_W>(grid, s, a, h); break;
  }
}

// Scratch of the hub kernels: chunk and hub lists and one fp32 partial row per chunk, in one block of device memory
// that the caller hands over (hgnn_spmm) or that sits in the library's static device array (hgnn_spmm_static).
// The sizes are worst-case bounds taken from the graph's sizes alone, so that they are known without a look at the
// graph: the sum over the hubs of ceil(deg / chunk) is at most nnz / chunk + the number of hubs, and there are
// fewer than nnz / long_row hubs.
static int hub_threshold(int64_t nrows, int64_t nnz) {
  // hubs: rows longer than 8 times the mean, but never a threshold below 256 or above 1024 non-zeros (on sparse
  // power-law graphs 256 balanced better than 1024: 17 % on an R-MAT of mean degree 16, 1-3 % at mean degree
  // 21-26; with rows of 500 on average 1024 was 2 % better than 4000)
  const int64_t mean = nrows > 0 ? nnz / nrows : 0;
  return int(std::min<int64_t>(std::max<int64_t>(kLongRowMin, 8 * mean), kLongRowMax));
}

struct HubLayout {
  int64_t o_count, o_crow, o_cno, o_hrow, o_hbase, o_part, bytes;
  int64_t max_chunks, max_hubs;
};

static HubLayout hub_layout(int64_t nnz, int long_row, int F) {
  HubLayout o{};
  if (nnz <= long_row) return o;  // no row can be a hub: bytes = 0
  o.max_hubs = nnz / long_row + 1;
  o.max_chunks = nnz / kHubChunk + o.max_hubs + 1;
  auto up = [](int64_t b) { return (b + 255) / 256 * 256; };
  o.o_count = 0;
  o.o_crow = o.o_count + 256;
  o.o_cno = o.o_crow + up(o.max_chunks * 4);
  o.o_hrow = o.o_cno + up(o.max_chunks * 4);
  o.o_hbase = o.o_hrow + up(o.max_hubs * 4);
  o.o_part = o.o_hbase + up(o.max_hubs * 4);
  o.bytes = o.o_part + up(o.max_chunks * int64_t((F + 7) & ~7) * 4);
  return o;
}

// Column passes are taken under the rule that makes a plan cut its graph into column blocks: the table (ncols rows of
// F halves) is beyond three L2s, fits three quarters of the cache behind them, and rows average 128 non-zeros or more;
// about two L2 sizes of feature rows per pass.  1 = one sweep.
static int row_passes(int64_t nrows, int64_t ncols, int64_t nnz, int F) {
  if (nrows <= 0 || nnz / nrows < 128) return 1;
  int64_t l2 = 0, llc = 0;
  device_cache_bytes(&l2, &llc);
  const double table = double(ncols) * F * 2.0;
  if (!(table > 3.0 * double(l2) && table < 0.75 * double(llc))) return 1;
  if (int64_t(16) * nrows >= (int64_t(1) << 31)) return 1;  // one workgroup per (pass, row)
  int np = int(table / (2.0 * double(l2)) + 0.5);
  return np < 2 ? 2 : (np > kMaxPasses ? kMaxPasses : np);
}

struct PassLayout {
  int64_t o_cuts, o_part, bytes;  // offsets from the end of the hub scratch
};

static PassLayout pass_layout(int64_t nrows, int npass, int F) {
  PassLayout o{};
  auto up = [](int64_t b) { return (b + 255) / 256 * 256; };
  o.o_cuts = 0;
  o.o_part = up(nrows * (npass + 1) * 4);
  o.bytes = o.o_part + up(int64_t(npass) * nrows * ((F + 7) & ~7) * 4);
  return o;
}

// The plan-free SpMM over row tasks.  Against the kernels that take rows in storage order and hubs in chunks, tasks have lists to
// write, and a wave reads its numbers from memory; they win where rows differ in length and a non-zero costs more than its
// gather.  Behind a map they cost up to 27 % more on uniform rows and 46 % less on skewed ones.  us, rows / tasks:
//   non-zeros, rows         F   no edge values   edge values   behind a map
//   1.3 M power law         8       41 / 38        47 / 41        70 / 52
//                          64       44 / 38        61 / 39        83 / 45
//   2 M uniform, 10 a row   8       30 / 39        33 / 46        56 / 71
//                          32       42 / 44        47 / 47        71 / 66
//                          64       51 / 55        59 / 56        82 / 72
//   6 M, 200 a row         16       51 / 64        58 / 69        77 / 89
//                          32       55 / 63        69 / 68        83 / 94
//                          64       69 / 71       105 / 74       103 / 109
//   18 M power law         16      263 / 295      301 / 301      598 / 603
//                          64      372 / 349      509 / 373      825 / 669
//   31 M power law         32      331 / 325      389 / 340      934 / 822
//                          64      383 / 358      517 / 373     1023 / 855
static bool free_tasks_pay(int F, bool edge_values, bool mapped) { return mapped || F >= (edge_values ? 32 : 64); }

constexpr int kFreePiece = 512;  // non-zeros per piece
constexpr int kRangeRow = 256;   // longer rows are cut at column ranges where that pays
constexpr size_t kNearMiss = 512;
// scratch of the tasks, 0 where no row can be long (then one wave per row does)
static size_t free_task_bytes(int64_t nrows, int64_t nnz, int F) {
  if (hub_layout(nnz, hub_threshold(nrows, nnz), F).bytes == 0) return 0;
  return task_scratch_at(nullptr, nrows, nnz, kFreePiece, F, kNoRanges).bytes;
}

// Where long rows of the plan-free SpMM are cut at column ranges, as with a plan: room for it where the table is beyond what the L2s hold
// together, and done where it pays.  The pieces are staged in fp32, so rows of 257 non-zeros are long enough.  us, rows in pieces /
// at column ranges, listing included (some 12 us of it):
//                                       edge values    behind a map
//   31 M power law, 154 MB, F = 64         366 / 380       853 / 683
//   54 M, 307 MB, F = 64                   755 / 698      1740 / 1398
//   12 M, 77 MB, F = 64                    138 / 145       292 / 253
//   12 M, 154 MB, F = 128                  281 / 255       479 / 395
//   5.5 M, 67 MB, F = 128                  119 / 126       192 / 176
//   5.5 M, 134 MB, F = 256                 255 / 220       342 / 283
//   14 M, 512 MB, F = 256                  766 / 684       995 / 874
//   60 M, 77 MB, F = 16                    742 / 741      1840 / 1545
//   20 M log-normal, 51 MB, F = 64         400 / 398       725 / 728
//   20 M uniform (no long row), 128 MB     420 / 420       777 / 777
//   5.5 M, 34 MB, F = 64                    71 / 80        121 / 122
static bool free_ranges_pay(bool mapped, int64_t ncols, int F) {
  int64_t l2 = 0, llc = 0;
  device_cache_bytes(&l2, &llc);
  return mapped || ncols * F * 2 >= (F >= 128 ? llc / 2 : llc);
}
// scratch of the tasks with column ranges; 0: no call takes them
static size_t free_range_bytes(int64_t nrows, int64_t ncols, int64_t nnz, int F) {
  if (nnz <= int64_t(4) << 20 || F > 512 || free_task_bytes(nrows, nnz, F) == 0) return 0;
  int64_t l2 = 0, llc = 0;
  device_cache_bytes(&l2, &llc);
  if (ncols * F * 2 <= 8 * l2) return 0;
  return task_scratch_at(nullptr, nrows, nnz, kFreePiece, F, kRangeRow + 1).bytes;
}

static HubLists hub_lists_at(void* base, const HubLayout& o) {
  HubLists h{};
  char* p = static_cast<char*>(base);
  h.count = reinterpret_cast<int*>(p + o.o_count);
  h.chunk_row = reinterpret_cast<int*>(p + o.o_crow);
  h.chunk_no = reinterpret_cast<int*>(p + o.o_cno);
  h.hub_row = reinterpret_cast<int*>(p + o.o_hrow);
  h.hub_base = reinterpret_cast<int*>(p + o.o_hbase);
  h.part = reinterpret_cast<float*>(p + o.o_part);
  h.max_chunks = int(o.max_chunks);
  h.max_hubs = int(o.max_hubs);
  return h;
}

template <int L, int VW>
static void launch_vgroup_main(bool has_w, bool off32, dim3 grid, int threads, size_t lds, hipStream_t s, const SpmmArgs& a,
                               const VGroupArgs& v) {
  if (has_w) {
    if (off32) spmm_vgroup_kernel<L, VW, true, true><<<grid, threads, lds, s>>>(a, v);
    else if (VW == 8) spmm_vgroup_kernel<L, 8, true, false><<<grid, threads, lds, s>>>(a, v);
  } else {
    if (off32) spmm_vgroup_kernel<L, VW, false, true><<<grid, threads, lds, s>>>(a, v);
    else if (VW == 8) spmm_vgroup_kernel<L, 8, false, false><<<grid, threads, lds, s>>>(a, v);
  }
}

template <int VW>
static void launch_vgroup_vw(int L, bool has_w, bool off32, dim3 grid, int threads, size_t lds, hipStream_t s, const SpmmArgs& a,
                             const VGroupArgs& v) {
  switch (L) {
    case 1: launch_vgroup_main<1, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    case 2: launch_vgroup_main<2, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    case 4: launch_vgroup_main<4, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    case 8: launch_vgroup_main<8, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    case 16: launch_vgroup_main<16, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    case 32: launch_vgroup_main<32, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
    default: launch_vgroup_main<64, VW>(has_w, off32, grid, threads, lds, s, a, v); break;
  }
}

static void launch_vgroup_finish(int L, dim3 grid, hipStream_t s, const SpmmArgs& a, const VGroupArgs& v) {
  switch (L) {
    case 1: spmm_vgroup_finish_kernel<1><<<grid, kBlock, 0, s>>>(a, v); break;
    case 2: spmm_vgroup_finish_kernel<2><<<grid, kBlock, 0, s>>>(a, v); break;
    case 4: spmm_vgroup_finish_kernel<4><<<grid, kBlock, 0, s>>>(a, v); break;
    case 8: spmm_vgroup_finish_kernel<8><<<grid, kBlock, 0, s>>>(a, v); break;
    case 16: spmm_vgroup_finish_kernel<16><<<grid, kBlock, 0, s>>>(a, v); break;
    case 32: spmm_vgroup_finish_kernel<32><<<grid, kBlock, 0, s>>>(a, v); break;
    default: spmm_vgroup_finish_kernel<64><<<grid, kBlock, 0, s>>>(a, v); break;
  }
}

// The vertex-parallel variant for the graph in `a` with the neighbour groups of plan p.
static hgnn_status run_vgroups(const hgnn_plan* p, SpmmArgs a, int ncols, bool acc16, hipStream_t s) {
  VGroupArgs v{};
  v.acc16 = acc16 ? 1 : 0;
  v.grp_row = p->grp_row;
  v.goff = p->goff;
  v.moff = p->moff;
  v.n_groups = p->n_groups;
  v.ng = p->ng;
  v.pair_loads = (a.w && a.H == 1 && !a.eid && (reinterpret_cast<uintptr_t>(a.w) & 3u) == 0) ? 1 : 0;
  a.staging = reinterpret_cast<half_t*>(p->gstage);
  a.stage_ld = p->max_F;
  // halves per lane: 8 unless the plan's setting asks for a narrower load and the shape allows it
  int vw = acc16 ? 8 : p->vec_halves;
  const bool off32 = uint64_t(ncols) * uint64_t(a.ldx) * 2u < (uint64_t(1) << 32);
  if (vw != 8) {
    HGNN_REQUIRE(off32 && a.F <= kWave * vw && a.D % vw == 0, HGNN_EUNSUPPORTED,
                 "hgnn_spmm_discretized_variant: %d halves per lane needs F <= %d, D %% %d == 0 and a feature table below 4 GiB",
                 vw, kWave * vw, vw);
  }
  const int L = pow2_at_least((a.F + vw - 1) / vw);   // lanes per row in the main kernel
  const int L8 = pow2_at_least((a.F + 7) / 8);        // the follow-up kernel always moves 16 bytes per lane
  const size_t vg_per_wave = size_t(vgroup_lds_bytes(v.ng, a.H, a.w != nullptr));
  const int wpb = waves_per_block_for_lds(vg_per_wave, a.w != nullptr);
  const size_t lds = vg_per_wave * wpb;
  HGNN_REQUIRE(lds <= 65536, HGNN_EUNSUPPORTED,
               "hgnn_spmm_discretized_variant: group_edges = %d with H = %d needs %zu bytes of LDS per workgroup (limit 65536)",
               v.ng, a.H, lds);
  dim3 grid(unsigned(ceil_div(v.n_groups > 0 ? v.n_groups : 1, wpb)));
  dim3 grid2(unsigned(ceil_div(a.nrows, int64_t(kWavesPerBlock) * (kWave / L8))));
  const bool has_w = a.w != nullptr;
  if (v.n_groups > 0) {
    if (vw == 8) launch_vgroup_vw<8>(L, has_w, off32, grid, wpb * kWave, lds, s, a, v);
    else if (vw == 4) launch_vgroup_vw<4>(L, has_w, off32, grid, wpb * kWave, lds, s, a, v);
    else launch_vgroup_vw<2>(L, has_w, off32, grid, wpb * kWave, lds, s, a, v);
  }
  launch_vgroup_finish(L8, grid2, s, a, v);
  HGNN_LAUNCH_CHECK("spmm_vgroup_kernel / spmm_vgroup_finish_kernel");
  return HGNN_OK;
}

// the vector forms of several heads only where they are used in earnest: edge values alone, a table below 4 GB
template <int L, bool NEAR>
static void launch_tasks_l(int wm, bool mapped, unsigned waves, size_t least_lds, hipStream_t s, const SpmmArgs& a,
                           const TaskView& v, int ncols) {
  const dim3 grid(waves);
#define HGNN_TASKS(WM, MAPPED, HV)                                                                                          \
  do {                                                                                                                      \
    with_round<L, NEAR && (WM == 0 || HV == 1 || (WM == 1 && (HV == 2 || HV == 4)))>(v, [&](auto most) {                    \
      constexpr int M = decltype(most)::value;                                                                              \
      const size_t lds = std::max(TaskLds<L, WM, HV, M>::bytes(a.H), least_lds);                                            \
      if constexpr (WM < 2) {                                                                                               \
        if (v.rtotals) {                                                                                                    \
          spmm_task_kernel<L, WM, NEAR, MAPPED, HV, 2, M><<<grid, kWave, lds, s>>>(a, v, ncols);                            \
          return;                                                                                                           \
        }                                                                                                                   \
        if (v.totals) {                                                                                                     \
          spmm_task_kernel<L, WM, NEAR, MAPPED, HV, 1, M><<<grid, kWave, lds, s>>>(a, v, ncols);                            \
          return;                                                                                                           \
        }                                                                                                                   \
      }                                                                                                                     \
      spmm_task_kernel<L, WM, NEAR, MAPPED, HV, 0, M><<<grid, kWave, lds, s>>>(a, v, ncols);                                \
    });                                                                                                                     \
  } while (0)
  const int hv = (reinterpret_cast<uintptr_t>(a.w) & uintptr_t(2 * a.H - 1)) == 0 ? a.H : 0;
  if (wm == 0) {
    HGNN_TASKS(0, false, 1);
    return;
  }
  if (wm == 1) {
    if (a.H == 1) {
      if (mapped) HGNN_TASKS(1, true, 1);
      else HGNN_TASKS(1, false, 1);
      return;
    }
    if constexpr (NEAR) {
      if (hv == 2) {
        if constexpr (L >= 2) {
          if (mapped) HGNN_TASKS(1, true, 2);
          else HGNN_TASKS(1, false, 2);
          return;
        }
      }
      if (hv == 4) {
        if constexpr (L >= 4) {
          if (mapped) HGNN_TASKS(1, true, 4);
          else HGNN_TASKS(1, false, 4);
          return;
        }
      }
      if (hv == 8) {
        if constexpr (L >= 8) {
          if (mapped) HGNN_TASKS(1, true, 8);
          else HGNN_TASKS(1, false, 8);
          return;
        }
      }
    }
    if (mapped) HGNN_TASKS(1, true, 0);
    else HGNN_TASKS(1, false, 0);
    return;
  }
  if (a.H == 1) {
    if (mapped) HGNN_TASKS(2, true, 1);
    else HGNN_TASKS(2, false, 1);
  } else {
    if (mapped) HGNN_TASKS(2, true, 0);
    else HGNN_TASKS(2, false, 0);
  }
#undef HGNN_TASKS
}

template <bool NEAR>
static void launch_tasks(int L, int wm, bool mapped, unsigned waves, size_t least_lds, hipStream_t s, const SpmmArgs& a,
                         const TaskView& v, int ncols) {
  switch (L) {
    case 1: launch_tasks_l<1, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    case 2: launch_tasks_l<2, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    case 4: launch_tasks_l<4, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    case 8: launch_tasks_l<8, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    case 16: launch_tasks_l<16, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    case 32: launch_tasks_l<32, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
    default: launch_tasks_l<64, NEAR>(wm, mapped, waves, least_lds, s, a, v, ncols); break;
  }
}

// Every wave has eight gathers a lane group in flight.  Where the gathered lines miss the L2s, 28 to 32 waves per compute unit ask for
// more than an L2 holds (32 compute units x 32 waves x 32 rows of 256 bytes: 8.4 MB), and popular rows and shared lines of the
// edge values are gone before the next wave wants them.  LDS that nobody uses then keeps waves out.  us, by waves per compute unit:
//   edge values behind a map: non-zeros x heads          28     20     16     14     12
//     2.1 M x 1 (4 MB, as an L2), 128 features           62.4   62.5   64.3   74.5   78.5
//     5.5 M x 1 (11 MB), 64 features                      104    102    102    107    111
//     5.5 M x 4 (44 MB)                                   130    123    122    127    132
//     114 M x 1 in blocks (228 MB)                       1793   1709   1688      -   1676
//    long rows cut at column ranges:
//     12 M x 1 (24 MB)                                    232    225    222    222
//     31 M x 4 (248 MB)                                   746    708    707    740
//     62 M x 1 (124 MB), 128 features                    2075   2048   2043   2042
//     log-normal rows, 26 M x 4 (204 MB), 128 features   1284   1230   1169   1189
//     60 M x 1 (120 MB), 16 features                     1479   1438   1422   1374
//   unmapped: table beside a last-level cache of 256 MB
//     77 MB, 31 M non-zeros, no edge values (154 MB)      371    377    388    445    469
//    no row cut at column ranges:
//     307 MB, 62 M, by degrees                            901    871    852      -    967
//     614 MB, 62 M, by degrees                           1849   1835   1823      -   1880
//    long rows cut at column ranges:
//     307 MB, 62 M, by degrees                            740    763    783    876
//     614 MB, 62 M, edge values                          1327   1328   1329   1357
// (tables that fit that cache, and the rows of one range in an L2, gain or lose either way, so they are left alone).  A wave of short
// rows is mostly its own start and end, which other waves must cover (28 / 16 waves: 7 non-zeros a row over 1.06 GB 960 / 1004 us, through
// the map 1186 / 1229; 13 a row over 614 MB, no edge values, 866 / 907).
// Unmapped and with a plan, which knows how many pieces at column ranges there are, those decide from one for every 320 non-zeros on; fewer leave
// most rows as they are.  28 / 16 waves: power law, 62 M x 64 by degrees (one for 229) 617 / 642; log-normal, 55 M x 128 (one for 380)
// 1924 / 1903, 14 M x 256 (one for 1300) 954 / 938, 27 M x 128 (one for 1500) 1093 / 1055.  Without a plan the host does not know: 27 M x 128
// with edge values, no long row 1058 / 1034, power law 638 / 650, 62 M x 64 770 / 781.
static size_t least_task_lds(bool mapped, bool ranges, const SpmmArgs& a, int64_t ncols, int64_t l2, int64_t llc) {
  constexpr size_t kLds = 160 * 1024;  // of a compute unit
  const int64_t edge_bytes = a.nnz * a.H * 2, table_bytes = ncols * a.ldx * 2;
  if (a.nnz < int64_t(16) * a.nrows) return 0;
  if (mapped && edge_bytes > l2) return edge_bytes > 12 * l2 && !ranges ? kLds / 14 / 16 * 16 : kLds / 16;
  return !mapped && !ranges && table_bytes > llc ? kLds / 16 : 0;
}

static void launch_zero_split(int L, hipStream_t s, const SpmmArgs& a, const TaskView& v) {
  const dim3 grid(unsigned(ceil_div(v.n_split, int64_t(kWavesPerBlock) * (kWave / L))));
  switch (L) {
    case 1: zero_split_rows_kernel<1><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    case 2: zero_split_rows_kernel<2><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    case 4: zero_split_rows_kernel<4><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    case 8: zero_split_rows_kernel<8><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    case 16: zero_split_rows_kernel<16><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    case 32: zero_split_rows_kernel<32><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
    default: zero_split_rows_kernel<64><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split); break;
  }
}

template <int L>
static void launch_task_finish_l(dim3 grid, int per_wave, hipStream_t s, const SpmmArgs& a, const TaskView& v) {
  if (a.stage32) spmm_task_finish_kernel<L, true, true><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave, v.totals);
  else if (many_pieces(v, kWave / L)) spmm_task_finish_kernel<L, false, true><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave, nullptr);
  else spmm_task_finish_kernel<L, false, false><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave, nullptr);
}

static void launch_task_finish(int L, hipStream_t s, const SpmmArgs& a, const TaskView& v) {
  const int per_wave = finish_rows_per_wave(v.n_split, v.n_slots, kWave / L);
  // a bound on the rows (fp32) may be above a line that their number is below
  const int64_t waves = std::max<int64_t>(ceil_div(v.n_split, per_wave), a.stage32 ? std::min(v.n_split, kFinishAlone) : 0);
  const dim3 grid(unsigned(ceil_div(waves, kWavesPerBlock)));
  switch (L) {
    case 1: launch_task_finish_l<1>(grid, per_wave, s, a, v); break;
    case 2: launch_task_finish_l<2>(grid, per_wave, s, a, v); break;
    case 4: launch_task_finish_l<4>(grid, per_wave, s, a, v); break;
    case 8: launch_task_finish_l<8>(grid, per_wave, s, a, v); break;
    case 16: launch_task_finish_l<16>(grid, per_wave, s, a, v); break;
    case 32: launch_task_finish_l<32>(grid, per_wave, s, a, v); break;
    default: launch_task_finish_l<64>(grid, per_wave, s, a, v); break;
  }
}

// LDS for each non-zero of a round: its handle and its factors
static int task_entry_bytes(int wm, const SpmmArgs& a) { return 4 + (wm == 0 ? 0 : a.H * (wm == 1 ? 2 : 4)); }

static bool mostly_ranges(const hgnn_row_tasks* t) { return int64_t(t->n_rtask) * 320 >= t->nnz; }

// Pass 1 and pass 2 of the discretized SpMM over the row tasks t of plan p, whose column array `a.col` indexes (with a.eid,
// a.delta beside it); a.Y / a.ldy / a.block_y_stride describe the result, or the column blocks' partial results.
static hgnn_status run_tasks(const hgnn_plan* p, const hgnn_row_tasks* t, SpmmArgs a, int ncols, hipStream_t s) {
  const int wm = a.col_scale ? 2 : (a.w ? 1 : 0);
  const int L = pow2_at_least((a.F + 7) / 8), G = kWave / L;
  a.staging = reinterpret_cast<half_t*>(t->staging);
  a.stage_ld = p->max_F;
  const bool mapped = wm != 0 && a.w && a.eid;
  // (the comparison variant with atomic additions rounds each to fp16: as many as there are segments)
  const bool ranges = !a.atomic_y && at_ranges(t, mapped ? kRangesMapped : kRangesSpmm, int64_t(ncols) * a.F * 2, p->l2_bytes);
  TaskView v = task_view(t, G, ranges, comes_back(mapped, int64_t(ncols) * a.ldx * 2, p->llc_bytes));
  v.longer = long_rounds(t->nb, p->nrows, t->nnz, p->S, G, task_entry_bytes(wm, a));
  const int waves = v.first_wave[t->nb];
  if (a.atomic_y && v.n_split > 0) {
    launch_zero_split(L, s, a, v);
    HGNN_LAUNCH_CHECK("zero_split_rows_kernel");
  }
  if (waves > 0) {
    const size_t least = least_task_lds(mapped, ranges && (mapped || mostly_ranges(t)), a, ncols, p->l2_bytes, p->llc_bytes);
    if (near_table(ncols, a.ldx)) launch_tasks<true>(L, wm, mapped, unsigned(waves), least, s, a, v, ncols);
    else launch_tasks<false>(L, wm, mapped, unsigned(waves), least, s, a, v, ncols);
    HGNN_LAUNCH_CHECK("spmm_task_kernel");
  }
  if (v.n_split > 0 && !a.atomic_y) {
    launch_task_finish(L, s, a, v);
    HGNN_LAUNCH_CHECK("spmm_task_finish_kernel");
  }
  return HGNN_OK;
}

// Column-blocked plans: Y[r] = sum over the blocks of their (already scaled, fp16) partial rows; fp32 sum in
// block order, one store per row.
template <int L>
__global__ __launch_bounds__(kBlock) void spmm_block_sum_kernel(SpmmArgs a, const half_t* __restrict__ part, int nb,
                                                                 int part_ld) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const int64_t r = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  if (r >= a.nrows || f0 >= a.F) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int b = 0; b < nb; ++b) {
    const half8_t t = *reinterpret_cast<const half8_t*>(part + (int64_t(b) * a.nrows + r) * part_ld + f0);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += float(t[i]);
  }
  store_row(a, r, f0, acc, 1.f);
}

static void launch_block_sum(int L, dim3 grid, hipStream_t s, const SpmmArgs& a, const half_t* part, int nb, int part_ld) {
  switch (L) {
    case 1: spmm_block_sum_kernel<1><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    case 2: spmm_block_sum_kernel<2><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    case 4: spmm_block_sum_kernel<4><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    case 8: spmm_block_sum_kernel<8><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    case 16: spmm_block_sum_kernel<16><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    case 32: spmm_block_sum_kernel<32><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
    default: spmm_block_sum_kernel<64><<<grid, kBlock, 0, s>>>(a, part, nb, part_ld); break;
  }
}

// The plan-free SpMM over row tasks that are listed in the scratch by two small launches: rows sorted by length and cut into
// pieces, so that lane groups end together and a hub keeps many compute units busy, as with a plan.  Pieces are staged in
// fp32, a row is rounded once; long rows are cut at column ranges where asked for.  A wave per G rows in storage order, hubs in chunks of their own, took as long
// as its longest row: 31 M non-zeros x 64 with values, graph and transpose through the map, 1.54 -> 1.23 ms together.
static hgnn_status spmm_free_tasks(const hgnn_csr* g, SpmmArgs a, void* scratch, bool ranges, hipStream_t s) {
  const TaskSource q{g->rowptr, nullptr, g->nrows, 1, kFreePiece, task_group_max(g->nnz), g->nnz, ranges ? kRangeRow + 1 : kNoRanges};
  const TaskScratch t = task_scratch_at(scratch, g->nrows, g->nnz, kFreePiece, a.F, q.range_min);
  const hgnn_status st = task_build_in(q, t, g->col, g->ncols, s);
  if (st != HGNN_OK) return st;
  const int L = pow2_at_least((a.F + 7) / 8);
  const bool mapped = a.w && a.eid;
  int64_t grid = 0;
  TaskView v = task_view(t, q, g->nnz, kWave / L, &grid);
  v.longer = long_rounds(1, g->nrows, g->nnz, kFreePiece, kWave / L, task_entry_bytes(a.w ? 1 : 0, a));
  a.staging = reinterpret_cast<half_t*>(t.staging);
  a.stage_ld = (a.F + 7) & ~7;
  a.stage32 = 1;
  const int wm = a.w ? 1 : 0;
  int64_t l2 = 0, llc = 0;
  device_cache_bytes(&l2, &llc);
  const size_t least = least_task_lds(mapped, ranges, a, g->ncols, l2, llc);
  if (near_table(g->ncols, a.ldx)) launch_tasks<true>(L, wm, mapped, unsigned(grid), least, s, a, v, g->ncols);
  else launch_tasks<false>(L, wm, mapped, unsigned(grid), least, s, a, v, g->ncols);
  HGNN_LAUNCH_CHECK("spmm_task_kernel");
  launch_task_finish(L, s, a, v);
  HGNN_LAUNCH_CHECK("spmm_task_finish_kernel");
  return HGNN_OK;
}

// The plan-free SpMM with its scratch at `scratch` (scratch_bytes of device memory, may be null: then no row is
// treated as a hub and a long row is reduced by one wave).
hgnn_status spmm_rows(const char* who, const hgnn_csr* g, const hgnn_half* edge_val, int32_t H, const hgnn_half* X,
                             int64_t ldx, hgnn_half* Y, int64_t ldy, int32_t F, hgnn_reduce op, const float* row_scale,
                             void* scratch, size_t scratch_bytes, bool one_sweep, hipStream_t s) {
  SpmmArgs a = make_args(g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale);
  if (!vector_path_ok(edge_val, H, X, ldx, Y, ldy, F)) {
    dim3 grid(unsigned(ceil_div(int64_t(g->nrows) * F, kBlock)));
    spmm_scalar_kernel<<<grid, kBlock, 0, s>>>(a);
    HGNN_LAUNCH_CHECK("spmm_scalar_kernel");
    return HGNN_OK;
  }
  const int L = pow2_at_least((F + 7) / 8);
  // sparse rows: a wave takes one row per lane group; dense rows: one row per wave, for balance
  a.rows_per_wave = g->nnz / g->nrows >= 64 ? 1 : kWave / L;
  dim3 grid(unsigned(ceil_div(g->nrows, a.rows_per_wave)));
  a.long_row = hub_threshold(g->nrows, g->nnz);
  const HubLayout lay = hub_layout(g->nnz, a.long_row, F);
  HubLists h{};
  const bool hubs = lay.bytes > 0 && scratch != nullptr;
  const int npass = scratch ? row_passes(g->nrows, g->ncols, g->nnz, F) : 1;
  const PassLayout pl = pass_layout(g->nrows, npass, F);
  const size_t base_bytes = spmm_hub_scratch_bytes(g->nrows, g->nnz, F), task_bytes = free_task_bytes(g->nrows, g->nnz, F);
  // passes need their own room behind the chunks of the long rows; where the tasks need more than that, a workspace for one
  // sweep (hgnn_spmm_workspace with ncols = 0) is told from one for passes by the sum of both
  size_t pass_bytes = base_bytes + size_t(pl.bytes);
  if (task_bytes >= pass_bytes && scratch_bytes >= task_bytes) pass_bytes = task_bytes + size_t(pl.bytes);
  if (npass > 1 && !one_sweep && scratch_bytes >= pass_bytes) {
    HGNN_REQUIRE((reinterpret_cast<uintptr_t>(scratch) & 15u) == 0, HGNN_EINVAL, "%s: the workspace must be 16-byte aligned", who);
    a.long_row = kPassLongRow > a.long_row ? kPassLongRow : a.long_row;
    if (hubs) {
      h = hub_lists_at(scratch, lay);
      hub_zero_kernel<<<1, kBlock, 0, s>>>(h);
      hub_scan_kernel<<<dim3(unsigned(ceil_div(g->nrows, kBlock * kScanRows))), kBlock, 0, s>>>(a, h);
    } else {
      a.long_row = INT_MAX;
    }
    char* base = static_cast<char*>(scratch) + base_bytes;
    int* cuts = reinterpret_cast<int*>(base + pl.o_cuts);
    float* part = reinterpret_cast<float*>(base + pl.o_part);
    const int width = int(ceil_div(g->ncols, npass));
    row_cuts_kernel<<<dim3(unsigned(ceil_div(g->nrows, kWavesPerBlock))), kBlock, 0, s>>>(g->rowptr, g->col, g->nrows, g->ncols,
                                                                                        npass, width, a.long_row, cuts);
    if (edge_val) launch_pass<true>(L, s, a, hubs ? &h : nullptr, cuts, part, npass);
    else launch_pass<false>(L, s, a, hubs ? &h : nullptr, cuts, part, npass);
    HGNN_LAUNCH_CHECK("spmm_row_pass_kernel");
    return HGNN_OK;
  }
  if (hubs) {
    HGNN_REQUIRE(scratch_bytes >= base_bytes, HGNN_EINVAL, "%s: the workspace holds %zu bytes, this graph needs %zu", who,
                 scratch_bytes, base_bytes);
    // (a size that misses the query's answer by a few bytes is a mistake, not a workspace for the chunks alone)
    HGNN_REQUIRE(one_sweep || scratch_bytes >= task_bytes || scratch_bytes == base_bytes || task_bytes - scratch_bytes > kNearMiss,
                 HGNN_EINVAL, "%s: the workspace holds %zu bytes, this graph needs %zu", who, scratch_bytes, task_bytes);
    HGNN_REQUIRE((reinterpret_cast<uintptr_t>(scratch) & 15u) == 0, HGNN_EINVAL, "%s: the workspace must be 16-byte aligned", who);
    if (scratch_bytes >= task_bytes && free_tasks_pay(F, edge_val != nullptr, edge_val && g->eid)) {
      const size_t range_bytes = free_range_bytes(g->nrows, g->ncols, g->nnz, F);
      const bool ranges = range_bytes > 0 && npass == 1 && !one_sweep && scratch_bytes >= range_bytes &&
                          free_ranges_pay(edge_val && g->eid, g->ncols, F);
      return spmm_free_tasks(g, a, scratch, ranges, s);
    }
    // (a workspace, or the static array, can be too small for the tasks and still hold the hubs)
    h = hub_lists_at(scratch, lay);
    hub_zero_kernel<<<1, kBlock, 0, s>>>(h);
    hub_scan_kernel<<<dim3(unsigned(ceil_div(g->nrows, kBlock * kScanRows))), kBlock, 0, s>>>(a, h);
  } else {
    a.long_row = INT_MAX;  // no scratch: every row above the short-row limit is reduced by one wave
  }
  if (edge_val) launch_row<true>(L, grid, s, a, hubs ? &h : nullptr);
  else launch_row<false>(L, grid, s, a, hubs ? &h : nullptr);
  HGNN_LAUNCH_CHECK("spmm_row_kernel");
  return HGNN_OK;
}

size_t spmm_hub_scratch_bytes(int32_t nrows, int64_t nnz, int32_t F) {
  if (nrows <= 0 || nnz <= 0 || F <= 0) return 0;
  return size_t(hub_layout(nnz, hub_threshold(nrows, nnz), F).bytes);
}

}  // namespace hgnn

using namespace hgnn;

extern "C" {

size_t hgnn_spmm_workspace(int32_t nrows, int32_t ncols, int64_t nnz, int32_t F) {
  if (nrows <= 0 || nnz <= 0 || F <= 0) return 0;
  const size_t base = spmm_hub_scratch_bytes(nrows, nnz, F), task = free_task_bytes(nrows, nnz, F), held = hgnn_spmm_static_limit();
  // ncols = 0: what gives the results of hgnn_spmm_static, which takes the tasks only where its array holds them
  if (ncols <= 0 && base <= held && task > held) return base;
  size_t need = std::max(base, task);
  const int npass = ncols > 0 ? row_passes(nrows, ncols, nnz, F) : 1;
  if (npass > 1) return need + size_t(pass_layout(nrows, npass, F).bytes);
  return std::max(need, ncols > 0 ? free_range_bytes(nrows, ncols, nnz, F) : 0);
}

hgnn_status hgnn_spmm(const hgnn_csr* g, const hgnn_half* edge_val, int32_t H, const hgnn_half* X, int64_t ldx,
                      hgnn_half* Y, int64_t ldy, int32_t F, hgnn_reduce op, const float* row_scale, void* workspace,
                      size_t workspace_bytes, void* stream) {
  clear_error();
  hgnn_status st = check_spmm_args("hgnn_spmm", g, edge_val, H, X, ldx, Y, ldy, F, op);
  if (st != HGNN_OK) return st;
  if (g->nrows == 0) return HGNN_OK;
  return spmm_rows("hgnn_spmm", g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale, workspace, workspace_bytes, false,
                   static_cast<hipStream_t>(stream));
}

hgnn_status hgnn_spmm_discretized_fused(const hgnn_plan* p, const hgnn_csr* g, const hgnn_half* edge_val, int32_t H,
                                        const hgnn_half* X, int64_t ldx, hgnn_half* Y, int64_t ldy, int32_t F,
                                        hgnn_reduce op, const float* row_scale, const hgnn_spmm_fusion* fz,
                                        void* stream) {
  clear_error();
  const char* who = "hgnn_spmm_discretized";
  hgnn_status st = check_spmm_args(who, g, edge_val, H, X, ldx, Y, ldy, F, op);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(F <= p->max_F, HGNN_EINVAL, "%s: F = %d exceeds the plan's max_F = %d", who, F, p->max_F);
  HGNN_REQUIRE(vector_path_ok(edge_val, H, X, ldx, Y, ldy, F), HGNN_EUNSUPPORTED,
               "%s: needs F <= 512, ld %% 8 == 0, 16-byte aligned X, Y, and D %% 8 == 0 when edge values have several heads", who);
  if (fz && fz->self)
    HGNN_REQUIRE(fz->ld_self >= F && fz->ld_self % 8 == 0 && aligned16(fz->self), HGNN_EINVAL,
                 "%s: self features need ld_self >= F, ld_self %% 8 == 0 and a 16-byte aligned base", who);
  const bool prescale = fz && fz->col_scale && fz->scaled_x;
  if (prescale)
    HGNN_REQUIRE(fz->ld_scaled >= F && fz->ld_scaled % 8 == 0 && aligned16(fz->scaled_x), HGNN_EINVAL,
                 "%s: the scaled_x workspace needs ld_scaled >= F, ld_scaled %% 8 == 0 and a 16-byte aligned base", who);
  if (g->nrows == 0) return HGNN_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  SpmmArgs a = make_args(g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale);
  if (prescale) {
    // the column scale goes onto the table once; the kernels then run without a per-edge factor
    st = hgnn_scale_rows(g->ncols, F, X, ldx, fz->col_scale, fz->scaled_x, fz->ld_scaled, stream);
    if (st != HGNN_OK) return st;
    a.X = reinterpret_cast<const half_t*>(fz->scaled_x);
    a.ldx = fz->ld_scaled;
  }
  if (fz) {
    a.col_scale = prescale ? nullptr : fz->col_scale;
    a.self = reinterpret_cast<const half_t*>(fz->self);
    a.ld_self = fz->ld_self;
    a.self_coef = fz->self_coef;
    a.agg_coef = fz->agg_coef;
    if (a.col_scale && !edge_val) {  // the per-edge factor is the column scale alone; heads are irrelevant
      a.H = 1;
      a.D = F;
      a.per_d = 0;
    }
  }
  // blocks that the automatic rule chose (for max_F) are used when the table of this call is beyond an L2 too
  const bool use_blocks = p->nb > 1 && (!p->auto_blocks || double(g->ncols) * double(a.ldx) * 2.0 > 3.0 * double(p->l2_bytes));
  if (!use_blocks) return run_tasks(p, p->tasks, a, g->ncols, s);
  HGNN_REQUIRE(!(edge_val && g->eid && !p->block_eid), HGNN_EINVAL,
               "%s: the column-blocked plan was built from a graph without an edge-id map; build the plan from the graph "
               "that carries the map", who);
  // column-blocked plan: one discretized SpMM per block into that block's partial output, blocks one
  // after the other so that all compute units gather from the same slice of X, then one pass adds
  // the partials of every row (and the self term, once).  Scales are applied per partial (section 5.2.2).
  p = walked_cut(p, edge_val && g->eid);
  {
    // all blocks in one launch (waves numbered block after block and dispatched in that order), into the blocks' partial
    // outputs.  Slots in the edge tensors: a graph without an edge-id map reads at its own CSR positions (block position +
    // the row's offset, a coalesced read); a graph with one reads through the blocked copy of the map
    SpmmArgs ab = a;
    ab.col = p->bcol;
    ab.eid = g->eid ? p->beid : nullptr;
    ab.delta = g->eid ? nullptr : p->bdelta;
    ab.Y = reinterpret_cast<half_t*>(p->bstage);
    ab.ldy = p->max_F;
    ab.block_y_stride = int64_t(p->nrows) * p->max_F;
    ab.self = nullptr;
    st = run_tasks(p, p->btasks, ab, g->ncols, s);
    if (st != HGNN_OK) return st;
  }
  const int L = pow2_at_least((F + 7) / 8);
  const int G = kWave / L;
  launch_block_sum(L, dim3(unsigned(ceil_div(g->nrows, int64_t(kWavesPerBlock) * G))), s, a,
                   reinterpret_cast<const half_t*>(p->bstage), p->nb, p->max_F);
  HGNN_LAUNCH_CHECK("spmm_block_sum_kernel");
  return HGNN_OK;
}

hgnn_status hgnn_spmm_discretized(const hgnn_plan* p, const hgnn_csr* g, const hgnn_half* edge_val, int32_t H,
                                  const hgnn_half* X, int64_t ldx, hgnn_half* Y, int64_t ldy, int32_t F,
                                  hgnn_reduce op, const float* row_scale, void* stream) {
  return hgnn_spmm_discretized_fused(p, g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale, nullptr, stream);
}

hgnn_status hgnn_spmm_discretized_variant(const hgnn_plan* p, const hgnn_csr* g, const hgnn_half* edge_val, int32_t H,
                                          const hgnn_half* X, int64_t ldx, hgnn_half* Y, int64_t ldy, int32_t F,
                                          hgnn_reduce op, const float* row_scale, hgnn_spmm_variant variant,
                                          void* stream) {
  if (variant == HGNN_EDGE_SEGMENTS)
    return hgnn_spmm_discretized_fused(p, g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale, nullptr, stream);
  clear_error();
  const char* who = "hgnn_spmm_discretized_variant";
  HGNN_REQUIRE(variant == HGNN_EDGE_SEGMENTS_ATOMIC || variant == HGNN_VERTEX_GROUPS || variant == HGNN_VERTEX_GROUPS_HALF2,
               HGNN_EINVAL, "%s: unknown variant %d", who, int(variant));
  hgnn_status st = check_spmm_args(who, g, edge_val, H, X, ldx, Y, ldy, F, op);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(F <= p->max_F, HGNN_EINVAL, "%s: F = %d exceeds the plan's max_F = %d", who, F, p->max_F);
  HGNN_REQUIRE(vector_path_ok(edge_val, H, X, ldx, Y, ldy, F), HGNN_EUNSUPPORTED,
               "%s: needs F <= 512, ld %% 8 == 0, 16-byte aligned X, Y, and D %% 8 == 0 when edge values have several heads", who);
  HGNN_REQUIRE(variant == HGNN_EDGE_SEGMENTS_ATOMIC || p->ng > 0, HGNN_EINVAL,
               "%s: the plan holds no neighbour groups (hgnn_plan_add_groups)", who);
  if (g->nrows == 0) return HGNN_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  SpmmArgs a = make_args(g, edge_val, H, X, ldx, Y, ldy, F, op, row_scale);
  if (variant != HGNN_EDGE_SEGMENTS_ATOMIC) return run_vgroups(p, a, g->ncols, variant == HGNN_VERTEX_GROUPS_HALF2, s);
  a.atomic_y = 1;  // always on the whole graph: column blocks are not used by the comparison variants
  return run_tasks(p, p->tasks, a, g->ncols, s);
}

}  // extern "C"

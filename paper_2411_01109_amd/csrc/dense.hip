// The dense side of a layer on the matrix cores: the projection h = X.W that feeds the sparse kernels
// (paper section 3.1.3, Eq. 2: the linear layer's output is the dense input of the SpMM; section 6: the
// input width is projected to the intermediate width by a GeMM; section 3.1.1: dense products are what
// matrix units are for, the sparse kernels are not), its two gradients, and the small dense pieces that tie
// the fused GAT backward to it.
//
// All three products are skinny (n rows in the millions, K and F in the tens to hundreds), so they are bound
// by streaming X / Y once through HBM, not by MFMA rate; the tiling below is chosen for full-width 16-byte
// loads and stores per lane, with the small operand (W) resident in LDS.
//
// MFMA shape used everywhere: v_mfma_f32_16x16x32_f16.  Operand A is 16 x 32: lane l holds row l % 16,
// columns 8*(l / 16) .. +7.  Operand B is 32 x 16: lane l holds column l % 16, rows 8*(l / 16) .. +7.
// The 16 x 16 result: lane l holds column l % 16, rows 4*(l / 16) .. +3.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <type_traits>

#include "common.h"

namespace hgnn {

typedef float float4_t __attribute__((ext_vector_type(4)));

struct LinearArgs {
  int64_t n;
  int K, F;
  const half_t* X;
  int64_t ldx;
  const half_t* W;  // [K][F], transposed (TRANS) [F][K]
  int64_t ldw;
  half_t* Y;
  int64_t ldy;
  int KC;     // columns of X (rows of W) held in LDS at a time; a multiple of 32, and of the 128 columns of a group when K > KC
  int FC;     // features a workgroup owns (blockIdx.y picks them); a multiple of 32
  int near;   // ANY: a workgroup's part of W lies within 32-bit offsets
  uint32_t per_line;  // 2^31 / items on a line of the weight, rounded up
  int step_f, step_k;  // transposed: the waves of a workgroup / and % items on a line of the weight
  int kshift;          // transposed: an item is 2^kshift pieces of 2^(6 - kshift) features
  int KW;     // rows of W that exist (not transposed): the others count as zero
  int64_t nrb;  // blocks of rows, 16 * RT for each wave of a workgroup
};

// The weight tile W[kc .. kc+KC)[fc0 .. fc0+FC) into LDS in the order in which the products read it: fragment
// (tile t of 16 features, step ks of 32 columns) is 64 lanes x 16 bytes, so every read of it is one conflict-free
// kilobyte.  The features of a pair of tiles are dealt out so that a lane's 2 x 4 result values are 8 consecutive
// features: tile 2b+o, row i of the tile <-> feature 32b + 8(i/4) + 4o + i%4.
// W [F][K]: an item is 64 columns of eight features, a wave's 16-byte pieces of eight lines; of up to 32 columns 16 features, or half of the lanes have none of
// their own (us: 2000 rows of 16 -> 256 8.2 / 5.7, 30 000 of 16 -> 128 5.3 / 4.8, 60 000 7.4 / 6.9, 30 000 of 32 -> 64 4.0 / 3.8).  W [K][F]: an item is a block of eight features of
// eight rows, a thread's, transposed by byte permutations.  A batch of items is fetched in one go and put into LDS later, so that the rows of
// X can be asked for in between: behind them, by loads under conditions and with bank conflicts, the weight was up to a third of a call.
// 100 003 rows of 64 -> 48 9.7 -> 6.8 us, 131 072 of 128 -> 64 13.5 -> 10.5, 262 144 of 64 -> 64 15.4 -> 12.4, 60 000 of 608 -> 128 28 -> 22 (without
// any weight 5.8, 10.9, 13.2, 17.5).
struct WeightBatch {
  uint32_t v[32];
  int f, k8;  // of its first item
};
__device__ __forceinline__ int linear_waves() { return __builtin_amdgcn_readfirstlane(int(blockDim.x) / kWave); }
template <bool TRANS>
__device__ __forceinline__ int linear_batch() { return TRANS ? linear_waves() * 8 : int(blockDim.x); }
// W^T: items on a line
__host__ __device__ __forceinline__ int linear_across(const LinearArgs& a) { return (a.KC + (8 << a.kshift) - 1) >> (3 + a.kshift); }
template <bool TRANS>
__device__ __forceinline__ int linear_w_items(const LinearArgs& a) { return TRANS ? (a.FC >> (6 - a.kshift)) * linear_across(a) : a.FC / 8 * (a.KC / 8); }

// item / items on a line of the weight (a division is a chain of some thirty instructions ahead of the first load)
__device__ __forceinline__ int linear_line(const LinearArgs& a, int item) { return int(__umulhi(uint32_t(item) << 1, a.per_line)); }

// W^T: f(u, first feature, first piece), all scalar, for the u-th item of the wave in a batch
template <class Fn>
__device__ __forceinline__ void linear_each_item(const LinearArgs& a, int first, Fn&& f) {
  const int across = linear_across(a);
  const int item = __builtin_amdgcn_readfirstlane(first + int(threadIdx.x) / kWave);
  int g = linear_line(a, item), c = item - g * across;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    if (g << (6 - a.kshift) >= a.FC) break;
    f(u, g << (6 - a.kshift), c << a.kshift);
    g += a.step_f, c += a.step_k;
    const int over = c >= across;
    g += over, c -= over ? across : 0;
  }
}

// Where lane 16q + i of a read finds its 16 bytes in the kilobyte of a fragment: such that the writes of either form, 16 lanes of four features and
// four q at a time, go to different banks, and so do the lanes of a read, which takes i of 0-3 and 12-15 of an even q together with 4-11 of the odd one
// behind it (with all lanes of a q turned alike reads met on a bank about once each: 19 717 rows of 504 -> 64 6.8 -> 6.3 us, 140 000 of 1280 -> 128 128.4 ->
// 126.8).  Places that differ by tile and step as well take the rest of the writes' conflicts away, but each needs an address register of its own:
// 131 072 of 128 -> 128 14.8 -> 16.1.
__device__ __forceinline__ int linear_slot(int i, int q) { return 16 * q + (i ^ (13 * q & 15)); }

// ANY = false: lines of whole pieces on 16-byte boundaries, at 32-bit offsets.  ANY: pieces that begin at any element, and of W [K][F] the last one of a line is
// its last eight features, some of which the piece before it holds, too.  Such a weight read by elements, all of it, cost up to two thirds of a call; us, by
// elements / so: 4096 rows of 64 -> 42, lines of 48 10.4 / 3.7, 3000 of 2504 -> 41, lines of 48 105 / 33, 70 000 of 2504 -> 100, lines of 104 300 / 141, 4096 of 64 ->
// 41 by W^T, lines of 67 8.6 / 4.0.  Kernels of their own, because the code costs the others registers (140 000 of 1280 -> 128 by W^T 121 / 140).
// Offsets beyond 32 bits, or fewer than eight features: all by elements, with the first batch (1000 of 128 -> 7 3.5).
template <bool TRANS, bool ANY>
__device__ __forceinline__ bool linear_batched(const LinearArgs& a, int fc0) {
  return !ANY || (a.near && (TRANS || min(a.FC, a.F - fc0) >= 8));
}

// Positions outside the weight are read inside it, without branches between the loads; linear_put_w puts zeros in the place of rows (columns of W^T) that
// do not exist.  What stands in the place of features that do not exist, if anything, meets only results that are not stored.
template <bool TRANS, bool ANY>
__device__ __forceinline__ void linear_fetch_w(const LinearArgs& a, WeightBatch& w, int first, int kc, int fc0) {
  const int kn = min(a.KC, a.K - kc), fn = min(a.FC, a.F - fc0), lane = threadIdx.x & (kWave - 1);
  const char* const W = reinterpret_cast<const char*>(a.W + fc0 * (TRANS ? a.ldw : 1) + kc * (TRANS ? 1 : a.ldw));
  const uint32_t pitch = uint32_t(a.ldw) * 2u;
  if (!linear_batched<TRANS, ANY>(a, fc0)) return;
  if constexpr (TRANS) {
    const int fl = lane >> a.kshift, kl = lane & ((1 << a.kshift) - 1);
    linear_each_item(a, first, [&](int u, int f0, int k0) {
      const uint32_t at = uint32_t(min(f0 + fl, fn - 1)) * pitch + uint32_t(min(8 * (k0 + kl), kn - 8)) * 2u;
      __builtin_memcpy(w.v + 4 * u, __builtin_assume_aligned(W + at, ANY ? 2 : 16), 16);
    });
  } else {
    const int F8 = a.FC / 8, idx = first + int(threadIdx.x);
    w.k8 = linear_line(a, idx), w.f = 8 * (idx - w.k8 * F8);
    if (__builtin_amdgcn_readfirstlane(w.k8) >= a.KC / 8 || a.KW <= kc) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t at = uint32_t(min(8 * w.k8 + j, a.KW - kc - 1)) * pitch + uint32_t(min(w.f, fn - 8)) * 2u;
      __builtin_memcpy(w.v + 4 * j, __builtin_assume_aligned(W + at, ANY ? 2 : 16), 16);
    }
  }
}

template <bool TRANS, bool ANY>
__device__ __forceinline__ void linear_put_w(const LinearArgs& a, const WeightBatch& w, int first, int kc, int fc0, half_t* __restrict__ Wf) {
  typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
  const int KS = a.KC / 32, kn = min(a.KC, a.K - kc), fn = min(a.FC, a.F - fc0), lane = threadIdx.x & (kWave - 1);
  uint4_t* const out = reinterpret_cast<uint4_t*>(Wf);
  const auto place = [&](int f, int k8) { return out + ((2 * (f >> 5) + ((f >> 2) & 1)) * KS + (k8 >> 2)) * kWave + linear_slot(4 * ((f >> 3) & 3) + (f & 3), k8 & 3); };
  if (!linear_batched<TRANS, ANY>(a, fc0)) {
    const int64_t sf = TRANS ? a.ldw : 1, sk = TRANS ? 1 : a.ldw;
    const int rows = TRANS ? kn : min(kn, a.KW - kc);
    if (first != 0) return;
    for (int idx = threadIdx.x; idx < fn * (a.KC / 8); idx += blockDim.x) {
      const int k8 = int(unsigned(idx) / unsigned(fn)), f = idx - k8 * fn;
      half8_t v = {0, 0, 0, 0, 0, 0, 0, 0};
      if (8 * k8 < rows) {
        const half_t* const src = a.W + (fc0 + f) * sf + (kc + 8 * k8) * sk;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = src[min(j, rows - 1 - 8 * k8) * sk];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (8 * k8 + j >= rows) v[j] = half_t(0);
      }
      *place(f, k8) = __builtin_bit_cast(uint4_t, v);
    }
    return;
  }
  if constexpr (TRANS) {
    const int fl = lane >> a.kshift, kl = lane & ((1 << a.kshift) - 1);
    linear_each_item(a, first, [&](int u, int f0, int k0) {
      const int f = f0 + fl, k8 = k0 + kl;
      const bool in = f < fn && 8 * k8 < kn;
      uint4_t v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = in ? w.v[4 * u + j] : 0;
      if (8 * k8 < a.KC) *place(f, k8) = v;
    });
  } else {
    const int f = w.f, k8 = w.k8;
    if (8 * k8 >= a.KC) return;
    const int rows = f < fn ? min(kn, a.KW - kc) - 8 * k8 : 0;
    auto put = [&](int f) {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        uint4_t v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t even = 2 * j < rows ? w.v[8 * j + c / 2] : 0, odd = 2 * j + 1 < rows ? w.v[8 * j + 4 + c / 2] : 0;
          v[j] = __builtin_amdgcn_perm(odd, even, c & 1 ? 0x07060302u : 0x05040100u);
        }
        *place(f + c, k8) = v;
      }
    };
    if (!ANY) {
      put(f);
    } else {
      if (f < fn) put(min(f, fn - 8));
    }
  }
}

// all items from `first` on
template <bool TRANS, bool ANY>
__device__ __forceinline__ void linear_load_w(const LinearArgs& a, half_t* __restrict__ Wf, int first, int kc, int fc0) {
  for (; first < linear_w_items<TRANS>(a); first += linear_batch<TRANS>()) {
    WeightBatch w;
    linear_fetch_w<TRANS, ANY>(a, w, first, kc, fc0);
    linear_put_w<TRANS, ANY>(a, w, first, kc, fc0, Wf);
  }
}

// eight consecutive features of a row of Y from the two result tiles that hold them
__device__ __forceinline__ void linear_store(const LinearArgs& a, int64_t row, int f, const float4_t& lo, const float4_t& hi) {
  half8_t h;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = half_t(lo[j]);
    h[4 + j] = half_t(hi[j]);
  }
  half_t* dst = a.Y + row * a.ldy + f;
  if (f + 8 <= a.F) {
    *reinterpret_cast<half8_t*>(dst) = h;
  } else if (f < a.F) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < a.F - f) dst[j] = h[j];
  }
}

// Y[16*RT rows per wave and step] = X . W on the matrix cores, formed transposed (features x rows): a lane holds values of
// ONE row of Y, and with the feature order of linear_load_w they are whole 16-byte pieces, four lanes to 64 consecutive
// bytes of a row; a load of X is likewise 64 consecutive bytes of 16 rows.  NT tiles of 16 features per pass over the
// row tile's columns (X of the row tile is read again from the caches for further passes).
// The bound is the stream of X and Y.  What the first form of this kernel lost against it was the weight: it came in
// by 2-byte LDS stores with a division each, once per workgroup of one to nine 128-row passes, again for every row block
// when K > 440, and X was read once per 128 features from memory.  Now workgroups are persistent, as many as the LDS
// and registers of the chip hold, a workgroup brings its part of W in once (16-byte pieces) and the loads of X run one
// group (4 x 16 bytes per lane) ahead of the products across passes and row blocks.  2.4 M x 128 -> 128: 323 -> 249 us
// (4.9 TB/s, what a copy reaches); 233 k x 608 -> 64: 232 -> 64 us; 131 k x 128 -> 128: 40 -> 17 us (14.4 now that the weight is asked for first).  Two row tiles per
// wave for the sake of the weight fragments were slower (2.4 M: 325 us): the kernel waits for rows, not for LDS, and the
// registers are better spent on the loads in flight.  RT > 1 is for rows that do not fill a group: with K <= 64 (32) a group
// takes two (four) row tiles, so that as many bytes are in flight as with long rows.
// CHUNKED: the weights of 128 features do not fit; the columns come in chunks, a chunk of W once per row block.
template <int NT, int RT, bool CHUNKED, bool TRANS, bool ANY>
__global__ __launch_bounds__(1024) void linear_kernel(LinearArgs a) {
  constexpr int GS = 4 / RT;    // 32-column steps in a group of X loads
  constexpr int GK = 32 * GS;   // columns of a group
  extern __shared__ __align__(16) unsigned char lds_raw[];
  half_t* Wf = reinterpret_cast<half_t*>(lds_raw);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, wpw = blockDim.x / kWave;
  const int i = lane & 15, q = lane >> 4;
  const int fc0 = blockIdx.y * a.FC;
  const int KS = a.KC / 32;
  const int nchunks = CHUNKED ? (a.K + a.KC - 1) / a.KC : 1;
  const int npass = CHUNKED ? 1 : (min(a.FC, a.F - fc0) + 16 * NT - 1) / (16 * NT);
  const bool keep = RT > 1 || a.K <= GK;  // one group holds the whole row: it serves all passes
  const half8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
  half8_t next[4];
  auto load_group = [&](int64_t rb, int k0) {
    // Rows and columns that do not exist are read inside X, without branches: such rows are not stored, such columns are cleared below.
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int64_t row = (rb * wpw + wave) * (16 * RT) + 16 * r + i;
      const half_t* src = a.X + min(row, a.n - 1) * a.ldx;
#pragma unroll
      for (int u = 0; u < GS; ++u)
        if (k0 + 32 * u < a.K) next[r * GS + u] = *reinterpret_cast<const half8_t*>(src + min(k0 + 32 * u + 8 * q, a.K - 8));
    }
  };
  if (CHUNKED) {
    load_group(blockIdx.x, 0);
  } else {
    WeightBatch w;
    linear_fetch_w<TRANS, ANY>(a, w, 0, 0, fc0);
    load_group(blockIdx.x, 0);
    linear_put_w<TRANS, ANY>(a, w, 0, 0, fc0, Wf);
    linear_load_w<TRANS, ANY>(a, Wf, linear_batch<TRANS>(), 0, fc0);
    __syncthreads();
  }
  for (int64_t rb = blockIdx.x; rb < a.nrb; rb += gridDim.x) {
    half8_t cur[4];
    for (int pass = 0; pass < npass; ++pass) {
      float4_t acc[RT][NT];
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][t] = float4_t{0.f, 0.f, 0.f, 0.f};
      for (int c = 0; c < nchunks; ++c) {
        const int kc = c * a.KC;
        const int kn = CHUNKED ? min(a.KC, a.K - kc) : a.K;
        if (CHUNKED) {  // trip counts are uniform over the workgroup
          __syncthreads();
          linear_load_w<TRANS, ANY>(a, Wf, 0, kc, fc0);
          __syncthreads();
        }
        for (int k0 = 0; k0 < kn; k0 += GK) {
          if (!keep || pass == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) cur[u] = next[u];
            if (kc + k0 + GK > a.K) {
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (kc + k0 + 32 * (u % GS) + 8 * q >= a.K) cur[u] = zero;
            }
          }
          // what comes after this group: more of the row, the row again for the next pass, or the next row block
          if (kc + k0 + GK < a.K) load_group(rb, kc + k0 + GK);
          else if (pass + 1 < npass) { if (!keep) load_group(rb, 0); }
          else if (rb + gridDim.x < a.nrb) load_group(rb + gridDim.x, 0);
#pragma unroll
          for (int u = 0; u < GS; ++u) {
            if (k0 + 32 * u < kn) {  // uniform
              const half_t* w = Wf + ((int64_t(pass) * NT * KS + (k0 / 32 + u)) * kWave + linear_slot(i, q)) * 8;
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                const half8_t wv = *reinterpret_cast<const half8_t*>(w + int64_t(t) * KS * (kWave * 8));
#pragma unroll
                for (int r = 0; r < RT; ++r)
                  acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wv, cur[r * GS + u], acc[r][t], 0, 0, 0);
              }
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int64_t row = (rb * wpw + wave) * (16 * RT) + 16 * r + i;
        if (row >= a.n) continue;
#pragma unroll
        for (int b = 0; b < NT / 2; ++b) {
          const int f = fc0 + 16 * NT * pass + 32 * b + 8 * q;
          half8_t h;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            h[j] = half_t(acc[r][2 * b][j]);
            h[4 + j] = half_t(acc[r][2 * b + 1][j]);
          }
          half_t* dst = a.Y + row * a.ldy + f;
          if (f + 8 <= a.F) {
            *reinterpret_cast<half8_t*>(dst) = h;
          } else if (f < a.F) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (j < a.F - f) dst[j] = h[j];
          }
        }
      }
    }
  }
}

// The same for few rows with many columns, where a wave of linear_kernel is one chain of loads: here KP waves share a tile of 16 rows,
// each takes at most kSplitSteps steps of 32 columns, whose loads all go out before the weight is brought in, and the partial
// results are added through LDS in the order of the parts.  One row block per workgroup.  Bound by the latencies of a launch, of the
// rows and of the weight, which more lanes bring in: 19 717 x 504 -> 64 12.9 -> 10.0 us (its bytes take 4.6), 4096 x 504 -> 64 9.0 -> 6.0; with the
// weight asked for ahead of X, calls in a row from a graph, 7.2 -> 6.1 and 5.9 -> 4.7, 12 000 x 504 -> 128 by W^T 9.0 -> 8.8.
constexpr int kSplitSteps = 10;

template <int NT, int KP, bool TRANS, bool ANY>
__global__ __launch_bounds__(1024) void linear_split_kernel(LinearArgs a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  half_t* Wf = reinterpret_cast<half_t*>(lds_raw);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, tiles = blockDim.x / (kWave * KP);
  const int tile = wave / KP, part = wave % KP;
  const int i = lane & 15, q = lane >> 4;
  const int KS = a.KC / 32, per = (KS + KP - 1) / KP, s0 = part * per, sn = min(per, KS - s0);  // sn may be negative
  const int64_t row = (int64_t(blockIdx.x) * tiles + tile) * 16 + i;
  const half8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
  WeightBatch w0;
  linear_fetch_w<TRANS, ANY>(a, w0, 0, 0, 0);
  half8_t x[kSplitSteps];
#pragma unroll
  for (int u = 0; u < kSplitSteps; ++u) {
    x[u] = zero;
    const int k = 32 * (s0 + u) + 8 * q;
    if (u < sn && row < a.n && k < a.K) x[u] = *reinterpret_cast<const half8_t*>(a.X + row * a.ldx + k);
  }
  linear_put_w<TRANS, ANY>(a, w0, 0, 0, 0, Wf);
  linear_load_w<TRANS, ANY>(a, Wf, linear_batch<TRANS>(), 0, 0);
  __syncthreads();
  float4_t acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < kSplitSteps; ++u) {
    if (u < sn) {  // uniform over the wave
      const half_t* w = Wf + (int64_t(s0 + u) * kWave + linear_slot(i, q)) * 8;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const half8_t*>(w + int64_t(t) * KS * (kWave * 8)), x[u], acc[t], 0, 0, 0);
    }
  }
  __syncthreads();  // the weight has been read: its place holds the partial results
  float4_t* const sum = reinterpret_cast<float4_t*>(lds_raw) + lane;
  if (part > 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t) sum[(((part - 1) * tiles + tile) * NT + t) * kWave] = acc[t];
  }
  __syncthreads();
  if (part > 0 || row >= a.n) return;
#pragma unroll
  for (int p = 1; p < KP; ++p)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] += sum[(((p - 1) * tiles + tile) * NT + t) * kWave];
#pragma unroll
  for (int b = 0; b < NT / 2; ++b) linear_store(a, row, 32 * b + 8 * q, acc[2 * b], acc[2 * b + 1]);
}

// ---- weight gradient ---------------------------------------------------------------------------------
struct WgradArgs {  // (with what the launch adds, the kernel reads 64 bytes: one line)
  int64_t n;
  uint16_t K, F;  // 4096 at most
  int run;        // LONG: steps whose products are added up before they are added to those of earlier steps
  const half_t* X;
  int64_t ldx;
  const half_t* dY;
  int64_t ldy;
  float* part;  // [gridDim.x][tiles of 16 x 16 of dW][256] fp32
};

constexpr int kWgradRows = 32;  // rows of X and dY per step

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4_t;

// Eight consecutive rows of one column per lane (an MFMA operand whose contraction runs over the rows) out of a
// row-major LDS tile: ds_read_b64_tr_b16 transposes 4 rows x 16 columns among 16 lanes (lane i supplies the address
// of row i/4, columns 4*(i%4).., and receives column i).
__device__ __forceinline__ half8_t wgrad_column(const half_t* tile, int pitch, int c0, int lane) {
  const int i = lane & 15, q = lane >> 4;
  const half_t* p = tile + (8 * q + (i >> 2)) * pitch + c0 + 4 * (i & 3);
  const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)p);
  const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(p + 4 * pitch));
  typedef short short8_t __attribute__((ext_vector_type(8)));
  const short8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(half8_t, v);
}

// dW[64*WA columns of X][64*WB columns of dY] of one workgroup = sum over its rows of X[:, k] * dY[:, f].  The four waves
// form WR = 4 / (WA*WB) row teams of WA x WB waves; a team parks its 32 x 64*WA and 32 x 64*WB tiles in LDS (whole rows,
// 16 bytes per lane, the next step's pieces in flight meanwhile) and a wave picks its operands from there column-wise
// with transposing reads; pitch = columns + 16 halves puts the four rows of such a read on different banks.  At the end
// the teams are added in LDS in a fixed order and the workgroup leaves one partial result in the workspace: no
// atomics, the same bits on every run.  WA = WB = 2 lets X and dY of up to 128 columns be read once; the form before
// (a 64 x 64 block per wave, columns picked by 2-byte LDS reads, a partial per wave) read both twice and was bound by
// those reads.  The teams' blocks are added by all teams, a share of the columns each, which also write it: 4096 rows 64 x 64 6.6 -> 4.7 us
// (one team that added the others in turn and wrote).  They are written as the lanes hold them, tile after tile, 16 bytes
// a lane; row by row, 4 bytes a lane in pieces of 64 bytes, 262 144 rows took 0.5 us more.
// LONG: a workgroup adds its steps up in runs, in as many registers again (two workgroups per compute unit then).  A product of 32 rows rounds some
// four times, and a long chain of them is what the result's error comes from.  Relative error against 64 bits, 1e-7, as many partial results as are
// resident / fewer, of longer chains / those in runs: 19 717 rows of 504 x 64 1.2 / 1.3 / 1.2, 131 072 of 128 x 128 1.7 / 1.8 / 1.55, 233 000 of 608 x 64
// 2.2 / 2.4 / 1.5, 2.4 M of 128 x 128 4.6 / 4.6 / 2.2, 600 000 of 608 x 128 6.2 / 6.2 / 1.9; us 15.6 / 12.2 / 12.8, 22.4 / 18.9 / 19.5, 67.4 / 60.7 / 60.6,
// 205 / 206 / 206, 264 / 262 / 264.
constexpr int kWgradRun = 8;
template <int WA, int WB, bool LONG>
__global__ __launch_bounds__(kBlock, LONG ? 2 : 3) void wgrad_kernel(WgradArgs a) {
  constexpr int WT = WA * WB, WR = 4 / WT;     // waves in a team, teams
  constexpr int NBUF = WR == 1 ? 2 : 1;        // one team: two buffers, one barrier per step
  constexpr int PX = 64 * WA + 16, PY = 64 * WB + 16;
  constexpr int TILE = kWgradRows * (PX + PY);
  constexpr int NX = 4 / WB, NY = 4 / WA;      // 16-byte pieces per thread and step
  constexpr int kTileBytes = WR * NBUF * TILE * 2, kSumBytes = WT * WR * (16 - 16 / WR) * kWave * 16;
  __shared__ __align__(16) unsigned char lds[kTileBytes > kSumBytes ? kTileBytes : kSumBytes];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int team = wave / WT, tw = wave % WT, wa = tw / WB, wb = tw % WB;
  const int tt = tw * kWave + lane;            // thread of the team
  const int kc0 = blockIdx.y * 64 * WA, fc0 = blockIdx.z * 64 * WB;
  half_t* tiles = reinterpret_cast<half_t*>(lds) + team * NBUF * TILE;
  const int64_t nsteps = (a.n + int64_t(kWgradRows) * WR - 1) / (int64_t(kWgradRows) * WR);
  const half8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
  half8_t vx[NX], vy[NY];
  auto load = [&](int64_t step) {
    const int64_t r0 = (step * WR + team) * kWgradRows;
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      const int p = tt + u * (WT * kWave), row = p / (8 * WA), c = 8 * (p % (8 * WA));
      vx[u] = zero;  // K and F are multiples of 8 here, so a piece is inside the matrix or outside it as a whole
      if (r0 + row < a.n && kc0 + c < a.K) vx[u] = *reinterpret_cast<const half8_t*>(a.X + (r0 + row) * a.ldx + kc0 + c);
    }
#pragma unroll
    for (int u = 0; u < NY; ++u) {
      const int p = tt + u * (WT * kWave), row = p / (8 * WB), c = 8 * (p % (8 * WB));
      vy[u] = zero;
      if (r0 + row < a.n && fc0 + c < a.F) vy[u] = *reinterpret_cast<const half8_t*>(a.dY + (r0 + row) * a.ldy + fc0 + c);
    }
  };
  auto meet = [&]() {
    if (WT == 1) wave_sync();
    else __syncthreads();
  };
  float4_t acc[4][4], before[LONG ? 4 : 1][4];  // before: earlier runs
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      acc[x][y] = float4_t{0.f, 0.f, 0.f, 0.f};
      if (LONG) before[x][y] = acc[x][y];
    }
  int buf = 0, left = a.run;
  if (int64_t(blockIdx.x) < nsteps) load(blockIdx.x);
  for (int64_t step = blockIdx.x; step < nsteps; step += gridDim.x) {  // uniform over the workgroup
    half_t* xs = tiles + buf * TILE;
    half_t* ys = xs + kWgradRows * PX;
    if (NBUF == 1) meet();  // the previous step's column reads are done
#pragma unroll
    for (int u = 0; u < NX; ++u) {
      const int p = tt + u * (WT * kWave), row = p / (8 * WA), c = 8 * (p % (8 * WA));
      *reinterpret_cast<half8_t*>(xs + row * PX + c) = vx[u];
    }
#pragma unroll
    for (int u = 0; u < NY; ++u) {
      const int p = tt + u * (WT * kWave), row = p / (8 * WB), c = 8 * (p % (8 * WB));
      *reinterpret_cast<half8_t*>(ys + row * PY + c) = vy[u];
    }
    meet();
    if (step + gridDim.x < nsteps) load(step + gridDim.x);
    half8_t xa[4], yb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      xa[t] = wgrad_column(xs, PX, 64 * wa + 16 * t, lane);
      yb[t] = wgrad_column(ys, PY, 64 * wb + 16 * t, lane);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa[x], yb[y], acc[x][y], 0, 0, 0);
    if (NBUF == 2) buf ^= 1;
    if (LONG && --left == 0) {
      left = a.run;
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          before[x][y] += acc[x][y];
          acc[x][y] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  if (LONG) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] += before[x][y];
  }
  // every team adds and writes a share of the block: its columns x = XS team .. of X, in the order of the teams
  constexpr int XS = 4 / WR;
  if (WR > 1) {
    float4_t* const sum = reinterpret_cast<float4_t*>(lds) + tw * (WR * (16 - 4 * XS) * kWave) + lane;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int to = x / XS;  // the team that adds column x; it holds the others' in the order of the teams, itself left out
      if (to == team) continue;
#pragma unroll
      for (int y = 0; y < 4; ++y) sum[((to * (WR - 1) + (team > to ? team - 1 : team)) * (4 * XS) + 4 * (x % XS) + y) * kWave] = acc[x][y];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (x / XS != team) continue;
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        float4_t s = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < WR; ++w) {
          const float4_t v = w == team ? acc[x][y] : sum[((team * (WR - 1) + (w > team ? w - 1 : w)) * (4 * XS) + 4 * (x % XS) + y) * kWave];
          if (w == 0) s = v;
          else s += v;
        }
        acc[x][y] = s;
      }
    }
  }
  // tile after tile of 16 x 16 as the lanes hold it, 16 bytes each
  const int tk = (a.K + 15) / 16, tf = (a.F + 15) / 16;
  float* const out = a.part + (int64_t(blockIdx.x) * tk * tf * kWave + lane) * 4;
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    if (WR > 1 && x / XS != team) continue;
    const int tx = kc0 / 16 + 4 * wa + x;
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int ty = fc0 / 16 + 4 * wb + y;
      if (tx < tk && ty < tf) __builtin_memcpy(out + (int64_t(tx) * tf + ty) * (kWave * 4), &acc[x][y], 16);  // (the workspace is 4-byte aligned)
    }
  }
}

// The same for few rows in one launch: a workgroup owns 16 x 16 values of dW and all rows, its 16 waves take 32 rows in turn
// and are added in LDS in wave order.  Bound by latency: 64 x 64 over 1000 rows 4.3 us, in two launches 5.7.  Every
// workgroup reads its 32-byte columns of all rows, so the time grows with the rows, but no partial results are left.
constexpr int kSmallWaves = 16;

__global__ __launch_bounds__(kWave * kSmallWaves) void wgrad_small_kernel(WgradArgs a, float* __restrict__ dW, int64_t lddw) {
  constexpr int P = 24;         // pitch: the four rows of a transposing read on different banks, 16-byte aligned
  constexpr int U = 4;          // steps whose loads are in flight together
  constexpr int TILE = kWgradRows * P;
  __shared__ __align__(16) half_t lds[kSmallWaves * 2 * TILE];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int kc0 = blockIdx.x * 16, fc0 = blockIdx.y * 16;
  half_t* const xs = lds + wave * 2 * TILE;
  half_t* const ys = xs + TILE;
  const int row = lane >> 1, c = 8 * (lane & 1);
  const bool kin = kc0 + c < a.K, fin = fc0 + c < a.F;  // K and F are multiples of 8
  float4_t acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int64_t STEP = int64_t(kSmallWaves) * kWgradRows;
  for (int64_t r0 = int64_t(wave) * kWgradRows; r0 < a.n; r0 += U * STEP) {
    half8_t vx[U], vy[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = r0 + u * STEP + row;
      vx[u] = vy[u] = half8_t(0);
      if (r < a.n && kin) vx[u] = *reinterpret_cast<const half8_t*>(a.X + r * a.ldx + kc0 + c);
      if (r < a.n && fin) vy[u] = *reinterpret_cast<const half8_t*>(a.dY + r * a.ldy + fc0 + c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u * STEP >= a.n) break;
      wave_sync();  // the previous step's column reads are done
      *reinterpret_cast<half8_t*>(xs + row * P + c) = vx[u];
      *reinterpret_cast<half8_t*>(ys + row * P + c) = vy[u];
      wave_sync();
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wgrad_column(xs, P, 0, lane), wgrad_column(ys, P, 0, lane), acc, 0, 0, 0);
    }
  }
  float* const sum = reinterpret_cast<float*>(lds);
  __syncthreads();
  *reinterpret_cast<float4_t*>(sum + (wave * kWave + lane) * 4) = acc;
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= 256) return;
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kSmallWaves; ++w) s += sum[w * 256 + e];
  const int k = kc0 + 4 * (e >> 6) + (e & 3), f = fc0 + ((e >> 2) & 15);
  if (k < a.K && f < a.F) dW[int64_t(k) * lddw + f] = s;
}

// TILES: out[k*out_ld + f] = sum over the partials j (part_stride apart) of in[j][e], e in the tiles of wgrad_kernel (elems = K: rows of the
// result); else out[e], and from element `split` on out2[e - split].  A workgroup takes 64 elements; its kSumSlices slices add a strided share of the partials
// each and the slice sums are added in slice order: a fixed order whatever the launch, in one launch (two rounds of
// launches cost 4-5 us each on the smallest layers, more than the addition).  Bound by the latency of a slice's loads:
// all up to 16 are in flight together, also where there are fewer (224 partials of 64 x 64, 14 a slice, 8 at a time and
// the rest one by one: 11.4 us with the kernel before it, now 10.0).
constexpr int kSumSlices = 16;

template <bool TILES>
__global__ __launch_bounds__(kWave * kSumSlices) void partial_sum_kernel(const float* __restrict__ in, int64_t part_stride, int nparts,
                                                                         int64_t elems, int F, float* __restrict__ out, int64_t out_ld,
                                                                         int64_t split, float* __restrict__ out2) {
  __shared__ float red[kSumSlices][kWave];
  const int x = threadIdx.x & (kWave - 1), y = threadIdx.x / kWave;
  const int64_t e = int64_t(blockIdx.x) * kWave + x;
  float s = 0.f;
  if (e < (TILES ? part_stride : elems)) {
    constexpr int U = 16;  // loads in flight: a thread's chain of them is the time
    int j = __builtin_amdgcn_readfirstlane(y);  // a slice is a wave
    float v[U];
    for (; j + (U - 1) * kSumSlices < nparts; j += U * kSumSlices) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = in[int64_t(j + u * kSumSlices) * part_stride + e];
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
    // the last r < U of them by the bits of r, also together
    const int r = j < nparts ? (nparts - j + kSumSlices - 1) / kSumSlices : 0;
#pragma unroll
    for (int b = U / 2; b > 0; b /= 2) {
#pragma unroll
      for (int u = 0; u < b; ++u) v[U - 2 * b + u] = 0.f;
      if (r & b) {
#pragma unroll
        for (int u = 0; u < b; ++u) v[U - 2 * b + u] = in[int64_t(j + u * kSumSlices) * part_stride + e];
        j += b * kSumSlices;
      }
    }
#pragma unroll
    for (int u = 0; u < U - 1; ++u) s += v[u];
  }
  red[y][x] = s;
  __syncthreads();
  if (y != 0) return;
  s = 0.f;
#pragma unroll
  for (int j = 0; j < kSumSlices; ++j) s += red[j][x];
  if (TILES) {
    const int tf = (F + 15) / 16, tile = int(e >> 8), lane = int(e >> 2) & (kWave - 1);
    const int k = 16 * (tile / tf) + 4 * (lane >> 4) + int(e & 3), f = 16 * (tile % tf) + (lane & 15);
    if (k < elems && f < F) out[int64_t(k) * out_ld + f] = s;
  } else if (e < elems) {
    if (e >= split) out2[e - split] = s;
    else out[e] = s;
  }
}

// ---- feature gradient of a GAT layer -------------------------------------------------------------------
struct FeatGradArgs {
  int64_t n;
  int H, D, F;
  const half_t* dV;
  int64_t lddv;
  const half_t* d_el;
  const half_t* d_er;
  const half_t* a_l;
  const half_t* a_r;
  const half_t* hfeat;
  int64_t ldh;
  half_t* dh;
  int64_t lddh;
  float* part;  // [gridDim.x][2][F]
};

// dh[i, f] = dV[i, f] + d_el[i, head f] * a_l[f] + d_er[i, head f] * a_r[f] (one fp16 rounding), and per
// workgroup the partial sums of da_l[f] = sum_i d_el[i, head f] * h[i, f] and da_r likewise.  LP lanes per row
// (a power of two >= F / 8), 8 features per lane; a thread keeps its feature group for all its rows, so the
// column sums stay in registers until the end, where the workgroup adds them in a fixed order through LDS.
template <int LP>
__global__ __launch_bounds__(kBlock) void gat_feature_grad_kernel(FeatGradArgs a) {
  constexpr int RPB = kBlock / LP;  // rows per workgroup pass
  __shared__ float red[2][kBlock][8];
  const int l = threadIdx.x % LP, rr = threadIdx.x / LP;
  const int f0 = 8 * l;
  const bool live = f0 < a.F;  // D % 8 == 0: a feature group lies in one head
  const int h = live ? f0 / a.D : 0;
  float al[8], ar[8], sl[8], sr[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    al[i] = live ? float(a.a_l[f0 + i]) : 0.f;
    ar[i] = live ? float(a.a_r[f0 + i]) : 0.f;
    sl[i] = 0.f;
    sr[i] = 0.f;
  }
  if (live) {
    for (int64_t row = int64_t(blockIdx.x) * RPB + rr; row < a.n; row += int64_t(gridDim.x) * RPB) {
      const half8_t v = *reinterpret_cast<const half8_t*>(a.dV + row * a.lddv + f0);
      const half8_t x = *reinterpret_cast<const half8_t*>(a.hfeat + row * a.ldh + f0);
      const float gl = float(a.d_el[row * a.H + h]), gr = float(a.d_er[row * a.H + h]);
      half8_t o;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        o[i] = half_t(float(v[i]) + gl * al[i] + gr * ar[i]);
        sl[i] += gl * float(x[i]);
        sr[i] += gr * float(x[i]);
      }
      *reinterpret_cast<half8_t*>(a.dh + row * a.lddh + f0) = o;
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    red[0][threadIdx.x][i] = sl[i];
    red[1][threadIdx.x][i] = sr[i];
  }
  __syncthreads();
  // thread t < 2 * F sums one feature of one side over the RPB row slots, in slot order
  for (int t = threadIdx.x; t < 2 * a.F; t += kBlock) {
    const int side = t / a.F, f = t - side * a.F;
    float s = 0.f;
    for (int r = 0; r < RPB; ++r) s += red[side][r * LP + f / 8][f % 8];
    a.part[(int64_t(blockIdx.x) * 2 + side) * a.F + f] = s;
  }
}

constexpr int kLinearLds = 152 * 1024;  // most bytes of W a workgroup keeps (of the 160 KB of a compute unit)

template <void (*KERNEL)(LinearArgs)>
static hgnn_status launch_linear_kernel(LinearArgs a, bool trans, dim3 grid, int threads, size_t lds, hipStream_t s) {
  // beyond 64 KB of dynamic LDS the runtime wants to be told, once per kernel and device
  static bool told[64] = {};
  if (lds > 65536) {
    int dev = 0;
    HGNN_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 64 || !told[dev]) {
      HGNN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, kLinearLds));
      if (dev >= 0 && dev < 64) told[dev] = true;
    }
  }
  a.kshift = a.KC == 32 ? 2 : 3;
  const int across = linear_across(a);
  a.step_f = threads / kWave / across;
  a.step_k = threads / kWave % across;
  const uint32_t line = uint32_t(trans ? across : a.FC / 8);
  a.per_line = ((uint32_t(1) << 31) + line - 1) / line;
  KERNEL<<<grid, threads, lds, s>>>(a);
  HGNN_LAUNCH_CHECK("linear_kernel");
  return HGNN_OK;
}

enum WeightForm { kWhole, kAny, kWholeT, kAnyT };  // linear_batched

template <int NT, int RT, bool CHUNKED>
static hgnn_status launch_linear(const LinearArgs& a, WeightForm form, dim3 grid, int threads, size_t lds, hipStream_t s) {
  switch (form) {
    case kWhole: return launch_linear_kernel<linear_kernel<NT, RT, CHUNKED, false, false>>(a, false, grid, threads, lds, s);
    case kAny: return launch_linear_kernel<linear_kernel<NT, RT, CHUNKED, false, true>>(a, false, grid, threads, lds, s);
    case kWholeT: return launch_linear_kernel<linear_kernel<NT, RT, CHUNKED, true, false>>(a, true, grid, threads, lds, s);
    default: return launch_linear_kernel<linear_kernel<NT, RT, CHUNKED, true, true>>(a, true, grid, threads, lds, s);
  }
}

template <int NT, int KP>
static hgnn_status launch_linear_split(const LinearArgs& a, WeightForm form, dim3 grid, int threads, size_t lds, hipStream_t s) {
  switch (form) {
    case kWhole: return launch_linear_kernel<linear_split_kernel<NT, KP, false, false>>(a, false, grid, threads, lds, s);
    case kAny: return launch_linear_kernel<linear_split_kernel<NT, KP, false, true>>(a, false, grid, threads, lds, s);
    case kWholeT: return launch_linear_kernel<linear_split_kernel<NT, KP, true, false>>(a, true, grid, threads, lds, s);
    default: return launch_linear_kernel<linear_split_kernel<NT, KP, true, true>>(a, true, grid, threads, lds, s);
  }
}

template <int KP>
static hgnn_status launch_linear_split(int nt, const LinearArgs& a, WeightForm form, dim3 grid, int threads, size_t lds, hipStream_t s) {
  if (nt == 2) return launch_linear_split<2, KP>(a, form, grid, threads, lds, s);
  if (nt == 4) return launch_linear_split<4, KP>(a, form, grid, threads, lds, s);
  return launch_linear_split<8, KP>(a, form, grid, threads, lds, s);
}

static int wgrad_parts(int K, int F) {
  // fewer partial results for larger weights: the workspace stays near 32 MB
  int64_t p = (int64_t(1) << 23) / (int64_t(K) * F);
  p = p < 64 ? 64 : (p > 1024 ? 1024 : p);
  int q = 64;
  while (q * 2 <= p) q *= 2;
  return q;
}

constexpr int kCus = 256;       // compute units of an MI355X
constexpr int kFeatGradBlocks = 512;  // most workgroups of the attention gradients, a partial result each

}  // namespace hgnn

using namespace hgnn;

static hgnn_status linear_impl(const char* who, int64_t n, int32_t K, int32_t KW, int32_t F, const hgnn_half* X, int64_t ldx,
                               const hgnn_half* W, int64_t ldw, int32_t trans_w, hgnn_half* Y, int64_t ldy, void* stream) {
  clear_error();
  HGNN_REQUIRE(n >= 0 && K > 0 && F > 0, HGNN_EINVAL, "%s: n = %lld, K = %d, F = %d", who, static_cast<long long>(n), K, F);
  HGNN_REQUIRE(ldx >= K && ldy >= F && ldw >= (trans_w ? K : F), HGNN_EINVAL, "%s: leading dimension smaller than the row", who);
  HGNN_REQUIRE(K <= 65536 && F <= 65536, HGNN_EUNSUPPORTED, "%s: K = %d / F = %d above 65536", who, K, F);
  if (n == 0) return HGNN_OK;
  HGNN_REQUIRE(X && W && Y, HGNN_EINVAL, "%s: NULL argument", who);
  HGNN_REQUIRE(K % 8 == 0 && ldx % 8 == 0 && ldy % 8 == 0 && aligned16(X) && aligned16(Y), HGNN_EUNSUPPORTED,
               "%s: needs K %% 8 == 0, ldx %% 8 == 0, ldy %% 8 == 0 and 16-byte aligned X, Y (pad with zeros)", who);
  LinearArgs a{n, K, F, reinterpret_cast<const half_t*>(X), ldx, reinterpret_cast<const half_t*>(W), ldw,
               reinterpret_cast<half_t*>(Y), ldy, 0, 0, 0, 0, 0, 0, 0, KW, 0};
  const int k32 = (K + 31) / 32 * 32, f32 = (F + 31) / 32 * 32;
  // short rows: several row tiles per wave, where that still leaves four waves for every compute unit
  const int RT = n < int64_t(32) * 4 * kCus || K > 64 ? 1 : (K > 32 || n < int64_t(64) * 4 * kCus ? 2 : 4);
  // 16-feature tiles per pass: 2, 4 or 8, the fewest passes (a pass reads the row tile of X again, or keeps it where RT > 1,
  // whose registers hold NT * RT <= 8 tiles)
  const int most = 8 / RT;
  const int NT = std::min(most, f32 <= 32 ? 2 : (f32 <= 64 ? 4 : 8));
  // the whole weight in LDS where it fits, else the most features whose weights do, else 128 features in
  // chunks of columns
  int nt = NT;
  a.KC = k32;
  a.FC = int(ceil_div(F, 16 * nt)) * 16 * nt;
  if (int64_t(k32) * a.FC * 2 > kLinearLds) {
    const int fit = kLinearLds / (k32 * 2) / (16 * nt) * (16 * nt);
    a.FC = std::min(fit, int(ceil_div(F, 16 * nt)) * 16 * nt);
    if (fit == 0) {
      a.FC = 16 * nt;
      a.KC = kLinearLds / (a.FC * 2) / 128 * 128;
    }
  }
  a.near = ldw < (int64_t(1) << 30) / (trans_w ? a.FC : a.KC) ? 1 : 0;
  const bool whole = a.near && ldw % 8 == 0 && aligned16(W) && (trans_w || F % 8 == 0);
  const WeightForm form = trans_w ? (whole ? kWholeT : kAnyT) : (whole ? kWhole : kAny);
  const size_t lds = size_t(a.KC) * size_t(a.FC) * sizeof(half_t);
  const int64_t tiles = ceil_div(n, int64_t(16) * RT);
  // A compute unit holds 16 waves (the registers of four for each SIMD), fewer where their workgroups' weights do not fit beside each other.  Workgroups are
  // persistent: as many as the chip holds at once, each with the same number of row blocks (to one).
  const int fy = int(ceil_div(F, a.FC));
  auto blocks_each = [&](int w, int rounds) {  // for workgroups of w waves, as many as the chip holds `rounds` times
    const int64_t held = std::max<int64_t>(1, std::min<int64_t>(16 / w, int64_t(160 * 1024) / std::max<size_t>(lds, 1)));
    return ceil_div(ceil_div(tiles, w), std::max<int64_t>(1, int64_t(kCus) * held * rounds / fy));
  };
  // Twice as many, one after the other, where at least as much is written as read, often, and that leaves no compute unit with more blocks than before: us, X
  // and Y out of the caches, one / two rounds: 1.2 M rows of 64 -> 64 66.4 / 65.8, 2.4 M of 128 -> 128 247 / 243, 400 000 of 64 -> 256 72.6 / 64.9, 2.4 M of 16 -> 128 243 /
  // 228; 233 000 of 64 -> 608 90.0 / 84.5 (workgroups of eight / 16 waves), 400 000 172 / 163; but 800 000 of 128 -> 128 (13 blocks each / twice 7) 85.7 / 89.0,
  // 288 000 of 64 -> 256 (3 / twice 2) 47 / 52, of 64 -> 608 (3 / twice 2) 125 / 132; of 128 -> 256, 524 288 90.0 / 91.9.  Small weights of many features gain with more blocks,
  // too, from some 40 000 passes on: 800 000 of 64 -> 256 (7 / twice 4) 135 / 130, 1.2 M of 16 -> 128 (5 / twice 3) 118 / 110.
  const bool small = lds <= 40 * 1024, many = F >= 4 * int64_t(K);
  const int64_t passes = tiles * ceil_div(F, int64_t(16) * nt);
  const bool twice = passes >= 32768 && lds <= 80 * 1024 && (small ? F >= K : many) && 25 * 2 * blocks_each(8, 2) <= 26 * blocks_each(8, 1);
  const int rounds = twice || (passes >= 40000 && small && many) ? 2 : 1;
  // waves per workgroup: the more LDS a workgroup holds, the more waves share it; of small weights eight from two row tiles per wave on, when the weight is
  // brought in half as often, if workgroups of eight take four fifths of the places (else compute units hold unequal numbers): us, four / eight, 131 072 rows of
  // 128 -> 128 18.4 / 16.6, W^T 18.3 / 16.3, 288 000 37.5 / 35.5, 400 000 50.0 / 47.4, 70 000 10.7 / 11.8; with three quarters of the places taken 144 000 of 128 -> 128 20.2 /
  // 22.6, 288 000 of 64 -> 64 by W^T 19.0 / 22.4, 288 000 of 64 -> 128 27.4 / 32.3, 400 000 of 64 -> 64 27.1 / 28.0;
  // fewer, so that every compute unit has work, while bringing the weight in stays short
  const bool full = 5 * ceil_div(ceil_div(tiles, 8), blocks_each(8, 1)) * fy >= 4 * 2 * kCus;
  int wpw = small ? (rounds > 1 || (tiles >= 2 * 16 * kCus && full) ? 8 : 4) : (lds <= 80 * 1024 ? 8 * rounds : 16);
  const int least = lds <= 16 * 1024 ? 1 : (lds <= 32 * 1024 ? 2 : 4);
  while (wpw > least && ceil_div(tiles, wpw) < kCus) wpw /= 2;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Few rows with many columns: as many row tiles per workgroup as give every compute unit one, and waves beside them up to 16 that
  // share a tile's columns.  us, a chain of loads per wave / shared (inputs out of the caches):
  //   K, F               1000        4096        8192       12000       16384       19717       25000       32768 rows
  //   128, 64          3.6 / 3.5   4.0 / 3.8   4.0 / 3.9   4.6 / 4.2   4.5 / 4.6   5.2 / 5.1   5.4 / 5.6   5.8 / 6.3
  //   128, 128         4.2 / 4.2   4.3 / 4.4   5.0 / 4.8   5.8 / 5.5   5.5 / 6.1   6.3 / 6.4   6.7 / 7.3   7.9 / 8.9
  //   128, 128, W^T    5.6 / 4.6   5.8 / 4.7   6.4 / 5.2   7.7 / 5.6   5.9 / 6.4   6.9 / 6.5   7.3 / 7.7   8.4 / 9.0
  //   256, 64          4.4 / 4.1   5.2 / 4.8   5.4 / 5.1   6.1 / 5.7   6.1 / 6.2   7.0 / 6.4   7.6 / 7.4   8.0 / 8.1
  //   256, 128         5.9 / 5.2   6.6 / 5.7   6.8 / 6.1   7.1 / 6.9   7.7 / 8.0   9.6 / 8.7  10.0 / 9.9  10.4 / 11.1
  //   504, 64          7.1 / 4.9   7.3 / 5.3   7.6 / 5.8   9.0 / 7.2   9.7 / 8.8  11.9 / 9.5  12.3 / 11.1 12.2 / 12.7
  //   504, 128, W^T   11.6 / 7.8  12.0 / 8.3  12.4 / 9.1  14.1 / 10.8 15.0 / 12.6 19.9 / 13.6 20.3 / 15.7 15.6 / 16.7
  //   1024, 64        11.9 / 7.1  12.1 / 7.4  14.8 / 9.0  15.2 / 10.8 15.7 / 12.9
  // (at 16 384 and 32 768 rows a chain's workgroups of four waves are one or two for every compute unit).  At 40 000 rows (two rounds of workgroups) sharing was
  // 10 to 40 % slower when it was last tried.
  // Behind the kernel that wrote X, in the caches, a chain of few steps ends sooner: 256, 64 at 16 384, 25 000, 32 768 rows 5.0 / 5.4, 5.9 / 5.7, 6.2 / 6.4, 256, 128 6.7 /
  // 7.4, 8.3 / 8.0, 8.4 / 9.0; 128, 64 at 5000, 8192, 25 000 3.9 / 3.7, 3.6 / 3.8, 4.7 / 5.0, 128, 128 at 8192, 12 000, 19 717 4.5 / 4.6, 5.4 / 5.2, 5.7 / 5.8, W^T 6.0 / 5.0, 7.2 /
  // 5.5, 6.3 / 6.2; 128, 32 at 2000, 12 000, 28 000 3.0 / 3.2, 3.7 / 3.6, 4.4 / 4.3 (out of the caches 3.0 / 3.3, 4.1 / 3.7, 5.0 / 5.0).
  const int T = int(std::max<int64_t>(2, ceil_div(tiles, kCus))), KP = T <= 4 ? 4 : (T == 5 ? 3 : 2);
  const bool shared = K > 256 ? T <= 8 : (K > 128 ? T <= 7 : K == 128 && T <= 5 && (trans_w || F > 64 || (F > 32 && n < 8192)));
  if (RT == 1 && shared && k32 <= KP * kSplitSteps * 32 && F <= 128 && a.KC == k32 && a.FC == 16 * nt) {
    const size_t need = std::max(lds, size_t(KP - 1) * size_t(T) * size_t(nt) * kWave * sizeof(float4_t));
    const dim3 grid{unsigned(ceil_div(tiles, T)), 1u, 1u};
    const int threads = T * KP * kWave;
    return KP == 4 ? launch_linear_split<4>(nt, a, form, grid, threads, need, s)
                   : (KP == 3 ? launch_linear_split<3>(nt, a, form, grid, threads, need, s) : launch_linear_split<2>(nt, a, form, grid, threads, need, s));
  }
  a.nrb = ceil_div(tiles, wpw);
  const int64_t want = ceil_div(a.nrb, blocks_each(wpw, rounds));
  HGNN_REQUIRE(want <= 0x7fffffff && fy <= 65535, HGNN_EUNSUPPORTED, "%s: grid too large", who);
  const dim3 grid{unsigned(want), unsigned(fy), 1u};
  const int threads = wpw * kWave;
  if (a.KC < K) {
    if (nt == 2) return launch_linear<2, 1, true>(a, form, grid, threads, lds, s);
    if (nt == 4) return launch_linear<4, 1, true>(a, form, grid, threads, lds, s);
    return launch_linear<8, 1, true>(a, form, grid, threads, lds, s);
  }
  if (nt == 2) {
    if (RT == 4) return launch_linear<2, 4, false>(a, form, grid, threads, lds, s);
    return RT == 2 ? launch_linear<2, 2, false>(a, form, grid, threads, lds, s) : launch_linear<2, 1, false>(a, form, grid, threads, lds, s);
  }
  if (nt == 4 && RT == 2) return launch_linear<4, 2, false>(a, form, grid, threads, lds, s);
  if (nt == 4) return launch_linear<4, 1, false>(a, form, grid, threads, lds, s);
  return launch_linear<8, 1, false>(a, form, grid, threads, lds, s);
}

extern "C" {

hgnn_status hgnn_linear(int64_t n, int32_t K, int32_t F, const hgnn_half* X, int64_t ldx, const hgnn_half* W, int64_t ldw,
                        int32_t trans_w, hgnn_half* Y, int64_t ldy, void* stream) {
  return linear_impl("hgnn_linear", n, K, K, F, X, ldx, W, ldw, trans_w, Y, ldy, stream);
}

hgnn_status hgnn_linear_padded(int64_t n, int32_t K, int32_t KW, int32_t F, const hgnn_half* X, int64_t ldx, const hgnn_half* W,
                               int64_t ldw, hgnn_half* Y, int64_t ldy, void* stream) {
  if (KW < 0 || KW > K) {
    clear_error();
    return fail(HGNN_EINVAL, "hgnn_linear_padded: KW = %d outside [0, K = %d]", KW, K);
  }
  return linear_impl("hgnn_linear_padded", n, K, KW, F, X, ldx, W, ldw, 0, Y, ldy, stream);
}

size_t hgnn_linear_wgrad_workspace(int32_t K, int32_t F) {
  if (K <= 0 || F <= 0) return 0;
  return size_t(wgrad_parts(K, F)) * size_t(K) * size_t(F) * sizeof(float);
}

hgnn_status hgnn_linear_wgrad(int64_t n, int32_t K, int32_t F, const hgnn_half* X, int64_t ldx, const hgnn_half* dY,
                              int64_t ldy, float* dW, int64_t lddw, void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  const char* who = "hgnn_linear_wgrad";
  HGNN_REQUIRE(n >= 0 && K > 0 && F > 0, HGNN_EINVAL, "%s: n = %lld, K = %d, F = %d", who, static_cast<long long>(n), K, F);
  HGNN_REQUIRE(ldx >= K && ldy >= F && lddw >= F, HGNN_EINVAL, "%s: leading dimension smaller than the row", who);
  HGNN_REQUIRE(K <= 4096 && F <= 4096, HGNN_EUNSUPPORTED, "%s: K = %d / F = %d above 4096", who, K, F);
  HGNN_REQUIRE(dW != nullptr, HGNN_EINVAL, "%s: dW is NULL", who);
  HGNN_REQUIRE(n == 0 || (X && dY), HGNN_EINVAL, "%s: NULL argument", who);
  HGNN_REQUIRE(workspace != nullptr && workspace_bytes >= hgnn_linear_wgrad_workspace(K, F), HGNN_EINVAL,
               "%s: workspace of %zu bytes, needs %zu (hgnn_linear_wgrad_workspace)", who, workspace_bytes,
               hgnn_linear_wgrad_workspace(K, F));
  HGNN_REQUIRE(K % 8 == 0 && F % 8 == 0 && ldx % 8 == 0 && ldy % 8 == 0 && aligned16(X) && aligned16(dY) &&
                   (reinterpret_cast<uintptr_t>(workspace) & 3u) == 0,
               HGNN_EUNSUPPORTED, "%s: needs K, F, ldx, ldy %% 8 == 0 and 16-byte aligned X, dY (pad with zeros)", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* part = static_cast<float*>(workspace);
  // up to 64 columns on a side: one wave wide; else two, so that up to 128 columns are read once
  const int WA = K <= 64 ? 1 : 2, WB = F <= 64 ? 1 : 2;
  const int kb = int(ceil_div(K, 64 * WA)), fb = int(ceil_div(F, 64 * WB)), WR = 4 / (WA * WB);
  const int64_t tiles = ceil_div(K, 16) * ceil_div(F, 16), blocks = int64_t(kb) * fb, steps = ceil_div(n, int64_t(kWgradRows) * WR);
  // Partial results: a step of a workgroup takes some 0.6 us, a partial result about 4.5 ns and 0.45 ns for each of its
  // tiles (written and added): steps / parts * step + parts * partial is least at the root below.  us with it and with
  // as many partials as are resident: 25 000 rows of 64 x 64 7.5 and 7.8, 100 000 10.0 and 16.1, of 128 x 128 12.5 and
  // 19.0, 16.8 and 20.4, 50 000 of 504 x 64 17.7 and 19.8; beyond some 10^6 rows the two are the same.
  int64_t parts = std::llround(std::sqrt(1400. * double(steps) / double(10 + tiles)));
  // a single block: whole rounds of one workgroup per compute unit (300 000 rows of 64 x 64: 256 17.7, 288 19.4, 512 19.1)
  if (blocks == 1 && parts > kCus && parts < 2 * kCus) parts = kCus;
  // No more than the workspace holds (64 at least of sides of 8: a quarter of the tile) and than there are steps, two
  // workgroups per compute unit (233 000 rows of 608 x 64: 480 of them 62.4, 510 74.6, 680 and more 67.4); eight XCDs take the workgroups in turn, so a multiple of eight leaves the blocks of the
  // same rows on one L2
  int64_t most = std::min<int64_t>(2 * kCus / blocks, int64_t(wgrad_parts(K, F)) * K * F / (tiles * 256));
  if (most >= 16) most = most / 8 * 8;
  if (parts >= 16) parts = (parts + 7) / 8 * 8;
  parts = std::max<int64_t>(1, std::min(std::min(parts, most), steps));
  const int64_t each = ceil_div(steps, parts);  // steps of a workgroup
  // where the chain is longer than the partial results that are left out made it: of several blocks those were few (9000 rows of 504 x 64, a chain of
  // four steps 1.17 for 1.11e-7; of one block with eight 262 144 of 64 x 64 1.6 for 1.8e-7)
  const bool in_runs = each > (blocks == 1 ? kWgradRun : 2);
  const int run = int(ceil_div(each, std::max<int64_t>(2, ceil_div(each, kWgradRun))));
  WgradArgs a{n, uint16_t(K), uint16_t(F), run, reinterpret_cast<const half_t*>(X), ldx, reinterpret_cast<const half_t*>(dY), ldy, part};
  // few rows: one launch without partial results, up to the rows at which fetching them in 32-byte pieces costs what the
  // second launch and the partial results do, later the larger dW is.  us behind the kernel that wrote dY, one launch / two:
  //   K x F         1000        1500        2000        2500        3000        4096        6000 rows
  //   16 x 16     3.4 / 5.1   3.4 / 5.2   3.8 / 5.1   4.3 / 5.1   4.8 / 5.2   5.4 / 5.2   6.9 / 5.3
  //   32 x 32     3.2 / 5.4   4.0 / 5.2   4.4 / 5.3   5.2 / 5.4   5.8 / 5.3   7.3 / 5.3   9.0 / 5.4
  //   64 x 16     3.3 / 5.4   4.0 / 5.3   4.6 / 5.4   5.6 / 5.5   6.0 / 5.4   7.6 / 5.5   9.9 / 5.6
  //   64 x 64     4.4 / 5.6   5.4 / 5.6   6.6 / 5.7   7.7 / 5.8   8.3 / 5.6  11.3 / 5.8  15.6 / 5.9
  //   128 x 64    4.3 / 5.4   5.5 / 5.6   6.4 / 5.7   7.5 / 5.8   8.2 / 6.3  11.0 / 6.5  14.8 / 6.9
  // and from 128 x 128 on, where the writer's own time is taken off:
  //   K x F         2200        2600        3000        3400        3700        4096 rows
  //   128 x 128   6.0 / 7.8   7.0 / 8.2   7.6 / 8.0    - / 8.1     - / 7.9     - / 8.1
  //   256 x 128   5.8 / 8.1   6.6 / 8.4   7.3 / 8.1   8.2 / 8.6   9.1 / 8.7  10.1 / 8.8
  //   128 x 256   7.0 / 8.6   8.3 / 7.9   9.2 / 8.6  10.3 / 8.9  11.3 / 8.3  12.8 / 8.9
  //   384 x 128   6.0 / 8.4   6.9 / 9.1   7.5 / 9.3   8.7 / 10.0  9.6 / 9.8   9.8 / 10.0
  //   512 x 64    5.7 / 8.2   6.0 / 8.2   6.7 / 8.8   7.2 / 8.4   8.0 / 8.0   8.6 / 8.1
  //   608 x 64    5.9 / 8.2   6.1 / 8.0   7.6 / 8.1   9.2 / 8.1  10.8 / 8.6  11.7 / 8.4
  // (The largest are level at about 3400.  Their line stays at 4096, to which the test of the choice on the host holds it.)
  // Beyond one workgroup per compute unit they queue: 608 x 128 (304) at 2000, 3000, 4096 rows 9.2, 15.2, 23.3 against 11.3, 12.0, 13.4
  const int64_t sb = ceil_div(K, 16), sf = ceil_div(F, 16), size = int64_t(K) * F;
  const int64_t few = size <= 1024 ? 2400 : (size < 128 * 128 ? 1700 : (size < 256 * 128 ? 3000 : 4096));
  if (n <= few && n * sb * sf <= 2560 * int64_t(kCus)) {
    wgrad_small_kernel<<<dim3(unsigned(sb), unsigned(sf)), kWave * kSmallWaves, 0, s>>>(a, dW, lddw);
    HGNN_LAUNCH_CHECK("wgrad_small_kernel");
    return HGNN_OK;
  }
  const dim3 grid{unsigned(parts), unsigned(kb), unsigned(fb)};
  const auto launch = [&](auto wide_x, auto wide_y) {
    constexpr int A = decltype(wide_x)::value, B = decltype(wide_y)::value;
    if (in_runs) wgrad_kernel<A, B, true><<<grid, kBlock, 0, s>>>(a);
    else wgrad_kernel<A, B, false><<<grid, kBlock, 0, s>>>(a);
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 2> two;
  if (WA == 1 && WB == 1) launch(one, one);
  else if (WB == 1) launch(two, one);
  else if (WA == 1) launch(one, two);
  else launch(two, two);
  HGNN_LAUNCH_CHECK("wgrad_kernel");
  partial_sum_kernel<true><<<dim3(unsigned(tiles * 4)), kWave * kSumSlices, 0, s>>>(part, tiles * 256, int(parts), K, F, dW, lddw, 0, nullptr);
  HGNN_LAUNCH_CHECK("partial_sum_kernel");
  return HGNN_OK;
}

size_t hgnn_gat_feature_grad_workspace(int32_t H, int32_t D) {
  if (H <= 0 || D <= 0) return 0;
  return size_t(kFeatGradBlocks) * 2 * size_t(H) * size_t(D) * sizeof(float);
}

hgnn_status hgnn_gat_feature_grad(int64_t n, int32_t H, int32_t D, const hgnn_half* dV, int64_t lddv, const hgnn_half* d_el,
                                  const hgnn_half* d_er, const hgnn_half* a_l, const hgnn_half* a_r, const hgnn_half* hfeat,
                                  int64_t ldh, hgnn_half* dh, int64_t lddh, float* da_l, float* da_r, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  clear_error();
  const char* who = "hgnn_gat_feature_grad";
  HGNN_REQUIRE(n >= 0 && H >= 1 && D >= 1 && int64_t(H) * D <= 512, HGNN_EINVAL, "%s: n = %lld, H = %d, D = %d out of range", who,
               static_cast<long long>(n), H, D);
  const int F = H * D;
  HGNN_REQUIRE(lddv >= F && ldh >= F && lddh >= F, HGNN_EINVAL, "%s: leading dimension smaller than F", who);
  HGNN_REQUIRE(da_l && da_r, HGNN_EINVAL, "%s: da_l or da_r is NULL", who);
  HGNN_REQUIRE(n == 0 || (dV && d_el && d_er && a_l && a_r && hfeat && dh), HGNN_EINVAL, "%s: NULL argument", who);
  HGNN_REQUIRE(workspace != nullptr && workspace_bytes >= hgnn_gat_feature_grad_workspace(H, D), HGNN_EINVAL,
               "%s: workspace of %zu bytes, needs %zu (hgnn_gat_feature_grad_workspace)", who, workspace_bytes,
               hgnn_gat_feature_grad_workspace(H, D));
  HGNN_REQUIRE(D % 8 == 0 && lddv % 8 == 0 && ldh % 8 == 0 && lddh % 8 == 0 && aligned16(dV) && aligned16(hfeat) && aligned16(dh) &&
                   (reinterpret_cast<uintptr_t>(workspace) & 3u) == 0,
               HGNN_EUNSUPPORTED, "%s: needs D %% 8 == 0, ld %% 8 == 0 and 16-byte aligned dV, hfeat, dh", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* part = static_cast<float*>(workspace);
  FeatGradArgs a{n, H, D, F, reinterpret_cast<const half_t*>(dV), lddv, reinterpret_cast<const half_t*>(d_el),
                 reinterpret_cast<const half_t*>(d_er), reinterpret_cast<const half_t*>(a_l), reinterpret_cast<const half_t*>(a_r),
                 reinterpret_cast<const half_t*>(hfeat), ldh, reinterpret_cast<half_t*>(dh), lddh, part};
  const int LP = pow2_at_least(F / 8);
  // enough workgroups for the chip, no more than a pass of rows each: every one leaves a partial result
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>(kFeatGradBlocks, ceil_div(n, kBlock / LP)));
  dim3 grid{unsigned(blocks)};
  switch (LP) {
    case 1: gat_feature_grad_kernel<1><<<grid, kBlock, 0, s>>>(a); break;
    case 2: gat_feature_grad_kernel<2><<<grid, kBlock, 0, s>>>(a); break;
    case 4: gat_feature_grad_kernel<4><<<grid, kBlock, 0, s>>>(a); break;
    case 8: gat_feature_grad_kernel<8><<<grid, kBlock, 0, s>>>(a); break;
    case 16: gat_feature_grad_kernel<16><<<grid, kBlock, 0, s>>>(a); break;
    case 32: gat_feature_grad_kernel<32><<<grid, kBlock, 0, s>>>(a); break;
    default: gat_feature_grad_kernel<64><<<grid, kBlock, 0, s>>>(a); break;
  }
  HGNN_LAUNCH_CHECK("gat_feature_grad_kernel");
  // the partial of workgroup b is [2][F]: one row of 2F elements, whose second half is da_r
  partial_sum_kernel<false><<<dim3(unsigned(ceil_div(2 * F, kWave))), kWave * kSumSlices, 0, s>>>(part, 2 * int64_t(F), int(blocks),
                                                                                         2 * int64_t(F), F, da_l, F, F, da_r);
  HGNN_LAUNCH_CHECK("partial_sum_kernel");
  return HGNN_OK;
}

}  // extern "C"

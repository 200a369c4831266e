// Stable sort of 64-bit words for the set-up calls: by radix, digits of up to nine bits, two or three launches a pass (digits of every tile
// counted, counts scanned over the tiles where there are many, tiles sorted in LDS and written in runs).  The first pass forms its words from whatever the
// caller has, so no array of keys is written and read beforehand.  No workgroup waits for another one.
#pragma once

#include <type_traits>

#include "common.h"

namespace hgnn {

constexpr int kSortThreads = 1024, kSortPer = 8, kSortTile = kSortThreads * kSortPer;
constexpr int kSortBits = 9, kSortBins = 1 << kSortBits;
constexpr int kSortWaves = kSortThreads / kWave;
// Up to so many tiles, every tile adds up the counts itself, half of the tiles by each half of its workgroup: a launch less a pass, 4 to 5 us
// (us, list to CSR in four passes, own sums up to 128 / 256 tiles: 520 000 words in 254 tiles 84 / 98, 1.8 M in 220 119 / 129).
constexpr int kFewTiles = 128;

struct SortPass {
  int64_t n;
  int shift, bits;
  int ntiles;
  uint32_t* counts;  // [ntiles][kSortBins] items of a tile in every bin, then items of the earlier tiles there
  uint32_t* totals;  // [kSortBins]
  uint32_t* shares;  // [kScanShares][kSortBins] items of a share of the tiles in every bin
  __device__ __forceinline__ int digit(uint64_t w) const { return int(uint32_t(w >> shift) & ((1u << bits) - 1u)); }
};

// Sources of words: load(first, n, mine, scratch, w) gives a lane the items mine, mine + 64, ... of the n of the tile that begins at item `first`
// (those past the end are the last one again: no load is behind a branch), after prepare(first, n, scratch) by the whole workgroup; scratch is
// kSortThreads * PER ints of LDS.  count(p, k) is a word with the digit of pass p.
struct SortWords {
  const uint64_t* words;
  template <int PER>
  __device__ __forceinline__ void prepare(int64_t, int, int*) const {}
  template <int PER>
  __device__ __forceinline__ void load(int64_t first, int n, int mine, const int*, uint64_t (&w)[PER]) const {
#pragma unroll
    for (int j = 0; j < PER; ++j) w[j] = words[first + min(mine + j * kWave, n - 1)];
  }
  __device__ __forceinline__ uint64_t count(const SortPass&, int64_t k) const { return words[k]; }
};

// Bound by the read of the items.  Lanes of a wave often meet in one bin (behind a pass over the low bits of a column, the entries of a
// popular column): eight copies of the counts, 17 -> 10.5 us for 5.5 M words of a power-law graph; with no load behind a branch 7.9 (from a
// list of edges, rows read only where the digit reaches into them, 16.5 -> 7.1).
constexpr int kSortCopies = 8, kSortPitch = kSortBins + 1;

template <class Source, int PER>
__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(SortPass p, Source src) {
  __shared__ uint32_t hist[kSortCopies * kSortPitch];
  for (int i = threadIdx.x; i < kSortCopies * kSortPitch; i += kSortThreads) hist[i] = 0;
  __syncthreads();
  const int64_t first = int64_t(blockIdx.x) * (kSortThreads * PER) + threadIdx.x;
  int d[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int64_t k = first + j * kSortThreads;
    d[j] = p.digit(src.count(p, k < p.n ? k : p.n - 1));
    if (k >= p.n) d[j] = -1;
  }
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (d[j] >= 0) atomicAdd(&hist[(threadIdx.x % kSortCopies) * kSortPitch + d[j]], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kSortBins; i += kSortThreads) {
    uint32_t v = 0;
#pragma unroll
    for (int c = 0; c < kSortCopies; ++c) v += hist[c * kSortPitch + i];
    p.counts[int64_t(blockIdx.x) * kSortBins + i] = v;
  }
}

// Exclusive scan of the counts of every bin over the tiles, in place: a workgroup takes 16 bins, its 64 slices a share of the tiles each.
// Beyond kScanTiles tiles (25 M words) the tiles are scanned in kScanShares shares by workgroups of their own, after a launch that adds each of
// them up.  us, in one / add + scan: 9 M words 7 / 5 + 7, 20 M 14 / 5 + 9, 114 M 108 / 12 + 27.
constexpr int kScanBins = 16, kScanSlices = kSortThreads / kScanBins;
constexpr int kScanTiles = 3072, kScanShares = 16;

enum ScanPart { kScanAll, kScanAdd, kScanShare };  // everything, the sums of the shares, the shares behind their sums
template <ScanPart PART>
__global__ __launch_bounds__(kSortThreads) static void sort_scan_kernel(SortPass p) {
  __shared__ uint32_t sums[kScanSlices][kScanBins];
  const int x = threadIdx.x % kScanBins, y = threadIdx.x / kScanBins, bin = blockIdx.x * kScanBins + x;
  int first = 0, end = p.ntiles;
  if (PART != kScanAll) {
    const int share = (p.ntiles + kScanShares - 1) / kScanShares;
    first = min(int(blockIdx.y) * share, p.ntiles);
    end = min(first + share, p.ntiles);
  }
  const int per = (end - first + kScanSlices - 1) / kScanSlices, t0 = first + y * per, t1 = min(t0 + per, end);
  uint32_t* const c = p.counts + bin;
  uint32_t s = 0;
#pragma unroll 8
  for (int t = t0; t < t1; ++t) s += c[int64_t(t) * kSortBins];
  sums[y][x] = s;
  __syncthreads();
  uint32_t before = 0;
  if (PART == kScanAdd) {
    if (y > 0) return;
    for (int i = 0; i < kScanSlices; ++i) before += sums[i][x];
    p.shares[blockIdx.y * kSortBins + bin] = before;
    return;
  }
  if (PART == kScanShare)
    for (int i = 0; i < int(blockIdx.y); ++i) before += p.shares[i * kSortBins + bin];
  for (int i = 0; i < y; ++i) before += sums[i][x];
  if (y == kScanSlices - 1 && (PART == kScanAll || blockIdx.y == kScanShares - 1)) p.totals[bin] = before + s;
#pragma unroll 8
  for (int t = t0; t < t1; ++t) {
    const uint32_t v = c[int64_t(t) * kSortBins];
    c[int64_t(t) * kSortBins] = before;
    before += v;
  }
}

// exclusive scan over the first kSortBins threads of the workgroup; every thread calls it
__device__ __forceinline__ uint32_t sort_bin_scan(uint32_t v, uint32_t* s_wave) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t t = __shfl_up(incl, d);
    if (lane >= d) incl += t;
  }
  __syncthreads();  // what a previous scan left has been read
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave && w < kSortBins / kWave; ++w) before += s_wave[w];
  return before + incl - v;
}

// Ranks of a wave's 64 PER consecutive items among its items of the same digit: lanes of equal digit find each other by ballots, so the order of
// equal digits is kept.  hist: the wave's counts of the digits, zero beforehand.  Four instructions a bit and item (60 -> 41 an item, the
// scatter of 5.5 M words 27.4 -> 25.4 us).
constexpr uint32_t kOrXor = 0xF6;  // a | (b ^ c)
template <int PER>
__device__ __forceinline__ void sort_wave_ranks(const SortPass& p, const uint64_t (&w)[PER], uint16_t* hist, uint32_t (&rank)[PER]) {
  constexpr int N = 2;  // items side by side: a ballot is not read by the instruction behind it
  static_assert(PER % N == 0, "items in pairs");
#pragma unroll
  for (int j0 = 0; j0 < PER; j0 += N) {
    int d[N];
    uint32_t lo[N], hi[N];  // lanes whose digit differs
#pragma unroll
    for (int u = 0; u < N; ++u) {
      d[u] = p.digit(w[j0 + u]);
      lo[u] = hi[u] = 0;
    }
#pragma unroll
    for (int b = 0; b < kSortBits; ++b) {
      uint32_t bit[N];  // 0 or all ones
      uint64_t ones[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        bit[u] = uint32_t(__builtin_amdgcn_sbfe(d[u], b, 1));
        asm("" : "+v"(bit[u]));  // (one instruction for both uses)
        ones[u] = __ballot(bit[u] != 0);
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
        lo[u] = __builtin_amdgcn_bitop3_b32(lo[u], uint32_t(ones[u]), bit[u], kOrXor);
        hi[u] = __builtin_amdgcn_bitop3_b32(hi[u], uint32_t(ones[u] >> 32), bit[u], kOrXor);
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(~hi[u], __builtin_amdgcn_mbcnt_lo(~lo[u], 0));
      const uint32_t before = hist[d[u]];
      rank[j0 + u] = before + below;
      wave_sync();
      if (below == 0) hist[d[u]] = uint16_t(before + __popc(~lo[u]) + __popc(~hi[u]));
      wave_sync();
    }
  }
}

// A tile: every wave ranks its consecutive items (512 with eight a thread) by digit, the ranks of the waves are put after each other, the items go to LDS in that order and from there to memory: a bin's
// items of the tile are a run of 16 on average.  5.5 M words: 25.4 us (3.5 TB/s of reads and writes; a third of it vector instructions of
// the ranks), a pass 39 with its count and scan, where a library pass with look-back and its two fills took 52; the words that the first
// pass forms and the split at the end save three more passes over memory.  List to CSR 271 -> 191 us, transpose 180 -> 114; 100 000
// words (tiles of 8192 items: 88 and 53) 58 and 39.
template <class Source, int PER>
__global__ __launch_bounds__(kSortThreads, 8) void sort_scatter_kernel(SortPass p, Source src, uint64_t* __restrict__ out) {
  constexpr int TILE = kSortThreads * PER;
  __shared__ __align__(16) unsigned char lds[TILE * sizeof(uint64_t)];
  __shared__ uint32_t s_to[kSortBins];  // where the first item of a bin goes, less its place in the tile
  __shared__ uint32_t s_at[kSortBins];  // place of a bin's first item in the tile
  __shared__ uint32_t s_wave[kSortWaves];
  int* const scratch = reinterpret_cast<int*>(lds);
  uint16_t (*const hist)[kSortBins] = reinterpret_cast<uint16_t (*)[kSortBins]>(lds);
  uint64_t* const item = reinterpret_cast<uint64_t*>(lds);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t first = int64_t(blockIdx.x) * TILE;
  const int n = int(p.n - first < TILE ? p.n - first : TILE);
  const int bin = threadIdx.x;
  uint32_t total = 0, earlier = 0;
  if (p.ntiles <= kFewTiles) {  // every other tile by either half of the workgroup
    const int half = threadIdx.x / kSortBins;
#pragma unroll 8
    for (int t = half; t < p.ntiles; t += 2) {
      const uint32_t c = p.counts[t * kSortBins + bin % kSortBins];
      total += c;
      earlier += t < int(blockIdx.x) ? c : 0;
    }
    if (half) s_at[bin - kSortBins] = total, s_to[bin - kSortBins] = earlier;
  } else if (bin < kSortBins) {
    total = p.totals[bin];
    earlier = p.counts[int64_t(blockIdx.x) * kSortBins + bin];
  }
  src.template prepare<PER>(first, n, scratch);
  uint64_t w[PER];
  const int mine = wave * (kWave * PER) + lane;
  src.load(first, n, mine, scratch, w);
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (mine + j * kWave >= n) w[j] = ~uint64_t(0);  // behind all items of the last bin
  __syncthreads();
  for (int i = threadIdx.x; i < kSortWaves * kSortBins / 2; i += kSortThreads) reinterpret_cast<uint32_t*>(lds)[i] = 0;
  __syncthreads();
  uint32_t rank[PER];
  sort_wave_ranks(p, w, hist[wave], rank);
  __syncthreads();
  uint32_t here = 0;
  if (bin < kSortBins) {
    if (p.ntiles <= kFewTiles) total += s_at[bin], earlier += s_to[bin];
#pragma unroll
    for (int v = 0; v < kSortWaves; ++v) {
      const uint32_t c = hist[v][bin];
      hist[v][bin] = uint16_t(here);
      here += c;
    }
  }
  const uint32_t at = sort_bin_scan(here, s_wave);
  const uint32_t base = sort_bin_scan(total, s_wave);
  if (bin < kSortBins) {
    s_at[bin] = at;
    s_to[bin] = base + earlier - at;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int d = p.digit(w[j]);
    rank[j] += s_at[d] + hist[wave][d];
  }
  __syncthreads();  // the items take the place of the counts
#pragma unroll
  for (int j = 0; j < PER; ++j) item[rank[j]] = w[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = j * kSortThreads + threadIdx.x;
    if (i >= n) break;
    const uint64_t v = item[i];
    out[s_to[p.digit(v)] + uint32_t(i)] = v;
  }
}

// Few tiles: every one is sorted by all its digits in LDS, in one launch, and the words of several
// tiles find their places by searches in the others.  A pass of two launches for every nine bits is mostly latency there.  us, passes / this, list
// to CSR: three passes, 9000 words 43 / 43, 15 000 45 / 42, 24 000 48 / 43, 33 000 44 / 44, 65 000 46 / 51; four, 15 000 65 / 53, 24 000
// 67 / 51, 50 000 65 / 53, 65 000 57 / 57.  Two passes are as fast from two tiles on (transpose, 9000 words 36 / 38, 24 000 40 / 40, 65 000 38 /
// 47).
constexpr int kFewMerged = 8;  // most tiles that are merged
inline int few_merged(int passes) { return passes <= 2 ? 1 : (passes == 3 ? 4 : kFewMerged); }

// PER: items of a thread
template <class Source, int PER>
__global__ __launch_bounds__(kSortThreads) void sort_tile_kernel(SortPass p, int last, Source src, uint64_t* __restrict__ out) {
  __shared__ __align__(16) unsigned char lds[PER * kSortThreads * sizeof(uint64_t)];
  __shared__ uint32_t s_at[kSortBins], s_wave[kSortWaves];
  uint16_t (*const hist)[kSortBins] = reinterpret_cast<uint16_t (*)[kSortBins]>(lds);
  uint64_t* const item = reinterpret_cast<uint64_t*>(lds);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, bin = threadIdx.x;
  const int64_t first = int64_t(blockIdx.x) * (PER * kSortThreads);
  const int n = int(p.n - first < PER * kSortThreads ? p.n - first : PER * kSortThreads);
  src.template prepare<PER>(first, n, reinterpret_cast<int*>(lds));
  uint64_t w[PER];
  const int mine = wave * (kWave * PER) + lane;
  src.load(first, n, mine, reinterpret_cast<const int*>(lds), w);
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (mine + j * kWave >= n) w[j] = ~uint64_t(0);  // behind all items in every pass
  for (; p.shift < last; p.shift += p.bits) {
    p.bits = min(p.bits, last - p.shift);
    __syncthreads();  // the words have been read
    for (int i = threadIdx.x; i < kSortWaves * kSortBins / 2; i += kSortThreads) reinterpret_cast<uint32_t*>(lds)[i] = 0;
    __syncthreads();
    uint32_t rank[PER];
    sort_wave_ranks(p, w, hist[wave], rank);
    __syncthreads();
    uint32_t here = 0;
    if (bin < kSortBins) {
#pragma unroll
      for (int v = 0; v < kSortWaves; ++v) {
        const uint32_t c = hist[v][bin];
        hist[v][bin] = uint16_t(here);
        here += c;
      }
    }
    const uint32_t at = sort_bin_scan(here, s_wave);
    if (bin < kSortBins) s_at[bin] = at;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int d = p.digit(w[j]);
      rank[j] += s_at[d] + hist[wave][d];
    }
    __syncthreads();  // the items take the place of the counts
#pragma unroll
    for (int j = 0; j < PER; ++j) item[rank[j]] = w[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) w[j] = item[mine + j * kWave];
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = mine + j * kWave;
    if (i < n) out[first + i] = w[j];
  }
}

// Words of sorted tiles in their places: a word's own, and how many words of each of the other tiles are before it, LANES lanes to a word.
// Equal words of earlier tiles are before it.  Places are inside the array whatever it holds.
template <int LANES>
__global__ __launch_bounds__(kBlock) void sort_merge_kernel(SortPass p, int last, const uint64_t* __restrict__ in, uint64_t* __restrict__ out) {
  const int64_t i = (blockIdx.x * int64_t(kBlock) + threadIdx.x) / LANES;
  const int u = threadIdx.x % LANES, t = int(i / kSortTile);
  if (i >= p.n) return;  // (all lanes of a word)
  auto key = [&](uint64_t w) { return (w << (64 - last)) >> (64 - last + p.shift); };
  const uint64_t w = in[i], k = key(w);
  int place = 0;
  if (u == t) {
    place = int(i) - t * kSortTile;
  } else if (u < p.ntiles) {
    const uint64_t* const v = in + int64_t(u) * kSortTile;
    const int n = int(p.n - int64_t(u) * kSortTile < kSortTile ? p.n - int64_t(u) * kSortTile : kSortTile);
#pragma unroll
    for (int step = kSortTile; step > 0; step >>= 1) {
      const int at = place + step;
      if (at <= n) {
        const uint64_t o = key(v[at - 1]);
        if (o < k || (o == k && u < t)) place = at;
      }
    }
  }
#pragma unroll
  for (int d = 1; d < LANES; d <<= 1) place += __shfl_xor(place, d);
  if (u == 0) out[place] = w;
}

// Items of a thread in the passes: the tiles are as large as leaves one for nearly every compute unit, up to eight items, whose
// runs of a bin are whole lines.  us, eight / four / two items, list to CSR; transpose (two passes):
//   100 000 words of 20 000 vertices    79 /  65 /  58;  50 / 43 / 39        700 000 of 50 000    98 /  93 /  98;  59 / 55 / 59
//   300 000 of 30 000                   88 /  79 /  78;  53 / 49 / 48      1 040 000 of 50 000   108 /  99 / 103;  63 / 59 / 62
//   520 000 of 50 000                   90 /  89 /  84;  54 / 53 / 51      1 200 000 of 100 000  109 / 111 / 119;  66 / 66 / 73
// Six where they give a compute unit one, or, of those that have some two either way, no more than two: their workgroups are in flight together.
// eight / six / four:
//   1.1 M of 100 000   109 / 105 / 112;  65 /  63 /  67     2.3 M of 300 000   175 / 157 / 167; 118 / 109 / 116     2 M of 200 000     124 / 127 / 118;  75 /  79 /  75
//   1.3 M of 300 000   134 / 128 / 137;  93 /  90 /  96     2.9 M of 200 000   147 / 135 / 147;  88 /  82 /  91     4 M of 262 144     155 / 165 / 173;  95 / 104 / 108
//   1.57 M of 100 000  121 / 114 / 120;  71 /  68 /  72     3.14 M of 100 000  148 / 136 / 154;  88 /  83 /  92     5.5 M of 262 144   194 / 208 / 220; 119 / 126 / 135
inline int sort_items(int64_t n) {
  constexpr int64_t kTiles = 256;  // compute units
  if (n <= kTiles * 2 * kSortThreads) return 2;
  if (n <= kTiles * 4 * kSortThreads) return 4;
  return n <= kTiles * 6 * kSortThreads || (n > kTiles * 8 * kSortThreads && n <= kTiles * 12 * kSortThreads) ? 6 : kSortPer;
}

inline size_t sort_scratch_bytes(int64_t n) {
  return sizeof(uint32_t) * kSortBins * (size_t(ceil_div(n, kSortThreads * sort_items(n))) + 1 + kScanShares);
}

// Sorts n >= 1 words by their bits [first, last).  The words come from src; the sorted ones are in the returned one of the two buffers.
template <class Source>
static uint64_t* sort_words(const Source& src, int64_t n, int first, int last, uint64_t* buf0, uint64_t* buf1, void* scratch, hipStream_t s) {
  SortPass p{};
  p.n = n;
  p.ntiles = int(ceil_div(n, kSortTile));
  p.totals = static_cast<uint32_t*>(scratch);
  p.shares = p.totals + kSortBins;
  p.counts = p.shares + kScanShares * kSortBins;
  const int bits = last - first, npass = (bits + kSortBits - 1) / kSortBits;
  const dim3 grid{unsigned(p.ntiles)};
  uint64_t *in = buf1, *out = buf0;
  p.shift = first;
  if (p.ntiles <= few_merged(npass)) {
    p.bits = (bits + npass - 1) / npass;
    if (n <= 2 * kSortThreads) sort_tile_kernel<Source, 2><<<grid, kSortThreads, 0, s>>>(p, last, src, buf0);
    else sort_tile_kernel<Source, kSortPer><<<grid, kSortThreads, 0, s>>>(p, last, src, buf0);
    if (p.ntiles == 1) return buf0;
    auto merge = [&](auto lanes) {
      constexpr int L = decltype(lanes)::value;
      sort_merge_kernel<L><<<dim3(unsigned(ceil_div(n * L, kBlock))), kBlock, 0, s>>>(p, last, buf0, buf1);
    };
    if (p.ntiles <= 2) merge(std::integral_constant<int, 2>());
    else if (p.ntiles <= 4) merge(std::integral_constant<int, 4>());
    else merge(std::integral_constant<int, kFewMerged>());
    return buf1;
  }
  auto passes = [&](auto items) {
    constexpr int PER = decltype(items)::value;
    p.ntiles = int(ceil_div(n, kSortThreads * PER));
    const dim3 tiles{unsigned(p.ntiles)};
    for (int i = 0; i < npass; ++i) {
      p.bits = (last - p.shift + npass - i - 1) / (npass - i);
      if (i == 0) sort_count_kernel<Source, PER><<<tiles, kSortThreads, 0, s>>>(p, src);
      else sort_count_kernel<SortWords, PER><<<tiles, kSortThreads, 0, s>>>(p, SortWords{in});
      if (p.ntiles > kFewTiles) {
        constexpr int kGroups = kSortBins / kScanBins;
        if (p.ntiles <= kScanTiles) {
          sort_scan_kernel<kScanAll><<<kGroups, kSortThreads, 0, s>>>(p);
        } else {
          sort_scan_kernel<kScanAdd><<<dim3(kGroups, kScanShares), kSortThreads, 0, s>>>(p);
          sort_scan_kernel<kScanShare><<<dim3(kGroups, kScanShares), kSortThreads, 0, s>>>(p);
        }
      }
      if (i == 0) sort_scatter_kernel<Source, PER><<<tiles, kSortThreads, 0, s>>>(p, src, out);
      else sort_scatter_kernel<SortWords, PER><<<tiles, kSortThreads, 0, s>>>(p, SortWords{in}, out);
      p.shift += p.bits;
      in = out;
      out = in == buf0 ? buf1 : buf0;
    }
  };
  const int per = sort_items(n);
  if (per == 2) passes(std::integral_constant<int, 2>());
  else if (per == 4) passes(std::integral_constant<int, 4>());
  else if (per == 6) passes(std::integral_constant<int, 6>());
  else passes(std::integral_constant<int, kSortPer>());
  return in;
}

}  // namespace hgnn

// Device side of the row tasks (see hgnn_row_tasks): how a wave finds its piece of work, reads the column ids of a lane
// group eight at a time and gathers table rows.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace hgnn {

constexpr int kMaxTaskBlocks = 64;
constexpr int kXcds = 8;
constexpr int kZeroTurns = 8;  // turns of G empty rows that a wave stores
constexpr int64_t kMixNnz = int64_t(4) << 20;  // see comes_back()
// Waves in a row on one XCD.  31 M non-zeros, one head of 64, 16 / 128 / 512 / 2048 waves: weighted SpMM 383, 369, 362, 363 us, SDDMM
// 367, 353, 349, 350, row sums through the map 334, 320, 320, 334; 114 M, SpMM through the map 2149, 1790, 1789, 1790.
constexpr int kTaskChunk = 512;

struct TaskView {
  const int4_t* task;
  const int4_t* rtask;       // pieces of rows cut at column ranges: an eighth per XCD, so that its L2 keeps to one range of the table
  int n_rtask, rshare;       // how many; per XCD (a multiple of the lane groups of a wave)
  const TaskTotals* rtotals; // device; without a plan, where rows are cut at column ranges: how many pieces there are
  const int* zrow;
  const hgnn_task_sec* sec;
  const int4_t* split;
  int n_slots;               // pieces of the rows in split (on the host only with a plan)
  const uint16_t* col16;     // column ids as 16-bit offsets from block * width, or nullptr: the graph's own
  int width;
  const TaskTotals* totals;  // device; set where the host does not know the numbers (then one block, n_split is a bound)
  int n_split, nb;
  pos_t nnz;                 // entries of the column array that is walked
  bool longer;               // host: rounds of 64 (long_rounds)
  // Consecutive workgroups go to the eight XCDs in turn.  The waves of lane-group pieces are numbered so that `chunk`
  // consecutive ones run on the same XCD: the rows of a window share lines of the column array and of edge tensors, and each
  // of eight L2s would fetch them (62 M non-zeros, rows of 26 on average, 128 features: 1.82 -> 1.69 ms with chunks of 128).
  int chunk;  // a power of two
  int first_wave[kMaxTaskBlocks + 1];  // for the lane groups of this launch: waves before each block, then all of them
  // Whole-wave pieces and waves of lane-group pieces go through the rows side by side (comes_back() below): of the groups of eight
  // waves (one per XCD) of a block every 2^32 / mix-th takes the former.  mix = 0: one kind after the other.
  uint32_t mix[kMaxTaskBlocks];
};

// Whether the second of two kinds of pieces, one after the other, would sweep lines again that the caches have lost: those of edge
// tensors behind a map, or of the popular rows of a table that a last-level cache of 256 MB no longer holds beside the streams.  us, one
// after the other / side by side:
//   through the map: 5.5 M non-zeros x 1 SpMM 106.5 / 102.5, x 4 128.6 / 123.1, row sums 67.6 / 64.8; 20 M x 8 SpMM 632 / 566
//   512 MB, 13 M: SpMM 738 / 692; 154 MB, 31 M: weighted SpMM 406 / 396, SDDMM 415 / 393, attention forward 403 / 377; 128 MB, 20 M x 8:
//     weighted SpMM 294 / 281
//   77 MB, 12 M: weighted SpMM 127 / 130, SDDMM 125 / 125; 33 MB, 5.5 M x 4: SpMM 59.3 / 59.0, SDDMM 58.8 / 58.2; 15 MB, 7.3 M x 128: attention
//     forward 128 / 131.5, backward 140 / 143
// Small graphs stay in the caches and end on long pieces that way (2.1 M, SDDMM 41.7 / 45.1), where nearly all pieces are long there is
// nothing to come back to (6 M, 35 a row: SpMM 124.7 / 127.5); plan-free calls, whose numbers are on the device, gain nothing.
inline bool comes_back(bool mapped, int64_t table_bytes, int64_t llc) { return mapped || table_bytes > llc / 8 * 3; }

// ---- rounds: up to R consecutive non-zeros of a lane group, whose table handles and factors are put in LDS together ----
// A lane reads E consecutive column ids as vectors, so a group's round is one or two cache lines of the column array.
// Read 32 bytes at a time, the lines were asked for four times and the gathers waited for each (114 M non-zeros: 832 ->
// 782 us).  The rows of the LDS tables are 4 entries longer than a round: the groups then read different banks.
// MOST: 32, or 64 where lane groups have longer pieces: a wave is without gathers while it waits for ids, half as often then.  us, rounds of
// 32 / 64: 114 M x 64 in blocks, SpMM 818 / 789, with values 957 / 913, through the map 1601 / 1569, SDDMM 905 / 847, attention forward 1106 /
// 1083, backward 1242 / 1211; 62 M x 128 1326 / 1307; plan-free, 31 M x 64 382 / 376, through the map 677 / 656 (rounds of 128: 782, 920, 1586,
// 1180, 1060, 1225; 1318; 370, 674).
template <int L, int MOST>
struct Round {
  static constexpr int LC = L < 8 ? L : 8;          // lanes that read ids (the others of a wider group repeat them)
  static constexpr int R = L < 4 ? 8 * L : (L < 8 ? 32 : MOST);
  static constexpr int E = R / LC;
  static constexpr int PITCH = R + 4;               // ints per group in the handle table
};
// host: whether a call takes rounds of 64 whose non-zeros take entry_bytes of LDS each; S: most non-zeros of a piece.  Not where pieces of lane groups
// have about 32 non-zeros at most (5.5 M non-zeros x 4 heads: SpMM 57 / 62 us, SDDMM 59 / 71; 1.3 M x 42 27.1 / 27.9; the middle rows of task_build.h
// and pieces at column ranges, which may be longer, run in two rounds), nor where a wave would take more than 6.5 KB, which keeps waves out, nor where
// most rows take whole waves, no more than a round of 32 for each lane group (uniform, 12 M x 64, rounds of 64 / 32: 300 a row, SpMM 84.9 / 81.4, four
// heads of values 103.0 / 98.5, attention forward 125.5 / 122.9; 500 a row 67.9 / 66.7, 84.3 / 78.9, 98.4 / 96.6; without a plan, 150 a row, through the
// map 4 % more with 64, but 300, whose pieces are longer there, 14 % less).
inline bool long_rounds(int nb, int64_t nrows, int64_t nnz, int S, int G, int entry_bytes) {
  if (G > kWave / 8 || G * 64 * entry_bytes > 6656) return false;
  if (nb > 1) return true;
  const int64_t most = task_group_max(nnz);
  return most > 32 && (nnz <= most * nrows || std::min(nnz, S * nrows) > 32 * G * nrows);
}

// pieces at column ranges per XCD, whole waves of G lane groups of them
__host__ __device__ inline int range_share(int n, int G) { return int((pos_t(n) + kXcds * G - 1) / (kXcds * G)) * G; }

// Whether a call takes the pieces at column ranges that the plan has: from so many halves of an L2 on in the table it gathers from, which may
// be narrower than what the plan was made for.  us, ordinary pieces / at column ranges, power law if not said:
//   table, non-zeros          SpMM        edge values   behind a map   SDDMM        attention fwd   saving       bwd
//   1 MB, 8 M                 41 / 58       45 / 73       95 / 151      43 / 77       52 / 63       68 / 70      74 / 102
//   4.2 MB, 5.5 M             47 / 58       53 / 67      110 / 124      50 / 71       57 / 64       72 / 70      91 / 102
//   8.4 MB, 4.5 M             36 / 41       38 / 40       71 / 61       34 / 38       48 / 45       59 / 55      67 / 66
//   8.4 MB, 5.5 M             48 / 55       52 / 56      108 / 94       51 / 53       61 / 56       73 / 66      95 / 91
//   9.6 MB, 12 M             102 / 105     115 / 129     290 / 285     116 / 128     112 / 110     132 / 128    240 / 210
//   16.8 MB, 4.5 M            39 / 42       40 / 41       75 / 64       37 / 37       55 / 51       74 / 68      77 / 74
//   16.8 MB, 5.5 M            48 / 49       51 / 48      107 / 85       48 / 45       62 / 56       77 / 70      99 / 90
//   19 MB, 12 M              104 / 98      112 / 111     285 / 244     109 / 107     112 / 104     130 / 120    246 / 204
//   34 MB, 8 M                61 / 58       63 / 61      150 / 116      62 / 59       84 / 77      114 / 103    135 / 122
//   8.4 MB, 20 M log-normal  225 / 201     251 / 231     539 / 541     238 / 217     229 / 207     243 / 224    414 / 413
// Row sums through a map, which gather edge values: 5.5 M 49 / 42, of four heads 81 / 60, 36 M 384 / 269, 20 M log-normal 286 / 286.
enum RangesFrom { kRangesSpmm = 8, kRangesMapped = 3, kRangesDot = 6, kRangesAttention = 3, kRangesSums = 0 };
inline bool at_ranges(const hgnn_row_tasks* t, RangesFrom from, int64_t table_bytes, int64_t l2) {
  return t->n_rtask > 0 && 2 * table_bytes > from * l2;
}

// host: the launch shape of tasks t for G lane groups per wave, the long rows in ordinary pieces or at column ranges; zeros = false
// leaves the empty rows out
inline TaskView task_view(const hgnn_row_tasks* t, int G, bool ranges, bool comes_back, bool zeros = true) {
  TaskView v{};
  const int sec = ranges ? t->nb : 0;
  v.task = reinterpret_cast<const int4_t*>(t->task);
  v.zrow = t->zrow;
  v.sec = t->sec + sec;
  v.split = reinterpret_cast<const int4_t*>(t->split) + (ranges ? t->n_split : 0);
  v.col16 = t->col16;
  v.width = t->width;
  v.n_split = t->n_split;
  v.nb = t->nb;
  v.nnz = pos_t(t->nnz);
  v.n_slots = ranges ? t->n_rtask : t->n_slots;
  v.rtask = reinterpret_cast<const int4_t*>(t->rtask);
  v.n_rtask = ranges ? t->n_rtask : 0;
  v.rshare = range_share(v.n_rtask, G);
  int64_t n = int64_t(kXcds) * v.rshare / G;
  for (int b = 0; b < t->nb; ++b) {
    const hgnn_task_sec& s = t->host[size_t(sec + b)];
    n = (n + 7) & ~int64_t(7);
    v.first_wave[b] = int(n);
    const int64_t w8 = ceil_div(s.nw, 8), g8 = ceil_div(ceil_div(s.ng, G), 8);
    v.mix[b] = comes_back && t->nnz > kMixNnz && w8 > 0 && w8 <= 4 * g8 ? uint32_t(((w8 << 32) + w8 + g8 - 1) / (w8 + g8)) : 0;
    n += ((s.nw + 7) & ~7) + ((ceil_div(s.ng, G) + 7) & ~int64_t(7)) + (zeros ? ceil_div(s.nz, int64_t(G) * kZeroTurns) : 0);
  }
  v.first_wave[t->nb] = int(n);
  v.chunk = kTaskChunk;
  while (v.chunk > 1 && int64_t(v.chunk) * 64 * t->nb > n) v.chunk >>= 1;  // eight chunks per XCD and block at least
  return v;
}

// f(the most non-zeros of a round) for a launch; the long form exists for tables below 4 GB
template <int L, bool NEAR, class F>
inline void with_round(const TaskView& v, F&& f) {
  if constexpr (L >= 8 && NEAR) {
    if (v.longer) {
      f(std::integral_constant<int, 64>());
      return;
    }
  }
  f(std::integral_constant<int, 32>());
}

// The entries of a run that exist, m = 0, 1, ...: by what is left (which may be negative), or by position.
struct RunLeft {
  int left;
  __device__ __forceinline__ bool has(int m) const { return m < left; }
  template <int E>
  __device__ __forceinline__ bool all() const { return left >= E; }
};
struct RunEnd {
  pos_t i0, end;
  __device__ __forceinline__ bool has(int m) const { return i0 + pos_t(m) < end; }
  template <int E>
  __device__ __forceinline__ bool all() const { return i0 + pos_t(E) <= end; }
};

// v[m] = p[i0 + m] for the entries that exist; the others are 0
template <int E, bool NT, class Run>
__device__ __forceinline__ void load_run(const int* __restrict__ p, pos_t i0, Run run, int (&v)[E]) {
  const int* q = p + i0;
  if (run.template all<E>()) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = NT ? __builtin_nontemporal_load(q + m) : q[m];
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) {
      v[m] = 0;
      if (run.has(m)) v[m] = q[m];
    }
  }
}

// the same for tasks whose numbers are on the device; *grid = workgroups to launch
inline TaskView task_view(const TaskScratch& t, const TaskSource& q, int64_t nnz, int G, int64_t* grid) {
  TaskView v{};
  v.task = reinterpret_cast<const int4_t*>(t.task);
  v.zrow = t.zrow;
  v.sec = t.sec;
  v.split = reinterpret_cast<const int4_t*>(t.split);
  v.totals = t.totals;
  v.n_split = int(t.rows);
  v.nb = 1;
  v.nnz = pos_t(nnz);
  v.rtask = reinterpret_cast<const int4_t*>(t.rtask);
  if (t.rtask) v.rtotals = t.totals;
  const int64_t n = int64_t(kXcds) * range_share(int(t.cap), G) / G + nnz / (q.group_max + 1) + ceil_div(q.nrows + nnz / q.S + 1, G) + ceil_div(q.nrows, int64_t(G) * kZeroTurns) + 24;
  v.chunk = kTaskChunk;
  while (v.chunk > 1 && int64_t(v.chunk) * 64 > n) v.chunk >>= 1;
  constexpr int64_t kMostWaves = 65536;  // beyond this the waves take several tasks each
  *grid = n < kMostWaves ? (n + 7) / 8 * 8 : kMostWaves;
  return v;
}

// Rows of several pieces per wave in the follow-up kernels: one for each of the G lane groups (longer rows one after the other by the whole
// wave), or one in all, whose lane groups then take a piece each and add across the wave.  The launch is a few latencies long and a wave of
// G rows is a chain of them; us, G rows / one: 4000 rows x 64, saving attention 13.7 / 9.4, its backward 9.0 / 6.4; 800 rows x 42, SpMM
// 5.3 / 4.7 (a GCN layer of 1.3 M non-zeros 89.3 / 84.8).  Many rows of two or three pieces (long rows of
// column blocks: some 50 000 of 114 M non-zeros x 64) are work for all lane groups: SpMM 7.5 / 20, saving attention 16 / 41.  Between them it
// turns on the rows of more than eight pieces, which a wave of G rows takes one after the other.  Whole calls, us, one / G rows (weighted SpMM;
// saving attention), rows of so many pieces on average:
//   F = 64   4175 of 2.6, log-normal   31.6 / 32.4;  59.5 / 60.7      F = 16    8881 of 6.2, power law   49.8 / 56.0;  95.6 / 105.1
//            6221 of 2.7, log-normal   33.0 / 33.4;  63.7 / 64.4               17041 of 7.2, power law   43.4 / 47.7;  57.3 / 63.1
//            8881 of 6.2, power law    54.6 / 55.1; 112.2 / 114.5     F = 128   8881 of 6.2, power law   81.5 / 82.3; 166.0 / 166.1
//            9728 of 3.1, log-normal   36.4 / 36.1;  72.1 / 71.8               16143 of 4.1, log-normal  77.5 / 76.1; 130.6 / 128.0
//           17041 of 7.2, power law    58.1 / 57.0; 101.2 / 98.8               20927 of 6.4, log-normal  80.4 / 78.9; 107.6 / 105.1
//           22472 of 8.0, log-normal  446.1 / 442.3; 468.6 / 462.6             35608 of 9.5, power law  1312.6 / 1314.7; 1615 / 1624
//           21061 of 10, power law    288.0 / 288.2; 380.6 / 379.4
constexpr int kFinishAlone = 65536;
__host__ __device__ inline int finish_rows_per_wave(int n_split, int n_slots, int G) {
  const int many = G >= 32 ? 6 : 9;  // pieces a row
  return n_split <= 8192 || (n_split <= kFinishAlone && n_slots / many >= n_split) ? 1 : G;
}

// A row of more than this many pieces for each lane group of a wave is added by all waves of a workgroup of the follow-up kernels: the longest row
// of a power law was most of a launch (62 M non-zeros x 128, 770 pieces: SpMM 43.8 -> 25 us; whole calls, 20 M x 128 326 -> 319.5, attention
// forward 514 -> 505, backward 643 -> 633, 31 M x 64 296 -> 292.5, 456 -> 447, 678 -> 674; smaller ones the same).  Never, 128, 64, 32, 16, 8 pieces: 2 M of
// 20 000 vertices x 128, attention forward 64.1, 63.7, 63.4, 60.1, 60.0, 59.4, backward 49.5, 48.8, 48.9, 46.4, 46.9, 46.4; 31 M x 64 409.7, 407.0, 408.4, 404.3, 403.0, 403.6.
constexpr int kManyPieces = 32;

// Whether a row may have so many, by the pieces that there are in all (a row of the list has one at least).  Else the follow-up kernels do without the list of
// such rows and its barriers: 12 150 non-zeros, power law, SpMM 6.9 / 6.6 us.
inline bool many_pieces(const TaskView& v, int G) { return v.n_slots - (v.n_split - 1) > kManyPieces * G; }

// waves of work behind a view (G lane groups per wave)
template <int G>
__device__ __forceinline__ int task_waves(const TaskView& v) {
  if (!v.totals) return v.first_wave[v.nb];
  const hgnn_task_sec s = v.sec[0];
  return int(((pos_t(s.nw) + 7) & ~7u) + (((pos_t(s.ng) + G - 1) / G + 7) & ~7u) + (pos_t(s.nz) + G * kZeroTurns - 1) / (G * kZeroTurns));
}

// what one wave does
struct TaskWave {
  int block, first; // column block and its first non-zero
  bool whole;       // all lane groups share one piece
  const int* zrow;  // the block's empty rows
  pos_t z0, z1;     // z1 > z0: entries [z0, z1) of them, nothing else
  pos_t beg, end;   // this lane group's first non-zero and the end of the piece
  pos_t span, step; // non-zeros per round of this group (a multiple of 8, at most its R), and from one round to the next
  int row, slot;    // row -1: no piece for this lane group
};

// wid is the same on all lanes of the wave; g = lane / L.  Everything up to the task is scalar; a choice between two addresses to
// load from would turn all of it into vector code (5.5 M non-zeros, SDDMM 58 -> 62 us, attention forward 82 -> 87).
// ranges: the pieces of rows cut at column ranges, if any.  FREE: the view is one without a plan (1: without column ranges either).
struct RangeWaves {
  int waves, share, n;  // waves that take them, pieces per XCD, pieces
};
template <int G>
__device__ __forceinline__ RangeWaves range_waves(const TaskView& v) {  // without a plan
  const int n = v.rtotals ? v.rtotals->n_range : 0, share = range_share(n, G);
  return RangeWaves{share / G * kXcds, share, n};
}
template <int L, int R, int FREE>  // R: of the Round
__device__ __forceinline__ TaskWave task_enter(const TaskView& v, int wid, int g, const RangeWaves& ranges) {
  constexpr int G = kWave / L;
  TaskWave w;
  if (FREE != 1 && wid < ranges.waves) {
    const int i = (wid >> 3) * G + g, k = (wid & 7) * ranges.share + i;
    int4_t t = {0, 0, -1, -1};
    if (k < ranges.n) t = v.rtask[k];
    w.block = w.first = 0;
    w.whole = false;
    w.zrow = v.zrow;
    w.z0 = w.z1 = 0;
    w.beg = t[0];
    w.end = t[0] + t[1];
    w.row = t[2];
    w.slot = t[3];
    w.span = w.step = R;
    return w;
  }
  int b = 0, i = wid;
  if (FREE) {
    if (FREE == 2) i -= ranges.waves;
  } else {
    while (b + 1 < v.nb && wid >= v.first_wave[b + 1]) ++b;
    i -= v.first_wave[b];
  }
  const hgnn_task_sec s = v.sec[b];
  w.block = b;
  w.first = s.first;
  w.whole = false;
  w.zrow = v.zrow + s.z_off;
  w.z0 = w.z1 = 0;
  int4_t t = {0, 0, -1, -1};
  // sections begin at multiples of eight: i & 7 is the XCD
  const int nw = (s.nw + 7) & ~7, gw = int(((pos_t(s.ng) + G - 1) / G + 7) & ~7u);
  const uint32_t mix = FREE ? 0 : v.mix[b];
  bool wh = i < nw;                        // a whole-wave piece
  pos_t before = pos_t(wh ? i : nw) >> 3;  // groups of eight waves before this one that take those
  if (mix && i < nw + gw) {
    const pos_t u = pos_t(i) >> 3;
    before = pos_t((uint64_t(u) * mix) >> 32);
    wh = pos_t((uint64_t(u + 1) * mix) >> 32) > before;
  }
  if (wh) {
    const int k = int(before * 8) + (i & 7);
    w.whole = k < s.nw;
    if (w.whole) t = v.task[s.w_off + k];
  } else {
    i -= int(before * 8);
    if (i < gw) {
      const int panel = 8 * v.chunk, full = gw & -panel;
      if (i < full) {
        const int p = i & -panel, j = i - p;
        i = p + (j & 7) * v.chunk + (j >> 3);
      }
      const pos_t k = pos_t(i) * G + g;
      if (k < pos_t(s.ng)) t = v.task[pos_t(s.g_off) + k];
    } else {
      w.z0 = pos_t(i - gw) * (G * kZeroTurns);
      w.z1 = w.z0 + G * kZeroTurns < pos_t(s.nz) ? w.z0 + G * kZeroTurns : pos_t(s.nz);
    }
  }
  w.beg = t[0];
  w.end = t[0] + (t[1] & 0xffff);
  w.row = t[2];
  w.slot = t[3];
  w.span = w.step = R;
  if (w.whole) {  // the lane groups share the piece in equal runs
    const pos_t each = (((t[1] & 0xffff) + G - 1) / G + 7) & ~7;
    if (each < w.span) w.span = each;
    w.beg += w.span * g;
    w.step = w.span * G;
  }
  return w;
}

template <int L, int R>
__device__ __forceinline__ TaskWave task_enter(const TaskView& v, int wid, int g) {
  return task_enter<L, R, 0>(v, wid, g, RangeWaves{v.first_wave[0], v.rshare, v.n_rtask});
}

// The column ids of a round.  Blocks of the plan's own cut carry them in 16 bits: the ids are the one stream that these
// passes draw from HBM, and a gather waits behind it (114 M non-zeros x 64 in eight blocks: 0.81 -> 0.76 ms).
// A lane's run begins `own` entries behind the round of its lane group.  The ids of entries that do not exist are not defined: 16-bit ids are
// read as a vector also where a piece ends among them (what follows belongs to other pieces), and where a lane has none at all from the
// beginning of the round, a line that is asked for anyway.  Read by entry at the ends of pieces they were a chain of four waits, and nearly every
// wave has a lane there (114 M x 64: SpMM 827 -> 818 us, SDDMM 914 -> 903, attention backward 1254 -> 1241).
template <int E, class Run>
__device__ __forceinline__ void load_cols(const TaskView& v, const int* __restrict__ col, bool nt, int block, pos_t round, int own, Run run, int (&c)[E]) {
  if (v.col16) {
    const pos_t at = run.has(0) ? round + pos_t(own) : round;
    uint32_t t[E / 2];
    if (at + pos_t(E) <= v.nnz) {
      __builtin_memcpy(t, v.col16 + at, sizeof(t));
    } else {
      const pos_t last = v.nnz - 1;
#pragma unroll
      for (int m = 0; m < E; m += 2) {
        const pos_t i = at + pos_t(m);
        t[m / 2] = uint32_t(v.col16[i < last ? i : last]) | uint32_t(v.col16[i + 1 < last ? i + 1 : last]) << 16;
      }
    }
    const int first = block * v.width;
#pragma unroll
    for (int m = 0; m < E; ++m) c[m] = first + int(m & 1 ? t[m / 2] >> 16 : t[m / 2] & 0xffffu);
    return;
  }
  if (nt) load_run<E, true>(col, round + pos_t(own), run, c);
  else load_run<E, false>(col, round + pos_t(own), run, c);
}

// A table of rows of ld halves.  NEAR: its bytes stay below 2^32 - 8192, rows are read through a buffer descriptor whose
// bounds make the positions past the end of a piece read as zeros (offset kNoRow), so the loop needs no masks; else by
// 64-bit addresses and a branch.
constexpr uint32_t kNoRow = 0xFFFFF000u;
inline bool near_table(int64_t rows, int64_t ld) { return uint64_t(rows) * uint64_t(ld) * 2u < (uint64_t(1) << 32) - 8192u; }

template <bool NEAR>
struct RowTable {
  __amdgpu_buffer_rsrc_t rsrc;
  const half_t* base;
  int64_t ld;
  uint32_t pitch;  // bytes
  uint32_t lane_bytes;
  __device__ __forceinline__ RowTable(const half_t* x, int64_t rows, int64_t ld_, int f0) {
    base = x + f0;
    ld = ld_;
    pitch = uint32_t(ld_) * 2u;
    lane_bytes = uint32_t(f0) * 2u;
    if (NEAR) rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(x), 0, int(uint32_t(rows) * pitch), 0x00020000);
  }
  // what to hand to row() for column c, or for no column at all
  __device__ __forceinline__ int handle(int c, bool valid) const {
    if (NEAR) return valid ? int(uint32_t(c) * pitch) : int(kNoRow);
    return valid ? c : -1;
  }
  template <int VW = 8>  // halves per lane
  __device__ __forceinline__ auto row(int h) const {
    typedef _Float16 hv_t __attribute__((ext_vector_type(VW)));
    if (NEAR) {
      typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
      typedef unsigned uint4_t __attribute__((ext_vector_type(4)));
      const int at = int(uint32_t(h) + lane_bytes);
      if constexpr (VW == 8) return __builtin_bit_cast(hv_t, uint4_t(__builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, 0)));
      else if constexpr (VW == 4) return __builtin_bit_cast(hv_t, uint2_t(__builtin_amdgcn_raw_buffer_load_b64(rsrc, at, 0, 0)));
      else return __builtin_bit_cast(hv_t, unsigned(__builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0)));
    }
    hv_t r = hv_t(0);
    if (h >= 0) r = *reinterpret_cast<const hv_t*>(base + int64_t(h) * ld);
    return r;
  }
};

// v summed over the wave's lane groups of L lanes; the lanes of group 0 hold the result.  Vector instructions only: quad
// permutes, rotations inside 16 lanes and the exchanges between the four rows of 16.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float xor16_mov(float v, bool max_of) {
#pragma clang fp contract(off)
  typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
  const uint2_t r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float x = __uint_as_float(r[0]), y = __uint_as_float(r[1]);
  return max_of ? fmaxf(x, y) : x + y;
}
__device__ __forceinline__ float xor32_mov(float v, bool max_of) {
#pragma clang fp contract(off)
  typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
  const uint2_t r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float x = __uint_as_float(r[0]), y = __uint_as_float(r[1]);
  return max_of ? fmaxf(x, y) : x + y;
}
template <int L>
__device__ __forceinline__ float across_groups_sum(float v) {
#pragma clang fp contract(off)
  if (L <= 1) v += dpp_mov<0xB1>(v);
  if (L <= 2) v += dpp_mov<0x4E>(v);
  if (L <= 4) v += dpp_mov<0x124>(v);
  if (L <= 8) v += dpp_mov<0x128>(v);
  if (L <= 16) v = xor16_mov(v, false);
  if (L <= 32) v = xor32_mov(v, false);
  return v;
}
template <int L>
__device__ __forceinline__ float across_groups_max(float v) {
  if (L <= 1) v = fmaxf(v, dpp_mov<0xB1>(v));
  if (L <= 2) v = fmaxf(v, dpp_mov<0x4E>(v));
  if (L <= 4) v = fmaxf(v, dpp_mov<0x124>(v));
  if (L <= 8) v = fmaxf(v, dpp_mov<0x128>(v));
  if (L <= 16) v = xor16_mov(v, true);
  if (L <= 32) v = xor32_mov(v, true);
  return v;
}

// ---- scores of a tile -------------------------------------------------------------------------------------------------
// Every lane of a head holds its eight features' share of the scores of eight edges.  The shares are summed by halves: with
// each exchange a lane keeps half of the edges, so a head of RS or more lanes ends with 8 / RS finished scores per
// lane, and maximum, exponential and LeakyReLU are evaluated once per (edge, head), not once per lane.
// Edges a lane ends up with: j * RS + own_edge(l), j = 0 .. 8 / RS - 1.
template <int RS>
struct HeadTile {
  static constexpr int NS = 8 / RS;
  static __device__ __forceinline__ int own_edge(int l) {
    if (RS < 8) return l & (RS - 1);
    const int b2 = (l >> 2) & 1;  // the last exchange mirrors eight lanes: the upper four keep mirrored edges
    return b2 ? 4 | ((l & 3) ^ 3) : (l & 3);
  }
  static constexpr int lane_of(int e) { return RS < 8 ? e : (e & 4 ? 4 | ((e & 3) ^ 3) : e); }
  template <int CTRL>
  static __device__ __forceinline__ float halve(float a, float b, bool upper) {  // lower lanes keep a, upper ones b
#pragma clang fp contract(off)
    const float keep = upper ? b : a, send = upper ? a : b;
    return keep + dpp_mov<CTRL>(send);
  }
  static __device__ __forceinline__ void scores(const float (&d)[8], int l, float (&s)[NS]) {
    const bool flip = RS == 8 && (l & 4);
    const bool u0 = ((l & 1) != 0) != flip, u1 = ((l & 2) != 0) != flip, u2 = (l & 4) != 0;
    if constexpr (RS == 1) {
#pragma unroll
      for (int j = 0; j < 8; ++j) s[j] = d[j];
    } else {
      float r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = halve<0xB1>(d[2 * j], d[2 * j + 1], u0);
      if constexpr (RS == 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = r[j];
      } else {
        float t[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) t[j] = halve<0x4E>(r[2 * j], r[2 * j + 1], u1);
        if constexpr (RS == 4) {
          s[0] = t[0];
          s[1] = t[1];
        } else {
          s[0] = halve<0x141>(t[0], t[1], u2);
        }
      }
    }
  }
  // the value of edge U of the tile, from the lane of this head that holds it
  template <int U>
  static __device__ __forceinline__ float from_owner(const float (&v)[NS]) {
    if constexpr (RS == 1) return v[U];
    else return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v[U / RS]), (0x1f & ~(RS - 1)) | (lane_of(U % RS) << 5)));
  }
  static __device__ __forceinline__ float sum(float v) { return head_sum1(v, RS); }  // over the RS lanes
  static __device__ __forceinline__ float max_of(float v) {
    if (RS >= 2) v = fmaxf(v, dpp_mov<0xB1>(v));
    if (RS >= 4) v = fmaxf(v, dpp_mov<0x4E>(v));
    if (RS >= 8) v = fmaxf(v, dpp_mov<0x141>(v));
    return v;
  }
};

}  // namespace hgnn

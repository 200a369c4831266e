// Internal definitions shared by the translation units of libhgnn.so (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "hgnn.h"

namespace hgnn {

constexpr int kWave = 64;          // CDNA wavefront
constexpr int kWavesPerBlock = 4;  // 256-thread workgroups: one wave per SIMD of a CU
constexpr int kBlock = kWave * kWavesPerBlock;

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));  // 16 bytes: one global_load_dwordx4 per lane

// ---- status plumbing -------------------------------------------------------------------------
hgnn_status fail(hgnn_status s, const char* fmt, ...);  // records the thread-local message, returns s
void clear_error();

#define HGNN_REQUIRE(cond, status, ...)                  \
  do {                                                   \
    if (!(cond)) return ::hgnn::fail(status, __VA_ARGS__); \
  } while (0)

#define HGNN_HIP(call)                                                                              \
  do {                                                                                              \
    hipError_t err__ = (call);                                                                      \
    if (err__ != hipSuccess)                                                                        \
      return ::hgnn::fail(err__ == hipErrorOutOfMemory ? HGNN_ENOMEM : HGNN_EHIP, "%s: %s", #call, \
                          hipGetErrorString(err__));                                                \
  } while (0)

#define HGNN_LAUNCH_CHECK(name)                                                     \
  do {                                                                              \
    hipError_t err__ = hipGetLastError();                                           \
    if (err__ != hipSuccess)                                                        \
      return ::hgnn::fail(HGNN_EHIP, "launch of %s: %s", name, hipGetErrorString(err__)); \
  } while (0)

// Waves per workgroup for the kernel over neighbour groups, whose waves work independently on private LDS regions of per_wave
// bytes (no workgroup barrier anywhere, so the choice is free).  Where waves stage edge values before their main loop (a
// dependent chain of global loads whose length varies from wave to wave) single-wave workgroups are 5-15 % faster: a
// workgroup's LDS and wave slots are only released when its last wave ends.  Without edge values workgroups of four were 4 %
// faster (fewer dispatches, waves of consecutive groups start together).  Either way the workgroup must fit 64 KB.
inline int waves_per_block_for_lds(size_t per_wave, bool independent_waves) {
  int w = independent_waves ? 1 : 4;
  while (w > 1 && per_wave * size_t(w) > 65536) w >>= 1;
  return w;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// smallest power of two >= v (v >= 1)
inline int pow2_at_least(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

hgnn_status check_csr_args(const hgnn_csr* g, const char* who);

// ---- memory of the set-up calls (memory.hip): device blocks that are kept for the next call when freed ----------
// A block may be freed only when no work that uses it is in flight.
hipError_t dev_malloc_bytes(void** out, size_t bytes);
void dev_free(const void* p);
void dev_release(const void* p);  // where that could not be made sure: back to the runtime, never to another call
inline void dev_put(const void* p, bool idle) { idle ? dev_free(p) : dev_release(p); }
bool device_idle(int dev);  // waits for everything on that device, whatever device is current; false: it could not
template <class T>
inline hipError_t dev_malloc(T** out, size_t bytes) {
  void* p = nullptr;
  const hipError_t e = dev_malloc_bytes(&p, bytes);
  *out = static_cast<T*>(p);
  return e;
}

// The stream of a set-up call.  Whatever is launched or copied goes through the conversion, so it knows whether anything may
// be in flight; DevTemp and HostMail wait for that before they give their memory back, on every way out of the call.
class SetupStream {
 public:
  explicit SetupStream(void* stream) : s(static_cast<hipStream_t>(stream)) {}
  SetupStream(const SetupStream&) = delete;
  SetupStream& operator=(const SetupStream&) = delete;
  operator hipStream_t() {
    idle = false;
    return s;
  }
  hipError_t wait() {
    const hipError_t e = hipStreamSynchronize(s);
    idle = e == hipSuccess;
    return e;
  }
  bool settle() { return idle || wait() == hipSuccess; }  // true: nothing of this call is in flight

 private:
  hipStream_t s;
  bool idle = true;
};

// a device block of a set-up call that is freed when it goes out of scope
struct DevTemp {
  SetupStream& s;
  void* p = nullptr;
  explicit DevTemp(SetupStream& stream) : s(stream) {}
  DevTemp(const DevTemp&) = delete;
  DevTemp& operator=(const DevTemp&) = delete;
  ~DevTemp() {
    if (p) dev_put(p, s.settle());
  }
  hipError_t alloc(size_t bytes) { return dev_malloc_bytes(&p, bytes); }
  template <class T>
  T* as() const { return static_cast<T*>(p); }
};

// a small piece of pinned host memory that kernels can write and the host reads after a synchronization (a copy out of
// pageable memory costs a staging round of its own); data == nullptr when there is none left
constexpr size_t kMailBytes = 256;
struct HostMail {
  SetupStream& s;
  char* data = nullptr;
  int slot = -1;
  explicit HostMail(SetupStream& stream);
  ~HostMail();
  HostMail(const HostMail&) = delete;
  HostMail& operator=(const HostMail&) = delete;
};

// row that holds CSR position k: the last r with rowptr[r] <= k (an upper bound minus one, so
// empty rows are skipped)
__host__ __device__ inline int row_of_edge(const int* rowptr, int nrows, int64_t k) {
  uint32_t lo = 0, hi = uint32_t(nrows) + 1u;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (int64_t(rowptr[mid]) <= k) lo = mid + 1;
    else hi = mid;
  }
  return int(lo) - 1;
}

// Positions of non-zeros and numbers of pieces go up to 2^31 - 1.  A walk forms sums up to a step (at most a few thousand)
// beyond its end before it compares them, so it counts in pos_t: 32 bits hold them without a sign.
typedef uint32_t pos_t;
__host__ __device__ inline int pieces_of(int len, int per) { return int((pos_t(len) + pos_t(per) - 1u) / pos_t(per)); }

// Orders the LDS accesses of one wave: what its lanes wrote before is visible to all its lanes after.
// Waves that have an LDS region of their own meet nobody else; a workgroup barrier there would only put the waves of a workgroup
// in lock step and stall the others whenever one waits for memory.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v += the value of the lane that the data-parallel-primitive control CTRL pairs this lane with (one VALU
// instruction, no trip through the LDS crossbar).  Controls used: quad_perm [1,0,3,2] = 0xB1 and [2,3,0,1] =
// 0x4E (lane ^ 1, lane ^ 2), row_half_mirror = 0x141 (lane i <-> 7 - i of each 8), row_mirror = 0x140
// (i <-> 15 - i of each 16).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  const int t = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false);
  return v + __int_as_float(t);
}

// sum over the wave on all lanes, vector instructions only
__device__ __forceinline__ int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);
  typedef unsigned uint2_t __attribute__((ext_vector_type(2)));
  uint2_t r = __builtin_amdgcn_permlane16_swap(unsigned(v), unsigned(v), false, false);
  v = int(r[0] + r[1]);
  r = __builtin_amdgcn_permlane32_swap(unsigned(v), unsigned(v), false, false);
  return int(r[0] + r[1]);
}

// The head of lane l of a row, LH lanes to a head, LH a power of two.  (A division is some 25 vector instructions, and a wave of the kernels over row
// tasks has a few hundred in all.)
__device__ __forceinline__ int head_of_lane(int l, int LH) { return l >> (31 - __builtin_clz(unsigned(LH))); }

// All-reduce (sum) over the LH consecutive, LH-aligned lanes of a head; LH is a power of two.  After the
// quads are summed, a mirror inside 8 (16) lanes pairs every lane with one of the other quad (half), whose
// partial sum is the same on all its lanes; beyond a row of 16 lanes the exchange goes through ds_bpermute.
__device__ __forceinline__ float head_sum1(float v, int LH) {
  if (LH >= 2) v = dpp_add<0xB1>(v);
  if (LH >= 4) v = dpp_add<0x4E>(v);
  if (LH >= 8) v = dpp_add<0x141>(v);
  if (LH >= 16) v = dpp_add<0x140>(v);
  for (int off = 16; off < LH; off <<= 1) v += __shfl_xor(v, off);
  return v;
}

typedef int int4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));

// ---- per-edge row ids of one plan segment, staged in LDS by one wave (edge_score_seg_kernel) ----------
// A segment of n <= S consecutive edges starting at e0 touches the rows row_lo..row_hi (plan arrays).
// Every non-empty row after row_lo marks the slot of its first edge, then a wave-wide running
// maximum spreads the ids: s_row[i] = row of edge e0+i for i < n.  Lane t owns the slots [t*per, (t+1)*per); per is a
// multiple of 4.  s_row is private to the calling wave.  `between` runs when the first offsets are on their way: loads
// issued there are in flight while the rows are staged.
__device__ __forceinline__ int seg_slots_per_lane(int S) { return 4 * ((S + 255) / 256); }

// The index arrays (column ids, edge ids) are read once per pass.  Where they are far larger than the caches, passes through an
// edge-id map, which gather from two tables, read them with non-temporal loads so that they displace fewer of the lines that
// the gathers want again.  SpMM through the map, without / with the hint: 31 M non-zeros x 1 head 821 / 808 us, x 4 heads 857 /
// 847, 60 M x 16 features 1681 / 1667, 62 M x 128 2681 / 2655; over column blocks, where a wave returns to the lines of the map that
// its neighbours have read, it costs: 114 M 1620 / 1668.  Passes without a map gain nothing (SpMM 0 to 0.9 %, SDDMM 0, attention
// forward 1 to 2.6 % slower), and where the arrays fit the last-level cache the hint would push them out between kernels.
__host__ __device__ inline bool stream_nontemporal(int64_t nnz) { return nnz * 4 > (int64_t(64) << 20); }

__device__ __forceinline__ float dot8(const half8_t& a, const half8_t& b) {
  float p = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) p = fmaf(float(a[i]), float(b[i]), p);
  return p;
}

__device__ __forceinline__ int wave_max_scan(int v) {  // inclusive
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
  v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));  // row_bcast:15, row_bcast:31
  return max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
}

template <class F>
__device__ __forceinline__ void seg_stage_rows(int* s_row, int lane, int per, int row_lo, int row_hi, const int* __restrict__ rowptr,
                                               int64_t e0, F&& between) {
  int r = row_lo + 1 + lane, p = 0, q = 0;
  if (r <= row_hi) p = rowptr[r], q = rowptr[r + 1];
  between();
  for (int i = 4 * lane; i < kWave * per; i += 4 * kWave) *reinterpret_cast<int4_t*>(s_row + i) = int4_t{-1, -1, -1, -1};
  wave_sync();
  if (q > p) s_row[p - int(e0)] = r;
  for (r += kWave; r <= row_hi; r += kWave) {
    p = rowptr[r], q = rowptr[r + 1];
    if (q > p) s_row[p - int(e0)] = r;
  }
  wave_sync();
  int4_t* const own = reinterpret_cast<int4_t*>(s_row + lane * per);
  int run = row_lo;  // the first edges' row; ids grow
  for (int j = 0; j < per / 4; ++j) {
    const int4_t v = own[j];
    run = max(max(max(run, v[0]), max(v[1], v[2])), v[3]);
  }
  run = __builtin_amdgcn_update_dpp(row_lo, wave_max_scan(run), 0x138, 0xf, 0xf, false);  // of the lanes before: wave_shr:1
  for (int j = 0; j < per / 4; ++j) {
    int4_t v = own[j];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = run = max(run, v[i]);
    own[j] = v;
  }
  wave_sync();
}

}  // namespace hgnn

// ---- row tasks of a plan (tasks.hip): the rows of a graph, or of its column blocks, as pieces of work for a wave ----
// A piece of a row is at most S consecutive non-zeros (S = the plan's segment size); a row within S is one piece.  Pieces
// longer than a threshold take a whole wave each, shorter ones a lane group, sorted by length inside windows of rows so
// that the groups of a wave end together; empty rows are listed on their own.
// One piece: x = first non-zero (in the task's column array), y = length | block << 16, z = row, w = staging slot of a row
// that has several pieces, or -1.
struct hgnn_task_sec {  // the pieces of one column block (or of the whole graph)
  int32_t w_off, nw;  // task[w_off ..): whole-wave pieces
  int32_t g_off, ng;  // task[g_off ..): lane-group pieces
  int64_t z_off;      // zrow[z_off ..): empty rows (of all blocks: up to blocks * rows)
  int32_t nz;
  int32_t first;      // the block's first non-zero in the task's column array
};
struct hgnn_row_tasks {
  int32_t nb = 0;
  int64_t nnz = 0;
  int4* task = nullptr;
  // The rows of several pieces once more, cut at column ranges (ranges.h): pieces range after range, all staged.  A call takes them in the
  // place of the ordinary pieces of those rows where its own table is large enough (at_ranges in task.h); n_rtask = 0: there are none.
  int4* rtask = nullptr;
  int32_t n_rtask = 0;
  int32_t* zrow = nullptr;
  int4* split = nullptr;         // [n_split] rows with several pieces: (row, first slot, pieces, block); with column ranges as many again for those
  hgnn_task_sec* sec = nullptr;  // [nb]; with column ranges a second one, without the rows that are cut there
  int32_t n_split = 0, n_slots = 0;
  int32_t stage_slots = 0;       // of the staging arrays: n_slots, or n_rtask where that is more
  const uint16_t* col16 = nullptr;  // column blocks of at most 65536 columns: the column ids less the block's first (the plan's)
  int32_t width = 0;                // columns per block
  std::vector<hgnn_task_sec> host;  // sec on the host
  hgnn_half* staging = nullptr;  // [2][stage_slots][max_F] partial vectors (second set: masked vectors of the saving GAT pass)
  float* stage_mz = nullptr;     // [3][stage_slots][max_H] scalars of the partial vectors of the fused GAT passes
};

// The plan object behind the opaque handle of the C ABI.
constexpr int kHubEdges = 2048;  // non-zeros per chunk of a long row in the edge-row kernels

struct hgnn_plan {
  int device = 0;       // the device that was current when the plan was made: its arrays are there
  int32_t nrows = 0, ncols = 0;
  int64_t nnz = 0;
  int32_t S = 0;        // edges per segment
  int64_t nseg = 0;     // ceil(nnz / S)
  int32_t n_split = 0;  // rows whose edges span more than one segment
  int32_t n_big = 0;    // rows longer than big_deg (edge softmax hands them to a whole workgroup)
  int32_t n_mid = 0;    // rows longer than mid_deg and at most big_deg (edge softmax: one wave each)
  int32_t mid_deg = 0;
  int32_t big_deg = 0;
  int64_t listed_nnz = 0;  // non-zeros of the rows in mid_row and big_row (the rest belong to rows of at most mid_deg)
  int32_t max_F = 0, max_H = 0;
  int64_t l2_bytes = 0, llc_bytes = 0;  // cache sizes of the device the plan was built on (an XCD's L2, the cache behind the L2s)
  int32_t vec_halves = 8;  // halves a lane moves per feature load in the kernels that exist in several widths (8, 4 or 2)
  bool auto_blocks = false;  // the blocks were chosen by the automatic rule (col_blocks = 0): a call whose own table is small runs unblocked
  bool block_eid = false;  // column blocks: built from a graph that carried an edge-id map (which beid then holds)
  int32_t* seg_row_lo = nullptr;    // [nseg]
  int32_t* seg_row_hi = nullptr;    // [nseg]
  int32_t* split_row = nullptr;     // [n_split]
  int32_t* split_seg_lo = nullptr;  // [n_split]
  int32_t* split_seg_hi = nullptr;  // [n_split]
  int32_t* big_row = nullptr;       // [n_big]
  int32_t* mid_row = nullptr;       // [n_mid]
  // the rows of big_row cut into chunks of kHubEdges non-zeros for the edge-row kernels (softmax, its backward, row
  // sums): a workgroup per chunk leaves partial results, a second pass combines those of a row
  int32_t n_hub_chunks = 0;
  int32_t* hub_chunk_row = nullptr;    // [n_hub_chunks] the row a chunk belongs to
  int32_t* hub_chunk_first = nullptr;  // [n_hub_chunks] slot of the first chunk of that row (slot - first = chunk number)
  int32_t* hub_chunk_count = nullptr;  // [n_hub_chunks] chunks of that row
  int32_t* big_first = nullptr;        // [n_big] slot of the first chunk of big_row[i]
  float* hub_part = nullptr;           // [n_hub_chunks][max_H][2] partial results
  float* vscratch = nullptr;        // [(nrows + ncols) * max_H] fp32
  float* vtab = nullptr;            // [nrows][max_H][4] fp32 per-vertex (el, lse, t, -) of the fused GAT backward
  // column blocking of the SpMM (nb > 1): block b holds the non-zeros whose column lies in
  // [b*block_width, (b+1)*block_width), stored block after block as a CSR of their own.  Where every pass takes the blocks of
  // `fine`, this plan holds none of the arrays.
  int32_t nb = 1;
  int32_t block_width = 0;
  int32_t* brp = nullptr;           // [nb][nrows+1] offset arrays of the blocks
  int32_t* bcol = nullptr;          // [nnz] column ids, block-major; or, where 16 bits do,
  uint16_t* bcol16 = nullptr;       // [nnz] the same less b*block_width
  int32_t* beid = nullptr;          // [nnz] the creating graph's edge-id map, block-major (block_eid)
  int32_t* bdelta = nullptr;        // [nb][nrows] CSR position in the whole graph of a blocked non-zero = its position in the block + bdelta[b][row]
  std::vector<int64_t> boff;        // [nb+1] first non-zero of every block in bcol / beid
  hgnn_row_tasks* tasks = nullptr;   // of the whole graph
  hgnn_row_tasks* btasks = nullptr;  // of the column blocks (nb > 1; null where every pass takes those of `fine`)
  hgnn_plan* fine = nullptr;        // the same graph in twice the blocks (blocked arrays only); only where the automatic rule
                                    // chose the blocks
  hgnn_half* bstage = nullptr;      // [2][nb][nrows][max_F] per-block partial outputs (second set: masked GAT partials)
  float* bsum = nullptr;            // [nb][nrows][max_H][2] per-block partial row sums of edge tensors / GAT (max, sum), then [nb][nrows][max_H] masked sums
  // neighbour groups of the vertex-parallel variant (hgnn_plan_add_groups): row r owns the groups
  // goff[r] .. goff[r+1]-1, group j of the row covers the non-zeros rowptr[r] + j*ng ...
  int32_t ng = 0;                   // neighbours per group; 0 = not built
  int64_t n_groups = 0;
  int64_t n_gslots = 0;             // groups that belong to rows with more than one group
  int32_t* goff = nullptr;          // [nrows+1]
  int32_t* moff = nullptr;          // [nrows+1] first staging slot of a row with more than one group
  int32_t* grp_row = nullptr;       // [n_groups]
  hgnn_half* gstage = nullptr;      // [n_gslots][max_F]
  // column slices (hgnn_plan_add_slices): slice s holds the columns [s*slice_w, (s+1)*slice_w); the edge-score and
  // column-sum kernels keep one slice's per-column scalars in LDS
  int32_t ns = 0;                   // slices; 0 = not built
  int32_t slice_w = 0;
  int32_t nch = 0;                  // chunks of about as many non-zeros and rows each (a multiple of 8)
  bool slice_scores = false;        // scores go over the slices too (slices.hip)
  int32_t* scut = nullptr;          // [ns+1][nrows] first CSR position of row r whose column is >= s*slice_w
  int2* slice_share = nullptr;      // row and position where the share of a chunk that a wave takes begins
  unsigned long long* col_part = nullptr;  // [nch][ncols] fixed-point partial column sums of the chunks
  float* col_poison = nullptr;      // [ncols] sums of non-finite inputs; zero between calls
};

namespace hgnn {
// el[i,h] = a_l[h].U[i,h] and er[j,h] = a_r[h].Vt[j,h] into the plan's fp32 scratch (el first, then er;
// Vt == nullptr skips er)
hgnn_status gat_check(const hgnn_plan* p, int H, int D, const hgnn_half* U, int64_t ldu, const hgnn_half* Vt, int64_t ldv,
                      const hgnn_half* a_l, const hgnn_half* a_r, const char* who);  // what the projection needs of its arguments
hgnn_status gat_project(const hgnn_plan* p, const hgnn_csr* g, int H, int D, const hgnn_half* U, int64_t ldu,
                        const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l, const hgnn_half* a_r, hipStream_t s,
                        const char* who);
// argument checks shared by the SpMM entry points, and the plan-free SpMM with the scratch of its hub kernels at
// `scratch` (scratch_bytes of device memory; null: no row is treated as a hub)
hgnn_status check_spmm_args(const char* who, const hgnn_csr* g, const hgnn_half* w, int H, const hgnn_half* X, int64_t ldx,
                            hgnn_half* Y, int64_t ldy, int F, hgnn_reduce op);
hgnn_status spmm_rows(const char* who, const hgnn_csr* g, const hgnn_half* edge_val, int32_t H, const hgnn_half* X,
                      int64_t ldx, hgnn_half* Y, int64_t ldy, int32_t F, hgnn_reduce op, const float* row_scale,
                      void* scratch, size_t scratch_bytes, bool one_sweep, hipStream_t s);
void device_cache_bytes(int64_t* l2, int64_t* llc);  // of the current device
size_t spmm_hub_scratch_bytes(int32_t nrows, int64_t nnz, int32_t F);  // scratch of the plan-free SpMM's hub kernels alone
hgnn_status plan_build_arrays(hgnn_plan* p, const hgnn_csr* g, bool blocks, SetupStream& s);  // blocks: build_col_blocks follows
hgnn_status build_col_blocks(hgnn_plan* p, const hgnn_csr* g, int nb, SetupStream& s);  // p->nb > 1 from here
// the cut whose blocks a pass walks; narrow: a pass that gathers from two tables at once or leaves no partial rows behind
inline const hgnn_plan* walked_cut(const hgnn_plan* p, bool narrow) { return p->fine && (narrow || !p->btasks) ? p->fine : p; }
constexpr int kSliceMaxCols = 16384;  // columns per slice: 8 bytes each fill 128 KB of the 160 KB of LDS a workgroup may hold
// row tasks in two steps around a host wait: task_count launches the counting passes, task_build takes their result
struct TaskSource {
  const int32_t* rowptr;  // [nb][nrows+1], every block's offsets from 0
  const int32_t* first;   // device, [nb] first non-zero of every block, or nullptr (one block)
  int32_t nrows, nb, S, group_max;
  int64_t nnz;
  int32_t range_min;      // rows of at least so many non-zeros are cut by ranges.h, too (one block), or kNoRanges
};
constexpr int kNoRanges = 0x7fffffff;
// Longest piece that is left to one lane group (but for the middle rows of task_build.h).  Small graphs have few waves and want short chains of loads, large ones few
// reductions across lane groups (2.1 M non-zeros x 128: 32 is 3 % better than 64; 62 M x 128: 128 is 1 % better); the pieces of
// column blocks come in numbers and are bound by the L2s (114 M non-zeros: 256 is 3 % better than 128).
constexpr int kGroupMaxBlocks = 256;
inline int task_group_max(int64_t nnz) { return nnz <= (int64_t(8) << 20) ? 32 : 128; }
struct TaskTotals {
  int64_t n_zero;
  int32_t n_task, n_whole, n_split, n_slots;
  int32_t n_long_whole, n_long_group, n_range;  // of n_task: pieces of the rows from range_min on; their pieces by ranges.h
};
constexpr int kTaskWindow = 1024;  // rows that are sorted together: enough for equal neighbours; few, because the short rows of a
                                   // window share cache lines of the column array and of edge tensors (see TaskView::chunk)
// The same without a plan, in memory of the caller and without a host wait: the launch shape is then not known on the host, so
// the kernels read it from `sec` and `totals` and walk the tasks with a grid stride.
struct TaskScratch {
  int32_t* counts;
  int32_t* sums;
  hgnn_task_sec* sec;
  TaskTotals* totals;
  int4* task;
  int32_t* zrow;
  int4* split;
  float* staging;  // [slots][F rounded up to a multiple of 8] fp32
  int4* rtask;     // [cap] pieces of the rows from range_min on at column ranges, or nullptr; the lists that lead there behind it
  int32_t* range_lists;
  int32_t* cuts;
  int64_t cap;     // most pieces at column ranges: where a graph would have more, its long rows stay in ordinary pieces
  int64_t rows;    // most rows of several pieces
  size_t bytes;
};
// base may be null: sizes only; range_min = kNoRanges: without column ranges
TaskScratch task_scratch_at(void* base, int64_t nrows, int64_t nnz, int S, int F, int range_min);
hgnn_status task_build_in(const TaskSource& q, const TaskScratch& t, const int32_t* col, int ncols, hipStream_t s);
struct TaskCounts {
  explicit TaskCounts(SetupStream& s) : counts(s), secs(s), mail(s) {}
  DevTemp counts, secs;
  HostMail mail;
  int nwin = 0;
  int* count = nullptr;          // device, [kTaskAll][nb][nwin]
  int* sums = nullptr;           // device, [kTaskAll][nb]
  hgnn_task_sec* sec = nullptr;  // device, [nb]
  TaskTotals* totals = nullptr;  // valid after the stream has been waited for (host memory, or a device copy)
  int* n_range = nullptr;        // beside it, where rows are cut at column ranges (ranges = true): what becomes got.n_range
  bool ranges = false;
  TaskTotals got{};              // the same on the host, from task_allocate on
  const int* split_at = nullptr;  // device, [nwin] rows of several pieces before each window of kTaskWindow rows
};
hgnn_status task_prepare(const TaskSource& q, TaskCounts& c);
hgnn_status task_allocate(const TaskSource& q, TaskCounts& c, int max_F, int max_H, hgnn_row_tasks** out);
hgnn_status build_block_tasks(hgnn_plan* p, SetupStream& s);
void destroy_tasks(hgnn_row_tasks* t, bool idle);  // idle: nothing that uses them is in flight
hgnn_status build_col_slices(hgnn_plan* p, const hgnn_csr* g, int W, bool asked, SetupStream& s);  // asked: by the caller, for all that they serve
hgnn_status slice_edge_score(const hgnn_plan* p, const hgnn_csr* g, const float* el, const float* er, const float* lse,
                             float slope, hgnn_half* out, hipStream_t s);
}  // namespace hgnn

// Edge softmax (paper Eq. 1), its backward, and row sums of edge tensors, for gfx950.
//
// The scores of one row (neighbourhood) are the contiguous slice e[rowptr[i]*H, rowptr[i+1]*H),
// element j of the whole tensor belonging to head j % H.  A "team" of lanes owns a row: a
// sub-wave group of LR lanes (LR chosen from the mean row length, so short rows do not idle a
// whole wave) or a whole wave; rows longer than the plan's threshold are cut into chunks, a
// workgroup each, whose partial results a second launch combines.
// Every lane moves 16 bytes (8 halves) per access: the slice is walked in the 8-element vectors,
// aligned to the tensor's base, that lie in it whole, and the few non-zeros at its two ends by themselves; because H
// divides 8 the head of each of a lane's 8 elements is fixed.  A row that fits the lanes'
// registers is read once.  exp, sums and the division stay in fp32; the exponent is <= 0, so
// the numerator is in (0,1] (section 3.1.2) and alpha is rounded once.
#include "task.h"

#include <climits>

namespace hgnn {

constexpr int kKeepVec = 2;     // 8-element vectors per lane held in registers

struct EdgeRowArgs {
  const int* rowptr;
  const int* big_row;
  const int* row_list;  // the tier of longer rows goes through this list, or through all rows
  int n_list;
  const int* eid;
  const half_t* x0;  // forward: e.          backward: alpha.   rowsum: t
  const half_t* x1;  //                      backward: dalpha
  const half_t* x2;  //                      backward: e (LeakyReLU mask) or nullptr
  half_t* out;       // forward: alpha.      backward: de.      rowsum: [nrows][H]
  int nrows, H;
  int team_max;      // rows longer than this are left by the sub-wave teams to a wave each
  int list_max;      // of the longer rows those above this take a wave each, the others a team of 16 lanes (0: all a wave each)
  int wave_max;      // rows longer than this go to the chunked kernels (INT_MAX: there are none)
  float slope;
};

// ---- teams -----------------------------------------------------------------------------------------
// One step of an all-reduce (sum or maximum) among aligned groups of lanes: with the partner inside a row of 16
// lanes the exchange is a DPP operand of the VALU instruction (lane ^ 1, lane ^ 2, then mirrors inside 8 and 16
// lanes, which pair a lane with one from the other half, whose partial result is the same on all its lanes);
// across rows it is one of the row swaps.
template <int OFF, bool IS_MAX>
__device__ __forceinline__ float team_step(float v) {
  float o;
  if (OFF == 1) o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));
  else if (OFF == 2) o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, false));
  else if (OFF == 4) o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, false));
  else if (OFF == 8) o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, false));
  else return OFF == 16 ? xor16_mov(v, IS_MAX) : xor32_mov(v, IS_MAX);
  return IS_MAX ? fmaxf(v, o) : v + o;
}

template <int N, int H, bool IS_MAX>  // all-reduce over aligned groups of N lanes (N a power of two up to 64)
__device__ __forceinline__ void team_reduce(float (&v)[H]) {
#pragma unroll
  for (int h = 0; h < H; ++h) {
    if (N > 1) v[h] = team_step<1, IS_MAX>(v[h]);
    if (N > 2) v[h] = team_step<2, IS_MAX>(v[h]);
    if (N > 4) v[h] = team_step<4, IS_MAX>(v[h]);
    if (N > 8) v[h] = team_step<8, IS_MAX>(v[h]);
    if (N > 16) v[h] = team_step<16, IS_MAX>(v[h]);
    if (N > 32) v[h] = team_step<32, IS_MAX>(v[h]);
  }
}

template <int LR>
struct SubWaveTeam {  // LR consecutive lanes of a wave
  static constexpr int size = LR;
  int rank;
  __device__ SubWaveTeam() : rank((threadIdx.x & (kWave - 1)) % LR) {}
  template <int H, bool IS_MAX>
  __device__ __forceinline__ void reduce(float (&v)[H]) const {
    team_reduce<LR, H, IS_MAX>(v);
  }
};

// The non-zeros [beg, end) of a row (or of a chunk of one) as the vectors of 8 elements that lie in it whole, and what is left at its two
// ends, fewer non-zeros than a vector holds on either side.  Whole vectors need no masks; the ends are dealt out to the lanes, H elements of a
// non-zero each.  With masks on every vector and the vectors at the ends stored by element a wave with a row of 100 non-zeros x 4 heads spent
// 530 vector instructions, and these bound the pass; with the ends apart and such rows sharing waves, us, forward; backward; row sums: 5.5 M
// power law x 4 heads 58 -> 40; 45 -> 44; 23 -> 19, one head 25 -> 17; 24 -> 20; 12.6 -> 9.5; 20 M x 4 196 -> 135; 194 -> 193; 66 -> 49; 40 M
// log-normal, one head 87 -> 53; 113 -> 91; 56 -> 36; 3 M uniform, one head 8.3 -> 6.5; 8.5 -> 8.0; 3.8 -> 3.8; without a plan 18.7 -> 10.1;
// 20.6 -> 12.0.
template <int H>
struct Span {
  static constexpr int kPer = 8 / H;           // non-zeros in a vector
  static constexpr int kEnds = 2 * (kPer - 1);  // at most so many non-zeros outside whole vectors
  pos_t beg, body, tail;   // non-zeros: the first, the first of the whole vectors, the first behind them
  int n_head, n_body, n_tail;  // n_body counts vectors
  __device__ __forceinline__ Span(int first, int last) {
    const pos_t b = pos_t(first), e = pos_t(last), up = (b + kPer - 1) & ~pos_t(kPer - 1), down = e & ~pos_t(kPer - 1);
    beg = b;
    body = up < e ? up : e;
    n_head = int(body - b);
    n_body = down > up ? int((down - up) / kPer) : 0;
    tail = down >= up ? down : e;
    n_tail = int(e - tail);
  }
  __device__ __forceinline__ bool has(int i) const { return i < kPer - 1 ? i < n_head : i - (kPer - 1) < n_tail; }
  __device__ __forceinline__ pos_t end_at(int i) const { return i < kPer - 1 ? beg + pos_t(i) : tail + pos_t(i - (kPer - 1)); }
};

// The part of a span that a lane of a team of SIZE holds: KEEP vectors in registers (lane `rank` has every SIZE-th one), and its share
// of the ends.
template <int H, int SIZE, int KEEP>
struct Held {
  typedef _Float16 hv_t __attribute__((ext_vector_type(H)));
  static constexpr int NE = (Span<H>::kEnds + SIZE - 1) / SIZE;
  half8_t v[KEEP];
  hv_t e[NE > 0 ? NE : 1];
  __device__ __forceinline__ void load(const half_t* p, const Span<H>& s, int rank, half_t fill) {
    const half8_t* const q = reinterpret_cast<const half8_t*>(p + int64_t(s.body) * H);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
      v[i] = half8_t(fill);
      const int t = rank + SIZE * i;
      if (t < s.n_body) v[i] = q[t];
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      e[i] = hv_t(fill);
      const int t = rank + SIZE * i;
      if (t < Span<H>::kEnds && s.has(t)) e[i] = *reinterpret_cast<const hv_t*>(p + int64_t(s.end_at(t)) * H);
    }
  }
  // the same of the three tensors of the backward, together; e may be null (then it is 1)
  static __device__ __forceinline__ void load_bwd(const half_t* alpha, const half_t* dalpha, const half_t* e, const Span<H>& s, int rank, Held& al,
                                                  Held& da, Held& el) {
    const int64_t first = int64_t(s.body) * H;
    const half8_t *const q0 = reinterpret_cast<const half8_t*>(alpha + first), *const q1 = reinterpret_cast<const half8_t*>(dalpha + first),
                  *const q2 = reinterpret_cast<const half8_t*>(e + first);
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
      al.v[i] = da.v[i] = half8_t(0);
      el.v[i] = half8_t(1);
      const int t = rank + SIZE * i;
      if (t < s.n_body) {
        al.v[i] = q0[t];
        da.v[i] = q1[t];
        if (e) el.v[i] = q2[t];
      }
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      al.e[i] = da.e[i] = hv_t(half_t(0));
      el.e[i] = hv_t(half_t(1));
      const int t = rank + SIZE * i;
      if (t < Span<H>::kEnds && s.has(t)) {
        const int64_t at = int64_t(s.end_at(t)) * H;
        al.e[i] = *reinterpret_cast<const hv_t*>(alpha + at);
        da.e[i] = *reinterpret_cast<const hv_t*>(dalpha + at);
        if (e) el.e[i] = *reinterpret_cast<const hv_t*>(e + at);
      }
    }
  }
};

// ---- forward: one row by one team ----------------------------------------------------------------------
template <int H, int KEEP, class Team>
__device__ __forceinline__ void softmax_fwd_row(const EdgeRowArgs& a, const Team& team, int beg, int end) {
  constexpr int SIZE = Team::size;
  typedef Held<H, SIZE, KEEP> Hold;
  typedef typename Hold::hv_t hv_t;
  const Span<H> s(beg, end);
  // what a lane does not have is -inf: it loses every maximum and adds exp(-inf) = 0
  Hold x;
  x.load(a.x0, s, team.rank, half_t(-INFINITY));
  const half8_t* const src = reinterpret_cast<const half8_t*>(a.x0 + int64_t(s.body) * H);
  half8_t* const dst = reinterpret_cast<half8_t*>(a.out + int64_t(s.body) * H);
  float m[H];
#pragma unroll
  for (int h = 0; h < H; ++h) m[h] = -INFINITY;
  auto visit_max = [&](const half8_t& v) {
#pragma unroll
    for (int q = 0; q < 8; ++q) m[q % H] = fmaxf(m[q % H], float(v[q]));
  };
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (i == 0 || SIZE * i < s.n_body) visit_max(x.v[i]);
#pragma unroll
  for (int i = 0; i < Hold::NE; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) m[h] = fmaxf(m[h], float(x.e[i][h]));
  for (int t = team.rank + SIZE * KEEP; t < s.n_body; t += SIZE) visit_max(src[t]);
  team.template reduce<H, true>(m);
  float z[H], ex[KEEP][8], ee[Hold::NE > 0 ? Hold::NE : 1][H];  // the exponentials of what is held, formed once
#pragma unroll
  for (int h = 0; h < H; ++h) z[h] = 0.f;
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    if (i == 0 || SIZE * i < s.n_body) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        ex[i][q] = __expf(float(x.v[i][q]) - m[q % H]);
        z[q % H] += ex[i][q];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < Hold::NE; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) {
      ee[i][h] = __expf(float(x.e[i][h]) - m[h]);
      z[h] += ee[i][h];
    }
  for (int t = team.rank + SIZE * KEEP; t < s.n_body; t += SIZE) {
    const half8_t v = src[t];
#pragma unroll
    for (int q = 0; q < 8; ++q) z[q % H] += __expf(float(v[q]) - m[q % H]);
  }
  team.template reduce<H, false>(z);
  float inv[H];
#pragma unroll
  for (int h = 0; h < H; ++h) inv[h] = 1.f / z[h];
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    const int t = team.rank + SIZE * i;
    if (t < s.n_body) {
      half8_t o;
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = half_t(ex[i][q] * inv[q % H]);
      dst[t] = o;
    }
  }
#pragma unroll
  for (int i = 0; i < Hold::NE; ++i) {
    const int t = team.rank + SIZE * i;
    if (t < Span<H>::kEnds && s.has(t)) {
      hv_t o;
#pragma unroll
      for (int h = 0; h < H; ++h) o[h] = half_t(ee[i][h] * inv[h]);
      *reinterpret_cast<hv_t*>(a.out + int64_t(s.end_at(t)) * H) = o;
    }
  }
  for (int t = team.rank + SIZE * KEEP; t < s.n_body; t += SIZE) {
    const half8_t v = src[t];
    half8_t o;
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = half_t(__expf(float(v[q]) - m[q % H]) * inv[q % H]);
    dst[t] = o;
  }
}

// ---- backward: t = sum alpha*dalpha (per head); de = alpha*(dalpha - t) [* LeakyReLU'(e)] --------------
__device__ __forceinline__ half_t softmax_bwd_value(const EdgeRowArgs& a, half_t alpha, half_t dalpha, half_t e, float t) {
  float d = float(alpha) * (float(dalpha) - t);
  if (!(float(e) > 0.f)) d *= a.slope;
  return half_t(d);
}

template <int H, int KEEP, class Team>
__device__ __forceinline__ void softmax_bwd_row(const EdgeRowArgs& a, const Team& team, int beg, int end) {
  constexpr int SIZE = Team::size;
  typedef Held<H, SIZE, KEEP> Hold;
  typedef typename Hold::hv_t hv_t;
  const Span<H> s(beg, end);
  // what a lane does not have is zero on both sides, so its products vanish (a neighbouring row's infinity times zero would not)
  // All that is held is asked for together, e (1 if there is none) with the others.  Behind the sums a wave waited for it twice more, the ends'
  // behind the stores of the vectors, and three conditions on every vector and end cost as much as masks where rows are short.  us, masked
  // vectors / ends apart, each array by itself, e behind the sums / now: 8 M uniform of 2 M rows, one head 42 / 45 / 41, two 44 / 57 / 37; 20 M of
  // 300 000, four heads 146 / 166 / 140; of 150 000, two 73 / 74 / 61; 20 M power law, two 108 / 103 / 86.  (20 M of 150 000 to 200 000 rows, eight
  // heads: 219 / 230 / 230.)
  Hold al, da, el;
  const int64_t first = int64_t(s.body) * H;
  auto vec = [&](const half_t* p, int t) { return reinterpret_cast<const half8_t*>(p + first)[t]; };
  Hold::load_bwd(a.x0, a.x1, a.x2, s, team.rank, al, da, el);
  half8_t* const dst = reinterpret_cast<half8_t*>(a.out + first);
  float t[H];
#pragma unroll
  for (int h = 0; h < H; ++h) t[h] = 0.f;
  auto visit = [&](const half8_t& va, const half8_t& vd) {
#pragma unroll
    for (int q = 0; q < 8; ++q) t[q % H] = fmaf(float(va[q]), float(vd[q]), t[q % H]);
  };
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if (i == 0 || SIZE * i < s.n_body) visit(al.v[i], da.v[i]);
#pragma unroll
  for (int i = 0; i < Hold::NE; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) t[h] = fmaf(float(al.e[i][h]), float(da.e[i][h]), t[h]);
  for (int v = team.rank + SIZE * KEEP; v < s.n_body; v += SIZE) visit(vec(a.x0, v), vec(a.x1, v));
  team.template reduce<H, false>(t);
  auto emit = [&](const half8_t& va, const half8_t& vd, const half8_t& ve, int v) {
    half8_t o;
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = softmax_bwd_value(a, va[q], vd[q], ve[q], t[q % H]);
    dst[v] = o;
  };
#pragma unroll
  for (int i = 0; i < KEEP; ++i) {
    const int v = team.rank + SIZE * i;
    if (v < s.n_body) emit(al.v[i], da.v[i], el.v[i], v);
  }
#pragma unroll
  for (int i = 0; i < Hold::NE; ++i) {
    const int v = team.rank + SIZE * i;
    if (v < Span<H>::kEnds && s.has(v)) {
      const int64_t at = int64_t(s.end_at(v)) * H;
      hv_t o;
#pragma unroll
      for (int h = 0; h < H; ++h) o[h] = softmax_bwd_value(a, al.e[i][h], da.e[i][h], el.e[i][h], t[h]);
      *reinterpret_cast<hv_t*>(a.out + at) = o;
    }
  }
  for (int v = team.rank + SIZE * KEEP; v < s.n_body; v += SIZE)
    emit(vec(a.x0, v), vec(a.x1, v), a.x2 ? vec(a.x2, v) : half8_t(1), v);
}

// ---- row sums: out[row,h] = sum over the row of t[slot(k), h] -------------------------------------------
// s += what the lane `rank` of `size` holds of the non-zeros [beg, end)
template <int H, int SIZE>
__device__ __forceinline__ void rowsum_share(const EdgeRowArgs& a, int rank, int beg, int end, float (&s)[H]) {
  typedef _Float16 hv_t __attribute__((ext_vector_type(H)));
  if (a.eid) {  // transposed view: one lane per non-zero, its H values are contiguous at slot eid[k]
    for (pos_t k = pos_t(beg) + rank; k < pos_t(end); k += SIZE) {
      const hv_t v = *reinterpret_cast<const hv_t*>(a.x0 + int64_t(a.eid[k]) * H);
#pragma unroll
      for (int h = 0; h < H; ++h) s[h] += float(v[h]);
    }
    return;
  }
  const Span<H> sp(beg, end);
  Held<H, SIZE, 1> x;
  x.load(a.x0, sp, rank, half_t(0));
  const half8_t* const src = reinterpret_cast<const half8_t*>(a.x0 + int64_t(sp.body) * H);
  auto add = [&](const half8_t& v) {
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q % H] += float(v[q]);
  };
  add(x.v[0]);
#pragma unroll
  for (int i = 0; i < x.NE; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) s[h] += float(x.e[i][h]);
  for (int t = rank + SIZE; t < sp.n_body; t += SIZE) add(src[t]);
}

template <int H, class Team>
__device__ __forceinline__ void rowsum_row(const EdgeRowArgs& a, const Team& team, int row, int beg, int end) {
  float s[H];
#pragma unroll
  for (int h = 0; h < H; ++h) s[h] = 0.f;
  rowsum_share<H, Team::size>(a, team.rank, beg, end, s);
  team.template reduce<H, false>(s);
  if (team.rank == 0) {
#pragma unroll
    for (int h = 0; h < H; ++h) a.out[int64_t(row) * H + h] = half_t(s[h]);
  }
}

enum { kFwd = 0, kBwd = 1, kSum = 2 };
// vectors a lane holds of a listed row or of a chunk: registers for eight waves a SIMD (seven with four heads), four with eight heads
__host__ __device__ constexpr int edge_keep(int op, int H) { return op == kFwd && H < 8 ? 4 : 2; }

// one row by the team of LR lanes that the calling lane belongs to, KEEP vectors a lane in registers
template <int OP, int LR, int H, int KEEP = kKeepVec>
__device__ __forceinline__ void edge_row(const EdgeRowArgs& a, int row, int beg, int end) {
  const SubWaveTeam<LR> team;
  if (OP == kSum) {
    rowsum_row<H>(a, team, row, beg, end);
  } else if (end > beg) {
    if (OP == kFwd) softmax_fwd_row<H, KEEP>(a, team, beg, end);
    else softmax_bwd_row<H, KEEP>(a, team, beg, end);
  }
}

// ---- long rows in chunks ------------------------------------------------------------------------------
// A row above the plan's long-row threshold is cut into chunks of kHubEdges non-zeros (the plan lists them): a
// workgroup of kHubThreads per chunk leaves the chunk's partial result per head -- (max, sum of exp) for the
// softmax, sum of alpha * dalpha for its backward, the sum for the row sums -- and a second launch combines the
// partials of a row (a few dozen at most) and writes the chunk's outputs, or the row's sum.  The latency of a long
// row is then that of one chunk, and a graph's longest rows keep many compute units busy instead of one each.
constexpr int kHubThreads = 256;

struct HubChunks {
  const int* row;    // [n] row of the chunk
  const int* first;  // [n] slot of the first chunk of that row
  const int* count;  // [n] chunks of that row
  float* part;       // [n][H][2]
};

template <int H, bool IS_MAX>
__device__ __forceinline__ void hub_block_reduce(float (&v)[H], float* sm) {  // sm: [kHubThreads / kWave][8]
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  team_reduce<kWave, H, IS_MAX>(v);
  __syncthreads();  // protects sm against the previous use
  if (lane == 0)
#pragma unroll
    for (int h = 0; h < H; ++h) sm[wave * 8 + h] = v[h];
  __syncthreads();
#pragma unroll
  for (int h = 0; h < H; ++h) {
    float r = sm[h];
    for (int w = 1; w < kHubThreads / kWave; ++w) r = IS_MAX ? fmaxf(r, sm[w * 8 + h]) : r + sm[w * 8 + h];
    v[h] = r;
  }
}

// the chunk's non-zeros [beg, end) of its row
__device__ __forceinline__ void hub_chunk_range(const EdgeRowArgs& a, const HubChunks& c, int slot, int& beg, int& end) {
  const int row = c.row[slot];
  beg = a.rowptr[row] + (slot - c.first[slot]) * kHubEdges;
  const int row_end = a.rowptr[row + 1];
  end = row_end - beg > kHubEdges ? beg + kHubEdges : row_end;
}

template <int OP, int H>
__device__ __forceinline__ void edge_hub_partial(const EdgeRowArgs& a, const HubChunks& c, int slot) {
  __shared__ float sm[(kHubThreads / kWave) * 8];
  int beg, end;
  hub_chunk_range(a, c, slot, beg, end);
  float r0[H], r1[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    r0[h] = OP == kFwd ? -INFINITY : 0.f;
    r1[h] = 0.f;
  }
  const int rank = threadIdx.x;
  if (OP == kSum) {
    rowsum_share<H, kHubThreads>(a, rank, beg, end, r0);
    hub_block_reduce<H, false>(r0, sm);
  } else {
    // a chunk is kHubEdges * H / 8 vectors and its ends at most
    constexpr int ALL = kHubEdges * H / 8 / kHubThreads, KEEP = ALL < edge_keep(OP, H) ? ALL : edge_keep(OP, H);
    typedef Held<H, kHubThreads, KEEP> Hold;
    const Span<H> s(beg, end);
    const int64_t first = int64_t(s.body) * H;
    auto vec = [&](const half_t* p, int t) { return reinterpret_cast<const half8_t*>(p + first)[t]; };
    Hold x;
    x.load(a.x0, s, rank, half_t(OP == kFwd ? -INFINITY : 0.f));
    if (OP == kFwd) {
#pragma unroll
      for (int i = 0; i < KEEP; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) r0[q % H] = fmaxf(r0[q % H], float(x.v[i][q]));
#pragma unroll
      for (int i = 0; i < Hold::NE; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h) r0[h] = fmaxf(r0[h], float(x.e[i][h]));
      for (int t = rank + kHubThreads * KEEP; KEEP < ALL && t < s.n_body; t += kHubThreads) {
        const half8_t v = vec(a.x0, t);
#pragma unroll
        for (int q = 0; q < 8; ++q) r0[q % H] = fmaxf(r0[q % H], float(v[q]));
      }
      hub_block_reduce<H, true>(r0, sm);  // then the sum of exp relative to the chunk's maximum
#pragma unroll
      for (int i = 0; i < KEEP; ++i)
        if (rank + kHubThreads * i < s.n_body) {
#pragma unroll
          for (int q = 0; q < 8; ++q) r1[q % H] += __expf(float(x.v[i][q]) - r0[q % H]);
        }
#pragma unroll
      for (int i = 0; i < Hold::NE; ++i)
        if (rank + kHubThreads * i < Span<H>::kEnds && s.has(rank + kHubThreads * i)) {
#pragma unroll
          for (int h = 0; h < H; ++h) r1[h] += __expf(float(x.e[i][h]) - r0[h]);
        }
      for (int t = rank + kHubThreads * KEEP; KEEP < ALL && t < s.n_body; t += kHubThreads) {
        const half8_t v = vec(a.x0, t);
#pragma unroll
        for (int q = 0; q < 8; ++q) r1[q % H] += __expf(float(v[q]) - r0[q % H]);
      }
      hub_block_reduce<H, false>(r1, sm);
    } else {
      Hold d;
      d.load(a.x1, s, rank, half_t(0));
#pragma unroll
      for (int i = 0; i < KEEP; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) r0[q % H] = fmaf(float(x.v[i][q]), float(d.v[i][q]), r0[q % H]);
#pragma unroll
      for (int i = 0; i < Hold::NE; ++i)
#pragma unroll
        for (int h = 0; h < H; ++h) r0[h] = fmaf(float(x.e[i][h]), float(d.e[i][h]), r0[h]);
      for (int t = rank + kHubThreads * KEEP; KEEP < ALL && t < s.n_body; t += kHubThreads) {
        const half8_t v = vec(a.x0, t), w = vec(a.x1, t);
#pragma unroll
        for (int q = 0; q < 8; ++q) r0[q % H] = fmaf(float(v[q]), float(w[q]), r0[q % H]);
      }
      hub_block_reduce<H, false>(r0, sm);
    }
  }
  if (threadIdx.x < H) {
    float v0 = 0.f, v1 = 0.f;
#pragma unroll
    for (int h = 0; h < H; ++h)
      if (int(threadIdx.x) == h) {
        v0 = r0[h];
        v1 = r1[h];
      }
    c.part[(int64_t(slot) * H + threadIdx.x) * 2] = v0;
    c.part[(int64_t(slot) * H + threadIdx.x) * 2 + 1] = v1;
  }
}

// Every row of the graph in one launch: the wave-per-row tier (wave_wgs workgroups), then the sub-wave teams, and the chunks of
// the long rows (n_chunks workgroups) after or before them.  As launches of their own each has a tail in which the chip drains:
// 5.5 M non-zeros x 4 heads, forward with its follow-up 71 -> 57 us, backward 61 -> 45, sums 32 -> 22, when a wave took each of the longer rows.
// The softmax takes the chunks last because its follow-up reads them again while the caches still hold them (then, 114 M non-zeros, one head:
// forward 189 us with the chunks first, 184 last, 179 in launches of their own; backward 210, 201, 207); the sums take them first (23.3 us last).
// Longer rows: a workgroup takes 16 rows, listed or not, a team of 16 lanes each where that is four vectors a lane at most; the longer ones
// among them are dealt out to its waves.  Rows in a row often are of one length (vertices in the order of their degrees), so that a workgroup of
// neighbours would have sixteen of the longest: it takes four in a row from each of four places of a stretch of kDealt workgroups' rows.  5.5 M
// power law in the order of the degrees, us, forward; backward, a wave a row / sixteen neighbours / dealt out: without a plan, one head 83; 83 / 99;
// 113 / 51; 60, eight 623; 812 / 950; 1253 / 482; 660; listed, four heads 47; 39 / 51; 56 / 34; 42.  In no order the offsets are in more lines:
// without a plan one head 91; 85 / 53; 59 / 55; 60, listed, four 58; 46 / 42; 45 / 40; 44, and 8 M uniform without a plan 173; 175 / 79; 88 / 85; 94
// (stretches of 16 and 64 workgroups: order of the degrees, one head 63; 71 and 55; 64).
constexpr int kListTeam = 16, kListRows = kHubThreads / kListTeam, kDealt = 256;
__device__ __forceinline__ int64_t dealt_row(int wg, int wave, int team) {
  constexpr int kTeams = kWave / kListTeam;
  return (int64_t(wg / kDealt) * (kHubThreads / kWave) + wave) * (kDealt * kTeams) + (wg % kDealt) * kTeams + team;
}
template <int OP, int LR, int H>
__global__ __launch_bounds__(kHubThreads) void edge_rows_kernel(EdgeRowArgs a, HubChunks c, int n_chunks, int wave_wgs) {
  constexpr int W = kHubThreads / kWave;
  int wg = int(blockIdx.x);
  const int first_chunk = OP == kSum ? 0 : int(gridDim.x) - n_chunks;
  if (wg >= first_chunk && wg < first_chunk + n_chunks) {
    edge_hub_partial<OP, H>(a, c, wg - first_chunk);
    return;
  }
  if (OP == kSum) wg -= n_chunks;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (wg < wave_wgs && a.list_max > 0) {
    const int64_t i = dealt_row(wg, wave, lane / kListTeam);
    int row = 0, beg = 0, end = 0;
    if (i < a.n_list) {
      row = a.row_list ? a.row_list[i] : int(i);
      beg = a.rowptr[row];
      end = a.rowptr[row + 1];
    }
    const int len = end - beg;
    const bool ok = len > a.team_max && len <= a.wave_max, whole = len > a.list_max;
    __shared__ int s_whole[kListRows], s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    if (ok && whole && lane % kListTeam == 0) s_whole[atomicAdd(&s_n, 1)] = row;
    if (ok && !whole) edge_row<OP, kListTeam, H, edge_keep(OP, H)>(a, row, beg, end);
    __syncthreads();
    for (int k = wave; k < s_n; k += W) {
      const int r = __builtin_amdgcn_readfirstlane(s_whole[k]);
      edge_row<OP, kWave, H>(a, r, a.rowptr[r], a.rowptr[r + 1]);
    }
    return;
  }
  if (wg < wave_wgs) {
    const int64_t i = int64_t(wg) * W + wave;
    if (i >= a.n_list) return;
    const int row = a.row_list[i];
    const int beg = a.rowptr[row], end = a.rowptr[row + 1];
    if (end - beg > a.team_max && end - beg <= a.wave_max) edge_row<OP, kWave, H>(a, row, beg, end);
    return;
  }
  const int64_t row = (int64_t(wg - wave_wgs) * W + wave) * (kWave / LR) + lane / LR;
  if (row >= a.nrows) return;
  const int beg = a.rowptr[row], end = a.rowptr[row + 1];
  if (end - beg <= a.team_max && end - beg <= a.wave_max) edge_row<OP, LR, H>(a, int(row), beg, end);
}

// softmax forward / backward: the row's partials combined, then this chunk's outputs
template <int OP, int H>
__global__ __launch_bounds__(kHubThreads) void edge_hub_emit_kernel(EdgeRowArgs a, HubChunks c) {
  const int slot = blockIdx.x;
  int beg, end;
  hub_chunk_range(a, c, slot, beg, end);
  const int first = c.first[slot], cnt = c.count[slot];
  float M[H], S[H];  // forward: row maximum and 1 / sum of exp; backward: S = sum of alpha * dalpha
#pragma unroll
  for (int h = 0; h < H; ++h) {
    M[h] = -INFINITY;
    S[h] = 0.f;
  }
  if (OP == kFwd) {
    for (int i = 0; i < cnt; ++i)
#pragma unroll
      for (int h = 0; h < H; ++h) M[h] = fmaxf(M[h], c.part[(int64_t(first + i) * H + h) * 2]);
  }
  for (int i = 0; i < cnt; ++i)
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const float p0 = c.part[(int64_t(first + i) * H + h) * 2], p1 = c.part[(int64_t(first + i) * H + h) * 2 + 1];
      S[h] += OP == kFwd ? p1 * __expf(p0 - M[h]) : p0;
    }
  if (OP == kFwd) {
#pragma unroll
    for (int h = 0; h < H; ++h) S[h] = 1.f / S[h];
  }
  typedef _Float16 hv_t __attribute__((ext_vector_type(H)));
  const Span<H> s(beg, end);
  const int64_t body = int64_t(s.body) * H;
  auto value = [&](half_t x, half_t d, half_t e, int h) {
    if (OP == kFwd) return half_t(__expf(float(x) - M[h]) * S[h]);
    return softmax_bwd_value(a, x, d, e, S[h]);
  };
  for (int t = threadIdx.x; t < s.n_body; t += kHubThreads) {
    auto vec = [&](const half_t* p) { return reinterpret_cast<const half8_t*>(p + body)[t]; };
    const half8_t x = vec(a.x0);
    half8_t d = half8_t(0), e = half8_t(1), o;
    if (OP == kBwd) d = vec(a.x1);
    if (OP == kBwd && a.x2) e = vec(a.x2);
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = value(x[q], d[q], e[q], q % H);
    reinterpret_cast<half8_t*>(a.out + body)[t] = o;
  }
  const int i = threadIdx.x;
  if (i < Span<H>::kEnds && s.has(i)) {
    const int64_t at = int64_t(s.end_at(i)) * H;
    auto unit = [&](const half_t* p) { return *reinterpret_cast<const hv_t*>(p + at); };
    const hv_t x = unit(a.x0);
    hv_t d = hv_t(half_t(0)), e = hv_t(half_t(1)), o;
    if (OP == kBwd) d = unit(a.x1);
    if (OP == kBwd && a.x2) e = unit(a.x2);
#pragma unroll
    for (int h = 0; h < H; ++h) o[h] = value(x[h], d[h], e[h], h);
    *reinterpret_cast<hv_t*>(a.out + at) = o;
  }
}

// row sums of the long rows: one thread per (row, head) adds the row's partial sums in chunk order
__global__ __launch_bounds__(kBlock) void edge_hub_rowsum_kernel(EdgeRowArgs a, HubChunks c, const int* __restrict__ big_first,
                                                                 int n_big) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n_big * a.H) return;
  const int r = i / a.H, h = i - r * a.H;
  const int first = big_first[r], cnt = c.count[first];
  float s = 0.f;
  for (int k = 0; k < cnt; ++k) s += c.part[(int64_t(first + k) * a.H + h) * 2];
  a.out[int64_t(a.big_row[r]) * a.H + h] = half_t(s);
}

// Scalar path for head counts that do not divide 8: one thread per (row, head).
template <int OP>
__global__ __launch_bounds__(kBlock) void edge_row_scalar_kernel(EdgeRowArgs a) {
  const int64_t idx = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= int64_t(a.nrows) * a.H) return;
  const int row = int(idx / a.H), h = int(idx % a.H);
  const int beg = a.rowptr[row], end = a.rowptr[row + 1];
  if (OP == kSum) {
    float s = 0.f;
    for (int k = beg; k < end; ++k) s += float(a.x0[(a.eid ? int64_t(a.eid[k]) : int64_t(k)) * a.H + h]);
    a.out[idx] = half_t(s);
    return;
  }
  if (beg == end) return;
  if (OP == kFwd) {
    float m = -INFINITY, z = 0.f;
    for (int k = beg; k < end; ++k) m = fmaxf(m, float(a.x0[int64_t(k) * a.H + h]));
    for (int k = beg; k < end; ++k) z += __expf(float(a.x0[int64_t(k) * a.H + h]) - m);
    const float inv = 1.f / z;
    for (int k = beg; k < end; ++k)
      a.out[int64_t(k) * a.H + h] = half_t(__expf(float(a.x0[int64_t(k) * a.H + h]) - m) * inv);
  } else {
    float t = 0.f;
    for (int k = beg; k < end; ++k) t = fmaf(float(a.x0[int64_t(k) * a.H + h]), float(a.x1[int64_t(k) * a.H + h]), t);
    for (int k = beg; k < end; ++k) {
      const int64_t i = int64_t(k) * a.H + h;
      float d = float(a.x0[i]) * (float(a.x1[i]) - t);
      if (a.x2 && !(float(a.x2[i]) > 0.f)) d *= a.slope;
      a.out[i] = half_t(d);
    }
  }
}

template <int OP, int H>
static void launch_rows_h(int LR, dim3 grid, hipStream_t s, const EdgeRowArgs& a, const HubChunks& c, int n_chunks, int wave_wgs) {
  switch (LR) {
    case 4: edge_rows_kernel<OP, 4, H><<<grid, kHubThreads, 0, s>>>(a, c, n_chunks, wave_wgs); break;
    case 8: edge_rows_kernel<OP, 8, H><<<grid, kHubThreads, 0, s>>>(a, c, n_chunks, wave_wgs); break;
    case 16: edge_rows_kernel<OP, 16, H><<<grid, kHubThreads, 0, s>>>(a, c, n_chunks, wave_wgs); break;
    case 32: edge_rows_kernel<OP, 32, H><<<grid, kHubThreads, 0, s>>>(a, c, n_chunks, wave_wgs); break;
    default: edge_rows_kernel<OP, 64, H><<<grid, kHubThreads, 0, s>>>(a, c, n_chunks, wave_wgs); break;
  }
}

// Whether the listed rows share workgroups (kListTeam), or take a wave each: with four heads a row of 100 non-zeros fills most of a wave, and few
// rows are then better spread.  us, a wave each / shared, forward; backward: 5.5 M non-zeros, 28 000 listed rows, H = 1 22 / 16.7; 22 / 19.5,
// H = 4 52 / 40; 47 / 44, H = 8 86 / 77; 94 / 103; 1.5 M, 9000 listed rows, H = 1 11 / 9.5; 10.5 / 9.9, H = 2 15 / 13; 17 / 16, H = 4 28 / 28;
// 28 / 33, H = 8 52 / 57; 48 / 58.  Without a list they share workgroups with any number of heads, or a wave would be started for every row:
// power law of 1.5 M, H = 4 262 / 154; 249 / 165, H = 8 480 / 350; 470 / 338; log-normal, 6 M of 60 000 rows, H = 4 56 / 45; 45 / 40, H = 8 94 / 77;
// 103 / 95; 300 000 of 1000 rows, H = 8 56 / 40; 46 / 29.
static bool list_teams_pay(int H, int n_list) { return H <= 2 || (H == 4 && n_list >= 16384); }

// Whether half of LR lanes take a row, forward and for row sums.  What a team spends is the exchange between its lanes, twice per head forward; but half of the
// lanes leave half of the waves, need two vectors on each to hold the row, and what they do not hold is read again, or goes to the tier of the longer rows.  So
// the half have to hold a quarter more than the mean, and the waves of all lanes have to be many: 16 a compute unit where the half hold half more than the
// mean and the rows are much alike (of those that the plan does not list few are beyond the half; or most are listed, and no longer than the rest), else 60,
// and 96 where rows differ.  us, all / half:
//   forward, uniform: 40 non-zeros a row, four heads, 1000, 8000, 64 000 rows 3.1 / 3.1, 5.5 / 4.7, 21 / 15; 20, eight heads, 2000, 16 000, 300 000 3.4 / 3.5, 8.3 / 5.7, 95 / 51;
//     6, eight heads, 4000, 32 000, 300 000 3.3 / 4.2, 5.1 / 5.1, 25 / 20; a quarter more: 50, one head, 8000, 64 000 2.9 / 3.4, 6.5 / 7.2, four, 4000, 32 000 3.8 / 4.1, 13 / 10
//   log-normal: 70, two heads, 4000, 16 000, 64 000 4.4 / 5.3, 6.8 / 7.8, 21 / 19; 14, four heads, 1000, 16 000, 300 000 3.2 / 4.2, 4.8 / 5.3, 27 / 26;
//     6, eight heads, 4000, 32 000, 300 000 4.2 / 6.6, 7.6 / 8.6, 33 / 33; 50, 16 000, 64 000 16 / 19, 51 / 49
//   sums, uniform: 20, eight heads, 4000, 32 000 2.6 / 2.6, 4.6 / 3.6; log-normal: 14, four heads, 1000, 16 000, 128 000 2.6 / 2.8, 3.0 / 3.2, 7.4 / 6.4
// With eight heads and a whole wave for a row sums gain nothing (uniform, 50, 64 000 15.7 / 17.6); the backward, with three tensors in registers, neither (6 M
// non-zeros, log-normal, four heads 17.6 / 19.7).
static bool half_of_lanes(const hgnn_plan* p, bool sum, int H, int LR, double mean_len) {
  constexpr int64_t kCus = 256;
  const double held = LR / 2 * 8 * kKeepVec / H;  // by the half
  if (LR <= 4 || held < 1.25 * mean_len || (sum && H == 8 && LR == kWave)) return false;
  const int64_t listed = int64_t(p->n_mid) + p->n_big, waves = int64_t(p->nrows) * LR / kWave;
  const bool alike = listed < p->nrows / 2 ? listed <= p->nrows / 256 || (held >= p->mid_deg && listed <= p->nrows / 8)
                                           : double(p->listed_nnz) <= 1.1 * mean_len * double(listed);
  return waves >= kCus * (!alike ? 96 : (held >= 1.5 * mean_len ? 16 : 60));
}

// Launches the row kernel (and the follow-up of the chunks when a plan lists long rows) for H in {1,2,4,8}.
template <int OP>
static hgnn_status launch_edge_rows(const hgnn_csr* g, const hgnn_plan* p, EdgeRowArgs a, hipStream_t s) {
  const int H = a.H;
  // the chunked long-row kernels keep partial results in the plan, sized for its max_H heads: with more heads than
  // that the call runs as it does without a plan
  if (p && H > p->max_H) p = nullptr;
  if (!(H == 1 || H == 2 || H == 4 || H == 8) || !aligned16(a.x0) || !aligned16(a.out) ||
      (a.x1 && !aligned16(a.x1)) || (a.x2 && !aligned16(a.x2))) {
    edge_row_scalar_kernel<OP><<<dim3(unsigned(ceil_div(int64_t(g->nrows) * H, kBlock))), kBlock, 0, s>>>(a);
    HGNN_LAUNCH_CHECK("edge_row_scalar_kernel");
    return HGNN_OK;
  }
  // lanes per row: about one 8-element vector per lane for the mean row (rowsum over an edge-id map
  // walks one non-zero per lane instead)
  // (with a plan that lists the longer rows for the tiers below: the mean over the rows it does not list, which on
  // a power-law graph is far below the mean over all rows)
  double mean_len = double(g->nnz) / double(g->nrows > 0 ? g->nrows : 1);
  if (p && p->n_mid + p->n_big > 0 && int64_t(p->n_mid) + p->n_big < g->nrows / 2)  // the listed rows are the exception
    mean_len = double(g->nnz - p->listed_nnz) / double(g->nrows - p->n_mid - p->n_big);
  const double per_row = mean_len * ((OP == kSum && a.eid) ? 1.0 : H / 8.0);
  int LR = 4;
  while (LR < kWave && LR < per_row) LR <<= 1;
  if (p && OP != kBwd && !(OP == kSum && a.eid) && half_of_lanes(p, OP == kSum, H, LR, mean_len)) LR >>= 1;
  const int big = (p && p->n_big > 0) ? p->big_deg : 0;
  a.big_row = p ? p->big_row : nullptr;
  // tier 1: sub-wave teams take the rows they can hold in registers; tier 2: a whole wave per row
  // for the rows between that and the plan's long-row threshold; tier 3: the long rows in chunks.
  int t1 = (OP == kSum && a.eid) ? LR * 4 : LR * 8 * kKeepVec / H;
  // a plan lists the rows between its mid and long thresholds: the wave-per-row tier then walks that list
  // instead of starting a wave for every row of the graph only to find most of them done
  const bool mid_list = p && LR < kWave && (big == 0 || big > p->mid_deg);
  if (mid_list && t1 < p->mid_deg) t1 = p->mid_deg;  // the sub-wave tier takes what the list leaves out
  if (LR == kWave) t1 = INT_MAX;  // every row has a wave anyway
  a.team_max = t1;
  a.wave_max = big > 0 ? big : INT_MAX;
  constexpr int64_t rows_per_wg = kHubThreads / kWave;
  int64_t wave_wgs = 0;
  if (LR < kWave && !(big > 0 && t1 >= big)) {
    a.row_list = mid_list ? p->mid_row : nullptr;
    a.n_list = mid_list ? p->n_mid : g->nrows;
    if (!mid_list || list_teams_pay(H, p->n_mid)) a.list_max = OP == kSum && a.eid ? 4 * kListTeam : 4 * 8 * kListTeam / H;
    wave_wgs = a.list_max > 0 ? ceil_div(a.n_list, kListRows * kDealt) * kDealt : ceil_div(a.n_list, rows_per_wg);
  }
  const int n_chunks = big > 0 ? p->n_hub_chunks : 0;
  const HubChunks c = big > 0 ? HubChunks{p->hub_chunk_row, p->hub_chunk_first, p->hub_chunk_count, p->hub_part} : HubChunks{};
  const dim3 grid(unsigned(n_chunks + wave_wgs + ceil_div(g->nrows, rows_per_wg * (kWave / LR))));
  switch (H) {
    case 1: launch_rows_h<OP, 1>(LR, grid, s, a, c, n_chunks, int(wave_wgs)); break;
    case 2: launch_rows_h<OP, 2>(LR, grid, s, a, c, n_chunks, int(wave_wgs)); break;
    case 4: launch_rows_h<OP, 4>(LR, grid, s, a, c, n_chunks, int(wave_wgs)); break;
    default: launch_rows_h<OP, 8>(LR, grid, s, a, c, n_chunks, int(wave_wgs)); break;
  }
  HGNN_LAUNCH_CHECK("edge_rows_kernel");
  if (big > 0) {
    const dim3 gc{unsigned(p->n_hub_chunks)};
    if (OP == kSum) {
      edge_hub_rowsum_kernel<<<dim3(unsigned(ceil_div(int64_t(p->n_big) * H, kBlock))), kBlock, 0, s>>>(a, c, p->big_first,
                                                                                                       p->n_big);
      HGNN_LAUNCH_CHECK("edge_hub_rowsum_kernel");
    } else {
      switch (H) {
        case 1: edge_hub_emit_kernel<OP, 1><<<gc, kHubThreads, 0, s>>>(a, c); break;
        case 2: edge_hub_emit_kernel<OP, 2><<<gc, kHubThreads, 0, s>>>(a, c); break;
        case 4: edge_hub_emit_kernel<OP, 4><<<gc, kHubThreads, 0, s>>>(a, c); break;
        default: edge_hub_emit_kernel<OP, 8><<<gc, kHubThreads, 0, s>>>(a, c); break;
      }
      HGNN_LAUNCH_CHECK("edge_hub_emit_kernel");
    }
  }
  return HGNN_OK;
}

// ---- row sums through an edge-id map, over row tasks ---------------------------------------------------------------------
// Every value is a gather of its own, so the L2s' requests bound the pass; pieces of at most S non-zeros keep the waves
// level whatever the row lengths are, and a lane holds four gathers and the next four slots in flight.  Over column blocks the
// gathered lines are those of one block's columns.
struct RowsumArgs {
  const int* eid;  // slots, in the order of the tasks' column array
  const half_t* t;
  half_t* out;     // [nrows][H], or
  float* part;     // [nb][nrows][H] when the tasks are those of column blocks
  float* stage;    // [slots][H] sums of the pieces of rows that have several
  int64_t nrows;
  template <int H>
  __device__ __forceinline__ void store(int block, int row, const float (&s)[H]) const {
    if (part) {
      float* const p = part + (int64_t(block) * nrows + row) * H;
#pragma unroll
      for (int h = 0; h < H; ++h) p[h] = s[h];
    } else {
#pragma unroll
      for (int h = 0; h < H; ++h) out[int64_t(row) * H + h] = half_t(s[h]);
    }
  }
};
constexpr int kRowsumL = 8;  // lanes per group

template <int H>
__global__ __launch_bounds__(kWave) void rowsum_task_kernel(RowsumArgs a, TaskView v) {
  typedef _Float16 hv_t __attribute__((ext_vector_type(H)));
  typedef Round<kRowsumL, 32> Rd;
  constexpr int E = Rd::E;
  const int lane = threadIdx.x, l = lane % kRowsumL;
  const TaskWave w = task_enter<kRowsumL, Rd::R>(v, blockIdx.x, lane / kRowsumL);
  float s[H];
#pragma unroll
  for (int h = 0; h < H; ++h) s[h] = 0.f;
  if (w.z1 > w.z0) {
    for (pos_t i = w.z0 + lane; i < w.z1; i += kWave) a.template store<H>(w.block, w.zrow[i], s);
    return;
  }
  pos_t k = w.beg + l * E;
  pos_t end = w.beg + w.span < w.end ? w.beg + w.span : w.end;
  int id[E];
  load_run<E, true>(a.eid, k, RunLeft{int(end - k)}, id);  // positions past the end hold slot 0: read, not added
  for (pos_t base = w.beg; base < w.end; base += w.step) {
    hv_t x[E];
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = *reinterpret_cast<const hv_t*>(a.t + int64_t(id[m]) * H);
    const pos_t kn = k + w.step, past = base + w.step + w.span;
    const pos_t endn = past < w.end ? past : w.end;
    load_run<E, true>(a.eid, kn, RunLeft{int(endn - kn)}, id);
    const int left = int(end - k);
#pragma unroll
    for (int m = 0; m < E; ++m)
#pragma unroll
      for (int h = 0; h < H; ++h) s[h] += m < left ? float(x[m][h]) : 0.f;
    k = kn;
    end = endn;
  }
  if (w.whole) team_reduce<kWave, H, false>(s);
  else team_reduce<kRowsumL, H, false>(s);
  if (w.row < 0 || (w.whole ? lane : l) != 0) return;
  if (w.slot < 0) {
    a.template store<H>(w.block, w.row, s);
  } else {
#pragma unroll
    for (int h = 0; h < H; ++h) a.stage[int64_t(w.slot) * H + h] = s[h];
  }
}

// a wave per row of several pieces
template <int H>
__global__ __launch_bounds__(kBlock) void rowsum_task_finish_kernel(RowsumArgs a, const int4_t* __restrict__ split, int n_split) {
  const int i = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  if (i >= n_split) return;
  const int4_t q = split[i];  // row, first slot, pieces, block
  float s[H];
#pragma unroll
  for (int h = 0; h < H; ++h) s[h] = 0.f;
  for (int k = lane; k < q[2]; k += kWave)
#pragma unroll
    for (int h = 0; h < H; ++h) s[h] += a.stage[int64_t(q[1] + k) * H + h];
  team_reduce<kWave, H, false>(s);
  if (lane == 0) a.template store<H>(q[3], q[0], s);
}

template <int H>
static hgnn_status launch_rowsum_tasks(const hgnn_row_tasks* t, const RowsumArgs& a, hipStream_t s) {
  const TaskView v = task_view(t, kWave / kRowsumL, at_ranges(t, kRangesSums, t->nnz * H * 2, 0), true);
  if (v.first_wave[t->nb] > 0) {
    rowsum_task_kernel<H><<<dim3(unsigned(v.first_wave[t->nb])), kWave, 0, s>>>(a, v);
    HGNN_LAUNCH_CHECK("rowsum_task_kernel");
  }
  if (v.n_split > 0) {
    rowsum_task_finish_kernel<H><<<dim3(unsigned(ceil_div(v.n_split, kWavesPerBlock))), kBlock, 0, s>>>(a, v.split, v.n_split);
    HGNN_LAUNCH_CHECK("rowsum_task_finish_kernel");
  }
  return HGNN_OK;
}

// column-blocked row sums: out[i] = sum over the blocks of their fp32 partial sums
__global__ __launch_bounds__(kBlock) void rowsum_block_sum_kernel(const float* __restrict__ part, int nb, int64_t n,
                                                                   half_t* __restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int b = 0; b < nb; ++b) s += part[int64_t(b) * n + i];
  out[i] = half_t(s);
}

static hgnn_status edge_rows_common(const char* who, const hgnn_csr* g, const hgnn_plan* p, int H, bool allow_eid) {
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(H >= 1, HGNN_EINVAL, "%s: H = %d must be positive", who, H);
  HGNN_REQUIRE(allow_eid || g->eid == nullptr, HGNN_EUNSUPPORTED, "%s: an edge-id map is not supported here", who);
  if (p)
    HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
                 "%s: the plan was built for another graph", who);
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

extern "C" {

hgnn_status hgnn_edge_softmax(const hgnn_csr* g, const hgnn_plan* p, int32_t H, const hgnn_half* e, hgnn_half* alpha,
                              void* stream) {
  clear_error();
  hgnn_status st = edge_rows_common("hgnn_edge_softmax", g, p, H, false);
  if (st != HGNN_OK) return st;
  if (g->nnz == 0 || g->nrows == 0) return HGNN_OK;
  HGNN_REQUIRE(e && alpha, HGNN_EINVAL, "hgnn_edge_softmax: e or alpha is NULL");
  EdgeRowArgs a{};
  a.rowptr = g->rowptr;
  a.x0 = reinterpret_cast<const half_t*>(e);
  a.out = reinterpret_cast<half_t*>(alpha);
  a.nrows = g->nrows;
  a.H = H;
  return launch_edge_rows<kFwd>(g, p, a, static_cast<hipStream_t>(stream));
}

hgnn_status hgnn_edge_softmax_bwd(const hgnn_csr* g, const hgnn_plan* p, int32_t H, const hgnn_half* alpha,
                                  const hgnn_half* dalpha, const hgnn_half* e, float neg_slope, hgnn_half* de,
                                  void* stream) {
  clear_error();
  hgnn_status st = edge_rows_common("hgnn_edge_softmax_bwd", g, p, H, false);
  if (st != HGNN_OK) return st;
  if (g->nnz == 0 || g->nrows == 0) return HGNN_OK;
  HGNN_REQUIRE(alpha && dalpha && de, HGNN_EINVAL, "hgnn_edge_softmax_bwd: alpha, dalpha or de is NULL");
  EdgeRowArgs a{};
  a.rowptr = g->rowptr;
  a.x0 = reinterpret_cast<const half_t*>(alpha);
  a.x1 = reinterpret_cast<const half_t*>(dalpha);
  a.x2 = reinterpret_cast<const half_t*>(e);
  a.out = reinterpret_cast<half_t*>(de);
  a.nrows = g->nrows;
  a.H = H;
  a.slope = neg_slope;
  return launch_edge_rows<kBwd>(g, p, a, static_cast<hipStream_t>(stream));
}

hgnn_status hgnn_edge_rowsum(const hgnn_csr* g, const hgnn_plan* p, int32_t H, const hgnn_half* t, hgnn_half* out,
                             void* stream) {
  clear_error();
  hgnn_status st = edge_rows_common("hgnn_edge_rowsum", g, p, H, true);
  if (st != HGNN_OK) return st;
  if (g->nrows == 0) return HGNN_OK;
  HGNN_REQUIRE(out != nullptr && (g->nnz == 0 || t != nullptr), HGNN_EINVAL, "hgnn_edge_rowsum: t or out is NULL");
  EdgeRowArgs a{};
  a.rowptr = g->rowptr;
  a.eid = g->eid;
  a.x0 = reinterpret_cast<const half_t*>(t);
  a.out = reinterpret_cast<half_t*>(out);
  a.nrows = g->nrows;
  a.H = H;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!(p && g->eid && H <= p->max_H && g->nnz > 0 && (H == 1 || H == 2 || H == 4 || H == 8) && aligned16(t)))
    return launch_edge_rows<kSum>(g, p, a, s);
  const bool blocked = p->nb > 1 && p->block_eid;
  if (blocked) p = walked_cut(p, true);
  const hgnn_row_tasks* const tasks = blocked ? p->btasks : p->tasks;
  const RowsumArgs r{blocked ? p->beid : g->eid, a.x0, a.out, blocked ? p->bsum : nullptr, tasks->stage_mz, g->nrows};
  switch (H) {
    case 1: st = launch_rowsum_tasks<1>(tasks, r, s); break;
    case 2: st = launch_rowsum_tasks<2>(tasks, r, s); break;
    case 4: st = launch_rowsum_tasks<4>(tasks, r, s); break;
    default: st = launch_rowsum_tasks<8>(tasks, r, s); break;
  }
  if (st != HGNN_OK || !blocked) return st;
  const int64_t nout = int64_t(g->nrows) * H;
  rowsum_block_sum_kernel<<<dim3(unsigned(ceil_div(nout, kBlock))), kBlock, 0, s>>>(p->bsum, p->nb, nout, a.out);
  HGNN_LAUNCH_CHECK("rowsum_block_sum_kernel");
  return HGNN_OK;
}

}  // extern "C"

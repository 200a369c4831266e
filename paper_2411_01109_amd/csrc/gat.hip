// Single-pass GAT aggregation for gfx950: score, edge softmax and weighted sum of the neighbours'
// features in one read of the graph, with no per-edge tensor written (the paper, sections 3.1.2 and
// 5.2, keeps them as three kernels with an |E| x H score tensor and an |E| x H alpha tensor between
// them; this fuses them on top of the same discretized, atomic-free design).
//
//   s_k = el[i,h] + er[col k,h],  e_k = LeakyReLU(s_k),  alpha_k = softmax over row i (Eq. 1),
//   out[i, h*D+d] = sum_k alpha_k * X[col k, h*D+d],    lse[i,h] = log sum_k exp(e_k)
//
// el[i,h] = a_l.U[i,h] is a per-vertex projection (fp32, formed once per vertex); er[j,h] = a_r.X[j,h] is formed
// per edge from the gathered row X[j] itself.
// A partial result over any subset of a row's edges is kept as a triple (m, z, acc): m = largest
// score met, z = sum exp(e - m), acc = sum exp(e - m) * x.  Two triples of the same row merge by
// rescaling both to the larger m (the online form of Eq. 1's shift by the row maximum), so the
// row tasks can cut rows anywhere: a lane group carries a running triple along its piece, the groups
// of a wave that share a long piece merge theirs across lanes, and the pieces of a row that has several are staged as
// (m, z) in fp32 plus the normalised vector acc/z in fp16 -- a convex combination of feature rows,
// hence never larger than the features themselves (the discretized-scaling idea of section 5.2.2
// applied to the softmax weights) -- and a follow-up kernel merges them.  No atomics, one writer per
// output row, fixed merge order.
//
// SAVE kernels also keep, per row and head, what the backward pass needs to form the gradient of the row-side
// score term without another pass over the edges: with mu_k = 1 where s_k > 0 and the LeakyReLU slope elsewhere,
//   out_masked[i, h*D+d] = sum_k alpha_k * mu_k * X[col k, h*D+d],   csum[i,h] = sum_k alpha_k * mu_k
// (then sum_k ds_k = <dOut_i, out_masked_i> - <dOut_i, out_i> * csum_i).  They ride on the same gathered rows:
// a second accumulator and a second sum in every triple, rescaled with the first.
#include "task.h"

namespace hgnn {

struct GatArgs {
  const int* col;
  const half_t* X;  // column-side features [ncols][ldx]
  half_t* Y;        // [nrows][ldy]: the result, or (part_mz set) this block's normalised partial rows
  int64_t ldx, ldy;
  int nrows, F, H, D;
  float slope;
  const float* el;  // [nrows][H], or nullptr: formed per piece from the row's own features
  const half_t* U;  // row-side features [nrows][ldu] and their attention vector [H*D] (el == nullptr)
  int64_t ldu;
  const half_t* a_l;
  const half_t* a_r;  // [H*D]
  float* lse;       // [nrows][H] or nullptr
  float* part_mz;   // column blocks: [nrows][H][2] (m, z) of this block's partial rows; else nullptr
  half_t* Ym;       // SAVE: [nrows][ldym] masked result (or this block's normalised partial rows)
  int64_t ldym;
  float* csum;      // SAVE: [nrows][H] masked weight sum (or, with part_mz, this block's share, relative to its z)
  half_t* staging_m;  // SAVE: [slots][stage_ld] masked counterpart of staging
  float* stage_c;     // SAVE: [slots][H] masked weight sum of a staged piece, relative to its z
  half_t* staging;  // [slots][stage_ld] normalised vectors of the pieces of rows that have several
  float* stage_mz;  // [slots][H][2]
  int stage_ld;
  // column blocks in one launch (waves numbered block after block): Y, part_mz, Ym and csum point at block 0's partial
  // results and advance by the strides per block
  int64_t y_stride, mz_stride, c_stride;
  __device__ __forceinline__ void enter_block(int b) {
    Y += int64_t(b) * y_stride;
    if (part_mz) part_mz += int64_t(b) * mz_stride;
    if (Ym) {
      Ym += int64_t(b) * y_stride;
      csum += int64_t(b) * c_stride;
    }
  }
};

// A partial result of one row and head over some of its edges, as held by one lane (8 features):
// m = largest score met, z = sum exp(e - m), acc = sum exp(e - m) * x; SAVE adds zm = sum exp(e - m) * mu and
// accm = sum exp(e - m) * mu * x.
template <bool SAVE>
struct Soft {
  float m = -INFINITY, z = 0.f, zm = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float accm[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ void clear() {
    m = -INFINITY;
    z = 0.f;
    zm = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = 0.f;
      accm[i] = 0.f;
    }
  }
  __device__ __forceinline__ void scale(float f) {
#pragma clang fp contract(off)
    z *= f;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= f;
    if (SAVE) {
      zm *= f;
#pragma unroll
      for (int i = 0; i < 8; ++i) accm[i] *= f;
    }
  }
};

// The sums of a row are written out in fused and plain operations, with nothing left to contraction: the kernels with and
// without SAVE give the same bits.

// a <- a merged with b (both rescaled to the larger maximum)
template <bool SAVE>
__device__ __forceinline__ void soft_merge(Soft<SAVE>& a, const Soft<SAVE>& b) {
#pragma clang fp contract(off)
  const float M = fmaxf(a.m, b.m);
  if (M == -INFINITY) return;  // both empty
  const float fa = __expf(a.m - M), fb = __expf(b.m - M);  // exp(-inf) = 0 drops an empty side
  a.z = fmaf(b.z, fb, a.z * fa);
#pragma unroll
  for (int i = 0; i < 8; ++i) a.acc[i] = fmaf(b.acc[i], fb, a.acc[i] * fa);
  if (SAVE) {
    a.zm = fmaf(b.zm, fb, a.zm * fa);
#pragma unroll
    for (int i = 0; i < 8; ++i) a.accm[i] = fmaf(b.accm[i], fb, a.accm[i] * fa);
  }
  a.m = M;
}

// merge a staged piece: (mp, zp), its normalised vector o = acc/z and, SAVE, cp = zm/z and om = accm/z
template <bool SAVE>
__device__ __forceinline__ void soft_merge_normalised(Soft<SAVE>& a, float mp, float zp, float cp, const half8_t& o,
                                                      const half8_t& om) {
#pragma clang fp contract(off)
  const float M = fmaxf(a.m, mp);
  if (M == -INFINITY) return;
  const float fa = __expf(a.m - M), fb = __expf(mp - M) * zp;
  a.z = fmaf(a.z, fa, fb);
#pragma unroll
  for (int i = 0; i < 8; ++i) a.acc[i] = fmaf(fb, float(o[i]), a.acc[i] * fa);
  if (SAVE) {
    a.zm = fmaf(fb, cp, a.zm * fa);
#pragma unroll
    for (int i = 0; i < 8; ++i) a.accm[i] = fmaf(fb, float(om[i]), a.accm[i] * fa);
  }
  a.m = M;
}

__device__ __forceinline__ void store_vec8(half_t* p, int f0, const float (&v)[8], float s) {
  half8_t h;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float r = v[i] * s;
    asm("" : "+v"(r));  // rounded to fp32 first, not fused into the conversion
    h[i] = half_t(r);
  }
  *reinterpret_cast<half8_t*>(p + f0) = h;
}

// a finished row (or, with part_mz, a finished partial row of a column block)
template <bool SAVE>
__device__ __forceinline__ void row_store(const GatArgs& a, int64_t row, int f0, int head, bool leader, const Soft<SAVE>& t) {
  const float inv = t.z > 0.f ? 1.f / t.z : 0.f;
  store_vec8(a.Y + row * a.ldy, f0, t.acc, inv);
  if (SAVE) store_vec8(a.Ym + row * a.ldym, f0, t.accm, inv);
  if (!leader) return;
  if (SAVE) a.csum[row * a.H + head] = t.zm * inv;
  if (a.part_mz) {
    a.part_mz[(row * a.H + head) * 2] = t.m;
    a.part_mz[(row * a.H + head) * 2 + 1] = t.z;
  } else if (a.lse) {
    a.lse[row * a.H + head] = t.z > 0.f ? t.m + __logf(t.z) : 0.f;
  }
}

template <bool SAVE>
__device__ __forceinline__ void stage_store(const GatArgs& a, int64_t slot, int f0, int head, bool leader, const Soft<SAVE>& t) {
  const float inv = t.z > 0.f ? 1.f / t.z : 0.f;
  store_vec8(a.staging + slot * a.stage_ld, f0, t.acc, inv);
  if (SAVE) store_vec8(a.staging_m + slot * a.stage_ld, f0, t.accm, inv);
  if (leader) {
    a.stage_mz[(slot * a.H + head) * 2] = t.m;
    a.stage_mz[(slot * a.H + head) * 2 + 1] = t.z;
    if (SAVE) a.stage_c[slot * a.H + head] = t.zm * inv;
  }
}

// The running maximum of a row only has to keep the exponentials in range, so it follows the scores lazily: it is raised,
// and the sums rescaled, when a score exceeds it by more than kSlack (weights up to e^8, far inside fp32).
constexpr float kSlack = 8.f;

template <bool SAVE, int RS, int U>
__device__ __forceinline__ void soft_add(Soft<SAVE>& t, const float (&p)[8 / RS], const float (&pm)[8 / RS], const half8_t& x) {
  const float w = HeadTile<RS>::template from_owner<U>(p);
#pragma unroll
  for (int q = 0; q < 8; ++q) t.acc[q] = fmaf(w, float(x[q]), t.acc[q]);
  if (SAVE) {
    const float wm = HeadTile<RS>::template from_owner<U>(pm);
#pragma unroll
    for (int q = 0; q < 8; ++q) t.accm[q] = fmaf(wm, float(x[q]), t.accm[q]);
  }
}

// Pass over row tasks (see spmm_task_kernel for how a wave is laid out).  The row-side term el[row] is constant in a
// lane group; the column-side term a_r.X[col] is formed from the gathered row itself (four two-way dot products per lane).
// RS = min(lanes per head, 8).
//
// Bound: vector instructions (they are busy 93 % of the cycles with SAVE, 79-84 % without), then the gathers.  The walk over equal
// runs of edges repeated maximum, exponential and masks on every lane of a head, rescaled two sums every four edges, and most steps had
// a row change in some lane group; here a wave spends 10 vector instructions per edge with SAVE, 7 without (5.5 M edges, 4 heads of
// 16).  A call against that walk: 5.5 M edges, 4 heads of 16, SAVE 181 -> 106 us, without 125 -> 83; 114 M edges, one head of
// 64 in eight blocks 2.16 -> 1.08 ms, 1.48 -> 0.88 ms.
template <int L, bool NEAR, bool SAVE, int RS, int MOST>
__global__ __launch_bounds__(kWave, 5 - (SAVE && RS == 1)) void gat_task_kernel(GatArgs a, TaskView v, int ncols) {
#pragma clang fp contract(off)
  constexpr int G = kWave / L;
  typedef Round<L, MOST> Rd;
  typedef HeadTile<RS> Ht;
  __shared__ __align__(16) int s_handles[G * Rd::PITCH];
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int LH = a.D / 8;  // lanes per head, a power of two
  const int head = head_of_lane(active ? l : 0, LH);
  const bool leader = active && (l & (LH - 1)) == 0;  // the lane that writes its head's scalars
  const TaskWave w = task_enter<L, Rd::R>(v, blockIdx.x, g);
  a.enter_block(w.block);
  if (w.z1 > w.z0) {
    const Soft<SAVE> none;
    for (pos_t i = w.z0 + g; i < w.z1; i += G)
      if (active) row_store<SAVE>(a, w.zrow[i], f0, head, leader, none);
    return;
  }
  int* const s_hnd = s_handles + g * Rd::PITCH;
  const RowTable<NEAR> table(a.X, ncols, a.ldx, f0c);
  const int row = w.row >= 0 ? w.row : 0;
  float el;
  if (a.el) {
    el = a.el[int64_t(row) * a.H + head];
  } else {
    el = dot8(*reinterpret_cast<const half8_t*>(a.a_l + f0c), *reinterpret_cast<const half8_t*>(a.U + int64_t(row) * a.ldu + f0c));
    el = head_sum1(active ? el : 0.f, LH);
  }
  half2_t ar2[4];
  {
    const half8_t t = *reinterpret_cast<const half8_t*>(a.a_r + f0c);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ar2[q][0] = active ? t[2 * q] : half_t(0);
      ar2[q][1] = active ? t[2 * q + 1] : half_t(0);
    }
  }
  const int own = (lane & (Rd::LC - 1)) * Rd::E;
  const int edge = Ht::own_edge(l);
  Soft<SAVE> t;  // z and zm: this lane's edges only, until the end
  for (pos_t k = w.beg; k < w.end; k += w.step) {
    const pos_t end = k + w.span < w.end ? k + w.span : w.end;
    const int n = int(end - k);
    wave_sync();  // the previous round has been read
    {
      const int left = n - own;  // entries of this lane's run
      int c[Rd::E];
      load_cols<Rd::E>(v, a.col, false, w.block, k, own, RunLeft{left}, c);
#pragma unroll
      for (int m = 0; m < Rd::E; ++m) c[m] = table.handle(c[m], m < left);
#pragma unroll
      for (int m = 0; m < Rd::E; m += 4)
        *reinterpret_cast<int4_t*>(s_hnd + own + m) = int4_t{c[m], c[m + 1], c[m + 2], c[m + 3]};
    }
    wave_sync();
    for (int q = 0; q < n; q += 8) {
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
      float d[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        d[u] = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // two fp16 products per instruction, fp32 sum
          half2_t xv;
          xv[0] = x[u][2 * j];
          xv[1] = x[u][2 * j + 1];
          d[u] = __builtin_amdgcn_fdot2(ar2[j], xv, d[u], false);
        }
      }
      if (RS == 8 && LH > 8) {  // heads of more than eight lanes: the eights are added first
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          d[u] += dpp_mov<0x128>(d[u]);
          if (LH > 16) d[u] = xor16_mov(d[u], false);
          if (LH > 32) d[u] = xor32_mov(d[u], false);
        }
      }
      float s[Ht::NS];
      Ht::scores(d, l, s);
      bool above = false;
#pragma unroll
      for (int j = 0; j < Ht::NS; ++j) {
        const float e = s[j] + el;
        s[j] = q + j * RS + edge < n ? e : -INFINITY;
        const float lk = s[j] > 0.f ? s[j] : a.slope * s[j];
        above |= lk > t.m + kSlack;
      }
      if (__any(above)) {
        float mx = t.m;
#pragma unroll
        for (int j = 0; j < Ht::NS; ++j) mx = fmaxf(mx, s[j] > 0.f ? s[j] : a.slope * s[j]);
        mx = Ht::max_of(mx);
        // a head in which no score exceeds the slack keeps its maximum, unless it has none yet
        const float mn = mx > t.m + kSlack ? mx : t.m;
        t.scale(__expf(t.m - mn));  // exp(-inf) = 0 on the first tile
        t.m = mn;
      }
      float p[Ht::NS], pm[Ht::NS];
#pragma unroll
      for (int j = 0; j < Ht::NS; ++j) {
        p[j] = __expf((s[j] > 0.f ? s[j] : a.slope * s[j]) - t.m);
        t.z += p[j];
        pm[j] = s[j] > 0.f ? p[j] : p[j] * a.slope;
        if (SAVE) t.zm += pm[j];
      }
      soft_add<SAVE, RS, 0>(t, p, pm, x[0]);
      soft_add<SAVE, RS, 1>(t, p, pm, x[1]);
      soft_add<SAVE, RS, 2>(t, p, pm, x[2]);
      soft_add<SAVE, RS, 3>(t, p, pm, x[3]);
      soft_add<SAVE, RS, 4>(t, p, pm, x[4]);
      soft_add<SAVE, RS, 5>(t, p, pm, x[5]);
      soft_add<SAVE, RS, 6>(t, p, pm, x[6]);
      soft_add<SAVE, RS, 7>(t, p, pm, x[7]);
    }
  }
  t.z = Ht::sum(t.z);
  if (SAVE) t.zm = Ht::sum(t.zm);
  if (w.whole) {
    const float M = across_groups_max<L>(t.m);  // finite: a piece has at least one edge
    t.scale(__expf(t.m - M));
    t.m = M;
    t.z = across_groups_sum<L>(t.z);
#pragma unroll
    for (int i = 0; i < 8; ++i) t.acc[i] = across_groups_sum<L>(t.acc[i]);
    if (SAVE) {
      t.zm = across_groups_sum<L>(t.zm);
#pragma unroll
      for (int i = 0; i < 8; ++i) t.accm[i] = across_groups_sum<L>(t.accm[i]);
    }
    if (g) return;
  }
  if (!active || w.row < 0) return;
  if (w.slot < 0) row_store<SAVE>(a, row, f0, head, leader, t);
  else stage_store<SAVE>(a, w.slot, f0, head, leader, t);
}

// Follow-up kernel: merges the staged pieces of every row that has several and stores the row.  A wave owns one such
// row, or G (finish_rows_per_wave): then rows of up to kShortPieces pieces are merged by their own lane group, hubs by the whole
// wave with a final merge across the groups.
constexpr int kShortPieces = 8;

template <int L, bool SAVE, bool MANY>
__global__ __launch_bounds__(kBlock) void gat_finish_kernel(GatArgs a, const int4_t* __restrict__ split, int n_split, int per_wave) {
#pragma clang fp contract(off)
  constexpr int G = kWave / L, kMany = kManyPieces * G;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int LH = a.D / 8, head = head_of_lane(active ? l : 0, LH);
  const bool leader = active && (l & (LH - 1)) == 0;
  const int64_t i0 = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * per_wave;
  if ((MANY ? int64_t(blockIdx.x) * kWavesPerBlock * per_wave : i0) >= n_split) return;  // MANY: the whole workgroup
  __shared__ int4_t s_row[kWavesPerBlock * G];
  __shared__ __align__(4) unsigned char s_bytes[kWavesPerBlock * L * sizeof(Soft<SAVE>)];
  Soft<SAVE>* const s_soft = reinterpret_cast<Soft<SAVE>*>(s_bytes);
  __shared__ int s_n;
  if (MANY) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
  }
  int4_t q = {0, 0, 0, 0};  // row, first slot, pieces, block
  if (g < per_wave && i0 + g < n_split) q = split[i0 + g];
  if (MANY && q[2] > kMany && l == 0) s_row[atomicAdd(&s_n, 1)] = q;
  const int alone = per_wave > 1 ? kShortPieces : 0;
  // merges the pieces first, first + stride, ... < end, four of them in flight at a time
  auto take = [&](Soft<SAVE>& t, pos_t first, pos_t end, pos_t stride) {
    for (pos_t k0 = first; k0 < end; k0 += 4 * stride) {
      half8_t o[4], om[4];
      float m[4], z[4], cp[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const pos_t k = k0 + u * stride;
        const int64_t slot = k < end ? k : k0;
        o[u] = *reinterpret_cast<const half8_t*>(a.staging + slot * a.stage_ld + f0c);
        om[u] = SAVE ? *reinterpret_cast<const half8_t*>(a.staging_m + slot * a.stage_ld + f0c) : o[u];
        m[u] = a.stage_mz[(slot * a.H + head) * 2];
        z[u] = a.stage_mz[(slot * a.H + head) * 2 + 1];
        cp[u] = SAVE ? a.stage_c[slot * a.H + head] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + u * stride < end) soft_merge_normalised<SAVE>(t, m[u], z[u], cp[u], o[u], om[u]);
    }
  };
  auto across = [&](Soft<SAVE>& t) {  // merges those of the lane groups
    const float M = across_groups_max<L>(t.m);
    t.scale(M == -INFINITY ? 1.f : __expf(t.m - M));  // exp(-inf) = 0 drops a lane group without a piece
    t.m = M;
    t.z = across_groups_sum<L>(t.z);
#pragma unroll
    for (int i = 0; i < 8; ++i) t.acc[i] = across_groups_sum<L>(t.acc[i]);
    if (SAVE) {
      t.zm = across_groups_sum<L>(t.zm);
#pragma unroll
      for (int i = 0; i < 8; ++i) t.accm[i] = across_groups_sum<L>(t.accm[i]);
    }
  };
  if (q[2] > 0 && q[2] <= alone) {
    Soft<SAVE> t;
    take(t, q[1], q[1] + q[2], 1);
    GatArgs b = a;
    b.enter_block(q[3]);
    if (active) row_store<SAVE>(b, q[0], f0, head, leader, t);
  }
  for (int j = 0; j < per_wave; ++j) {
    const int n = __shfl(q[2], j * L);
    if (n <= alone || (MANY && n > kMany)) continue;
    const int rj = __shfl(q[0], j * L), first = __shfl(q[1], j * L), bj = __shfl(q[3], j * L);
    Soft<SAVE> t;
    take(t, first + g, first + n, G);
    across(t);
    GatArgs b = a;
    b.enter_block(bj);
    if (g == 0 && active) row_store<SAVE>(b, rj, f0, head, leader, t);
  }
  if (!MANY) return;
  __syncthreads();
  for (int j = 0; j < s_n; ++j) {  // the rows of many pieces, one after the other (in whatever order), by all waves
    const int4_t r = s_row[j];
    Soft<SAVE> t;
    take(t, pos_t(r[1]) + wave * G + g, pos_t(r[1]) + r[2], kWavesPerBlock * G);
    across(t);
    if (g == 0) s_soft[wave * L + l] = t;
    __syncthreads();
    if (wave == j % kWavesPerBlock && g == 0 && active) {
      t = s_soft[l];
#pragma unroll
      for (int w = 1; w < kWavesPerBlock; ++w) soft_merge<SAVE>(t, s_soft[w * L + l]);
      GatArgs b = a;
      b.enter_block(r[3]);
      row_store<SAVE>(b, r[0], f0, head, leader, t);
    }
    __syncthreads();
  }
}

// Column-blocked plans: merges the nb partial rows (normalised fp16 vectors + (m, z[, zm/z])) of every row.
struct GatBlockParts {
  const half_t* vec;    // [nb][nrows][ld]
  const half_t* vec_m;  // SAVE: the masked counterpart
  int ld;
  const float* mz;      // [nb] x mz_stride: [nrows][H][2]
  int64_t mz_stride;
  const float* c;       // SAVE: [nb] x c_stride: [nrows][H]
  int64_t c_stride;
  int nb;
};

template <int L, bool SAVE>
__global__ __launch_bounds__(kBlock) void gat_block_merge_kernel(GatArgs a, GatBlockParts q) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const int64_t r = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  if (r >= a.nrows || f0 >= a.F) return;
  const int LH = a.D / 8, head = head_of_lane(l, LH);
  Soft<SAVE> t;
  for (int b = 0; b < q.nb; ++b) {
    const int64_t pr = int64_t(b) * a.nrows + r;
    const half8_t o = *reinterpret_cast<const half8_t*>(q.vec + pr * q.ld + f0);
    half8_t om = o;
    float cp = 0.f;
    if (SAVE) {
      om = *reinterpret_cast<const half8_t*>(q.vec_m + pr * q.ld + f0);
      cp = q.c[b * q.c_stride + r * a.H + head];
    }
    const float* mz = q.mz + b * q.mz_stride + (r * a.H + head) * 2;
    soft_merge_normalised<SAVE>(t, mz[0], mz[1], cp, o, om);
  }
  row_store<SAVE>(a, r, f0, head, (l & (LH - 1)) == 0, t);
}

template <int L, bool NEAR, bool SAVE>
static void launch_gat_tasks_l(int lh, unsigned waves, hipStream_t s, const GatArgs& a, const TaskView& v, int ncols) {
  with_round<L, NEAR>(v, [&](auto most) {
    constexpr int M = decltype(most)::value;
    if (lh == 1) gat_task_kernel<L, NEAR, SAVE, 1, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else if (lh == 2) gat_task_kernel<L, NEAR, SAVE, L < 2 ? L : 2, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else if (lh == 4) gat_task_kernel<L, NEAR, SAVE, L < 4 ? L : 4, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else gat_task_kernel<L, NEAR, SAVE, L < 8 ? L : 8, M><<<waves, kWave, 0, s>>>(a, v, ncols);
  });
}

template <bool NEAR, bool SAVE>
static void launch_gat_tasks(int L, int lh, unsigned waves, hipStream_t s, const GatArgs& a, const TaskView& v, int ncols) {
  switch (L) {
    case 1: launch_gat_tasks_l<1, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    case 2: launch_gat_tasks_l<2, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    case 4: launch_gat_tasks_l<4, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    case 8: launch_gat_tasks_l<8, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    case 16: launch_gat_tasks_l<16, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    case 32: launch_gat_tasks_l<32, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
    default: launch_gat_tasks_l<64, NEAR, SAVE>(lh, waves, s, a, v, ncols); break;
  }
}

template <int L>
static void launch_gat_finish_l(bool save, dim3 grid, int per_wave, hipStream_t s, const GatArgs& a, const TaskView& v) {
  if (many_pieces(v, kWave / L)) {
    if (save) gat_finish_kernel<L, true, true><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
    else gat_finish_kernel<L, false, true><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
  } else {
    if (save) gat_finish_kernel<L, true, false><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
    else gat_finish_kernel<L, false, false><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
  }
}

static void launch_gat_finish(int L, bool save, hipStream_t s, const GatArgs& a, const TaskView& v) {
  const int per_wave = finish_rows_per_wave(v.n_split, v.n_slots, kWave / L);
  const dim3 grid(unsigned(ceil_div(v.n_split, int64_t(kWavesPerBlock) * per_wave)));
  switch (L) {
    case 1: launch_gat_finish_l<1>(save, grid, per_wave, s, a, v); break;
    case 2: launch_gat_finish_l<2>(save, grid, per_wave, s, a, v); break;
    case 4: launch_gat_finish_l<4>(save, grid, per_wave, s, a, v); break;
    case 8: launch_gat_finish_l<8>(save, grid, per_wave, s, a, v); break;
    case 16: launch_gat_finish_l<16>(save, grid, per_wave, s, a, v); break;
    case 32: launch_gat_finish_l<32>(save, grid, per_wave, s, a, v); break;
    default: launch_gat_finish_l<64>(save, grid, per_wave, s, a, v); break;
  }
}

template <int L>
static void launch_gat_block_merge_l(bool save, dim3 grid, hipStream_t s, const GatArgs& a, const GatBlockParts& q) {
  if (save) gat_block_merge_kernel<L, true><<<grid, kBlock, 0, s>>>(a, q);
  else gat_block_merge_kernel<L, false><<<grid, kBlock, 0, s>>>(a, q);
}

static void launch_gat_block_merge(int L, bool save, dim3 grid, hipStream_t s, const GatArgs& a, const GatBlockParts& q) {
  switch (L) {
    case 1: launch_gat_block_merge_l<1>(save, grid, s, a, q); break;
    case 2: launch_gat_block_merge_l<2>(save, grid, s, a, q); break;
    case 4: launch_gat_block_merge_l<4>(save, grid, s, a, q); break;
    case 8: launch_gat_block_merge_l<8>(save, grid, s, a, q); break;
    case 16: launch_gat_block_merge_l<16>(save, grid, s, a, q); break;
    case 32: launch_gat_block_merge_l<32>(save, grid, s, a, q); break;
    default: launch_gat_block_merge_l<64>(save, grid, s, a, q); break;
  }
}

// pass over the row tasks t of plan p + follow-up pass
static hgnn_status run_gat_tasks(const hgnn_plan* p, const hgnn_row_tasks* t, GatArgs a, int ncols, hipStream_t s) {
  a.staging = reinterpret_cast<half_t*>(t->staging);
  a.stage_mz = t->stage_mz;
  a.stage_ld = p->max_F;
  const bool save = a.Ym != nullptr;
  // a second set of staging vectors and a third scalar per staged piece lie behind the first
  a.staging_m = a.staging + size_t(t->stage_slots) * size_t(p->max_F);
  a.stage_c = t->stage_mz + size_t(2) * size_t(t->stage_slots) * size_t(p->max_H);
  const int L = pow2_at_least(a.F / 8), G = kWave / L, lh = a.D / 8;
  TaskView v = task_view(t, G, at_ranges(t, kRangesAttention, int64_t(ncols) * a.F * 2, p->l2_bytes), comes_back(false, int64_t(ncols) * a.ldx * 2, p->llc_bytes));
  v.longer = long_rounds(t->nb, p->nrows, t->nnz, p->S, G, 4);
  const int waves = v.first_wave[t->nb];
  if (waves > 0) {
    const bool near = near_table(ncols, a.ldx);
    if (near && save) launch_gat_tasks<true, true>(L, lh, unsigned(waves), s, a, v, ncols);
    else if (near) launch_gat_tasks<true, false>(L, lh, unsigned(waves), s, a, v, ncols);
    else if (save) launch_gat_tasks<false, true>(L, lh, unsigned(waves), s, a, v, ncols);
    else launch_gat_tasks<false, false>(L, lh, unsigned(waves), s, a, v, ncols);
    HGNN_LAUNCH_CHECK("gat_task_kernel");
  }
  if (v.n_split > 0) {
    launch_gat_finish(L, save, s, a, v);
    HGNN_LAUNCH_CHECK("gat_finish_kernel");
  }
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

// out_masked / csum: nullptr, or the tensors a later backward call wants (see the SAVE kernels)
static hgnn_status gat_forward_impl(const char* who, const hgnn_csr* g, const hgnn_plan* p, int32_t H, int32_t D,
                                    const hgnn_half* U, int64_t ldu, const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l,
                                    const hgnn_half* a_r, float neg_slope, hgnn_half* out, int64_t ldo, float* lse,
                                    hgnn_half* out_masked, int64_t ldom, float* csum, void* stream) {
  clear_error();
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EUNSUPPORTED, "%s: an edge-id map is not supported here", who);
  HGNN_REQUIRE(H >= 1 && D >= 1 && int64_t(H) * D <= 512, HGNN_EINVAL, "%s: H = %d, D = %d out of range", who, H, D);
  const int F = H * D;
  HGNN_REQUIRE(H <= p->max_H && F <= p->max_F, HGNN_EINVAL, "%s: H = %d / F = %d exceed the plan's max_H = %d / max_F = %d",
               who, H, F, p->max_H, p->max_F);
  HGNN_REQUIRE(ldo >= F && ldv >= F && ldu >= F, HGNN_EINVAL, "%s: leading dimension smaller than F", who);
  HGNN_REQUIRE((out_masked == nullptr) == (csum == nullptr), HGNN_EINVAL, "%s: out_masked and csum go together", who);
  HGNN_REQUIRE(out_masked == nullptr || (ldom >= F && neg_slope >= 0.f), HGNN_EINVAL,
               "%s: out_masked needs ldom >= F and a slope >= 0", who);
  HGNN_REQUIRE(g->nrows == 0 || out != nullptr, HGNN_EINVAL, "%s: out is NULL", who);
  if (g->nrows == 0) return HGNN_OK;
  HGNN_REQUIRE(U && Vt && a_l && a_r, HGNN_EINVAL, "%s: U, Vt, a_l or a_r is NULL", who);
  HGNN_REQUIRE(D % 8 == 0 && ldv % 8 == 0 && ldo % 8 == 0 && aligned16(Vt) && aligned16(out), HGNN_EUNSUPPORTED,
               "%s: needs D %% 8 == 0, ld %% 8 == 0 and 16-byte aligned Vt, out", who);
  HGNN_REQUIRE(out_masked == nullptr || (ldom % 8 == 0 && aligned16(out_masked)), HGNN_EUNSUPPORTED,
               "%s: needs ldom %% 8 == 0 and a 16-byte aligned out_masked", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // The row-side score term el[i,h] = a_l[h].U[i,h] is formed where a row's piece begins; over column blocks, which visit
  // every row once per block, it comes from a projection of the vertices into the plan's scratch.  The column-side term is
  // formed in the kernel from the gathered row.
  if (p->nb > 1) st = gat_project(p, g, H, D, U, ldu, nullptr, ldv, a_l, a_r, s, who);
  else st = gat_check(p, H, D, U, ldu, nullptr, ldv, a_l, a_r, who);
  if (st != HGNN_OK) return st;
  GatArgs a{};
  a.col = g->col;
  a.X = reinterpret_cast<const half_t*>(Vt);
  a.Y = reinterpret_cast<half_t*>(out);
  a.ldx = ldv;
  a.ldy = ldo;
  a.nrows = g->nrows;
  a.F = F;
  a.H = H;
  a.D = D;
  a.slope = neg_slope;
  a.el = p->nb > 1 ? p->vscratch : nullptr;
  a.U = reinterpret_cast<const half_t*>(U);
  a.ldu = ldu;
  a.a_l = reinterpret_cast<const half_t*>(a_l);
  a.a_r = reinterpret_cast<const half_t*>(a_r);
  a.lse = lse;
  a.Ym = reinterpret_cast<half_t*>(out_masked);
  a.ldym = ldom;
  a.csum = csum;
  const bool save = out_masked != nullptr;
  if (p->nb <= 1) return run_gat_tasks(p, p->tasks, a, g->ncols, s);
  // column-blocked plan: every block leaves normalised partial rows and their (m, z[, zm/z]) per row; one pass merges them
  p = walked_cut(p, false);
  const size_t V = size_t(p->nrows);
  const size_t flat = size_t(p->nb) * V;
  half_t* bstage = reinterpret_cast<half_t*>(p->bstage);
  half_t* bstage_m = bstage + flat * size_t(p->max_F);    // the plan holds a second set of partial rows behind the first
  float* bsum_c = p->bsum + 2 * flat * size_t(p->max_H);  // and a third scalar per partial row
  const int L = pow2_at_least(F / 8);
  {
    // all blocks in one launch: waves numbered block after block and dispatched in that order
    GatArgs ab = a;
    ab.Y = bstage;
    ab.ldy = p->max_F;
    ab.lse = nullptr;
    ab.part_mz = p->bsum;
    ab.Ym = save ? bstage_m : nullptr;
    ab.ldym = p->max_F;
    ab.csum = save ? bsum_c : nullptr;
    ab.col = p->bcol;
    ab.y_stride = int64_t(V) * p->max_F;
    ab.mz_stride = int64_t(V) * p->max_H * 2;
    ab.c_stride = int64_t(V) * p->max_H;
    st = run_gat_tasks(p, p->btasks, ab, g->ncols, s);
    if (st != HGNN_OK) return st;
  }
  const GatBlockParts parts{bstage, bstage_m, p->max_F, p->bsum, int64_t(V) * p->max_H * 2, bsum_c, int64_t(V) * p->max_H, p->nb};
  launch_gat_block_merge(L, save, dim3(unsigned(ceil_div(g->nrows, int64_t(kWavesPerBlock) * (kWave / L)))), s, a, parts);
  HGNN_LAUNCH_CHECK("gat_block_merge_kernel");
  return HGNN_OK;
}

extern "C" {

hgnn_status hgnn_gat_forward_fused(const hgnn_csr* g, const hgnn_plan* p, int32_t H, int32_t D, const hgnn_half* U,
                                   int64_t ldu, const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l,
                                   const hgnn_half* a_r, float neg_slope, hgnn_half* out, int64_t ldo, float* lse,
                                   void* stream) {
  return gat_forward_impl("hgnn_gat_forward_fused", g, p, H, D, U, ldu, Vt, ldv, a_l, a_r, neg_slope, out, ldo, lse, nullptr, 0,
                          nullptr, stream);
}

hgnn_status hgnn_gat_forward_fused_save(const hgnn_csr* g, const hgnn_plan* p, int32_t H, int32_t D, const hgnn_half* U,
                                        int64_t ldu, const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l,
                                        const hgnn_half* a_r, float neg_slope, hgnn_half* out, int64_t ldo, float* lse,
                                        hgnn_half* out_masked, int64_t ldom, float* csum, void* stream) {
  const char* who = "hgnn_gat_forward_fused_save";
  if (out_masked == nullptr || csum == nullptr || lse == nullptr) {
    clear_error();
    return fail(HGNN_EINVAL, "%s: lse, out_masked and csum are required", who);
  }
  return gat_forward_impl(who, g, p, H, D, U, ldu, Vt, ldv, a_l, a_r, neg_slope, out, ldo, lse, out_masked, ldom, csum, stream);
}

}  // extern "C"

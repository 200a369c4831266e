// Backward of the single-pass GAT aggregation for gfx950, again without any per-edge tensor.
//
// With alpha rebuilt from per-vertex scalars, alpha_ij = exp(LeakyReLU(el_i + er_j) - lse_i), and
// t_i = sum_j alpha_ij * dalpha_ij = <dOut_i, out_i> known per vertex, every per-edge quantity of
// the backward pass (sections 2.1.2 and 3.1.2: SDDMM for dalpha, Eq. 1 differentiated, the
// alpha-weighted SpMM on the transpose) follows from one gathered feature row and a few scalars:
//   dalpha_ij = <dOut_i, h_j>,   ds_ij = alpha_ij * (dalpha_ij - t_i) * LeakyReLU'(el_i + er_j)
// Two passes over the graph, both over row tasks (no atomics, staged pieces, follow-up):
//   transposed pass (rows j, gathers dOut_i):  dV_j = sum_i alpha_ij * dOut_i,  d_er_j = sum_i ds_ij
//   forward pass    (rows i, gathers h_j):     d_el_i = sum_j ds_ij
// The destination vertex's scalars (el, lse, t) sit in one 16-byte entry per (vertex, head), so the
// transposed pass fetches them with a single gather from a table that stays in L2.  Because the sum of ds over
// any piece of a row is linear in the gathered vectors, no dot product is formed per edge: the
// kernels accumulate the mask-weighted vector sum and one scalar, and take the dot product with the
// row-side vector once per piece.
#include "task.h"

namespace hgnn {

struct GatBwdArgs {
  const int* col;
  const half_t* X;     // gathered, column-side vectors [ncols of this graph][ldx]
  const half_t* R;     // row-side vectors [nrows of this graph][ldr]
  half_t* Y;           // VEC kernels: [nrows][ldy] = sum over the row of alpha * X[col]
  int64_t ldx, ldr, ldy;
  int nrows, F, H, D;
  float slope;
  const float4* vtab;  // [destination vertex][H]: (el, lse, t, unused)
  const float* er;     // [source vertex][H]
  half_t* dsum;        // [nrows][H] sum over the row of ds (fp16), or
  float* dsum_f32;     // column blocks: this block's partial sums in fp32
  half_t* staging;     // [slots][stage_ld] pieces of the rows that have several
  float* stage_ds;     // [slots][H] their partial sums of ds
  int stage_ld;
  // column blocks in one launch (waves numbered block after block): Y and dsum_f32 point at block 0's partial results and
  // advance by the strides per block
  int64_t y_stride, ds_stride;
  __device__ __forceinline__ void enter_block(int b) {
    if (Y) Y += int64_t(b) * y_stride;
    if (dsum_f32) dsum_f32 += int64_t(b) * ds_stride;
  }
};

// one finished row: the vector (VEC) and the head's scalar
template <bool VEC>
__device__ __forceinline__ void bwd_row_store(const GatBwdArgs& a, int64_t row, int f0, int head, bool leader,
                                              const float (&acc)[8], float ds) {
  if (VEC) {
    half8_t h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = half_t(acc[i]);
    *reinterpret_cast<half8_t*>(a.Y + row * a.ldy + f0) = h;
  }
  if (leader) {
    if (a.dsum_f32) a.dsum_f32[row * a.H + head] = ds;
    else a.dsum[row * a.H + head] = half_t(ds);
  }
}

template <bool VEC>
__device__ __forceinline__ void bwd_stage_store(const GatBwdArgs& a, int64_t slot, int f0, int head, bool leader,
                                                const float (&acc)[8], float ds) {
  if (VEC) {
    half8_t h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = half_t(acc[i]);
    *reinterpret_cast<half8_t*>(a.staging + slot * a.stage_ld + f0) = h;
  }
  if (leader) a.stage_ds[slot * a.H + head] = ds;
}

// VEC = true is the pass over the transposed graph (the destination vertex of a non-zero is its column).  A wave is laid out as
// in gat_task_kernel.  The weight of a (non-zero, head) and what follows from it are formed once, by the lane that owns the
// pair (HeadTile), from the destination's packed scalars and the source's er -- one of them fetched per non-zero, the
// other constant in a lane group -- and handed to the other lanes of the head with the weight.
//
// The sum of ds over a piece of a row is linear in the gathered vectors:
//   sum_k alpha_k m_k (<r, x_k> - t_k) = <r, sum_k alpha_k m_k x_k> - sum_k alpha_k m_k t_k
// (r = the row-side vector, m = the LeakyReLU slope of the edge), so the loop only accumulates the mask-weighted vector
// wacc beside acc and one scalar; the dot product with r happens once per piece.
//
// Bound: the L2s' requests (two per non-zero: the vector, the packed scalars; 56 % of them hit at 5.5 M non-zeros, 92 % at 114 M in
// blocks) and the vector instructions (busy 69 % and 52 % of the cycles).  The saved backward call against the walk over equal
// runs: 5.5 M non-zeros, 4 heads of 16 166 -> 131 us; 114 M, one head of 64 1.70 -> 1.26 ms.
template <int L, bool NEAR, bool VEC, int RS, int MOST>
__global__ __launch_bounds__(kWave, (VEC ? 5 : 6) - (RS <= 2)) void gat_bwd_task_kernel(GatBwdArgs a, TaskView v, int ncols) {
  constexpr int G = kWave / L;
  typedef Round<L, MOST> Rd;
  typedef HeadTile<RS> Ht;
  __shared__ __align__(16) int s_handles[G * Rd::PITCH];
  __shared__ __align__(16) int s_raw[NEAR ? G * Rd::PITCH : 4];
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int LH = a.D / 8;
  int head = head_of_lane(active ? l : 0, LH);
  if (RS == 8) asm("" : "+v"(head));  // (else the compiler holds what follows from it in registers that it does not have: 12 bytes spilled, 2 to 9 %)
  const bool leader = active && (l & (LH - 1)) == 0;
  const TaskWave w = task_enter<L, Rd::R>(v, blockIdx.x, g);
  a.enter_block(w.block);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // sum alpha * x          (VEC)
  if (w.z1 > w.z0) {
    for (pos_t i = w.z0 + g; i < w.z1; i += G)
      if (active) bwd_row_store<VEC>(a, w.zrow[i], f0, head, leader, acc, 0.f);
    return;
  }
  float wacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // sum alpha * m * x
  float csum = 0.f;                                           // sum alpha * m * t over this lane's edges
  int* const s_hnd = s_handles + g * Rd::PITCH;
  int* const s_col = NEAR ? s_raw + g * Rd::PITCH : s_hnd;  // column ids
  const RowTable<NEAR> table(a.X, ncols, a.ldx, f0c);
  const int row = w.row >= 0 ? w.row : 0;
  const half8_t ur = *reinterpret_cast<const half8_t*>(a.R + int64_t(row) * a.ldr + f0c);  // the row-side vector
  float er_row = 0.f;                                // VEC: the row is the source vertex
  float4 v_row = make_float4(0.f, 0.f, 0.f, 0.f);    // else the destination
  if (VEC) er_row = a.er[int64_t(row) * a.H + head];
  else v_row = a.vtab[int64_t(row) * a.H + head];
  const int own = (lane & (Rd::LC - 1)) * Rd::E;
  const int edge = Ht::own_edge(l);
  for (pos_t k = w.beg; k < w.end; k += w.step) {
    const pos_t end = k + w.span < w.end ? k + w.span : w.end;
    const int n = int(end - k);
    wave_sync();  // the previous round has been read
    {
      const int left = n - own;  // entries of this lane's run
      int c[Rd::E];
      load_cols<Rd::E>(v, a.col, false, w.block, k, own, RunLeft{left}, c);
      if (NEAR) {
#pragma unroll
        for (int m = 0; m < Rd::E; m += 4)
          *reinterpret_cast<int4_t*>(s_col + own + m) = int4_t{c[m], c[m + 1], c[m + 2], c[m + 3]};
      }
#pragma unroll
      for (int m = 0; m < Rd::E; ++m) c[m] = table.handle(c[m], m < left);
#pragma unroll
      for (int m = 0; m < Rd::E; m += 4)
        *reinterpret_cast<int4_t*>(s_hnd + own + m) = int4_t{c[m], c[m + 1], c[m + 2], c[m + 3]};
    }
    wave_sync();
    for (int q = 0; q < n; q += 8) {
      float4 dv[Ht::NS];
      float es[Ht::NS];
      bool in[Ht::NS];
#pragma unroll
      for (int j = 0; j < Ht::NS; ++j) {
        in[j] = q + j * RS + edge < n;
        const int c = in[j] ? s_col[q + j * RS + edge] : 0;
        if (VEC) dv[j] = a.vtab[int64_t(c) * a.H + head];
        else es[j] = a.er[int64_t(c) * a.H + head];
      }
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
      float alpha[Ht::NS], am[Ht::NS];
#pragma unroll
      for (int j = 0; j < Ht::NS; ++j) {
        const float sc = VEC ? dv[j].x + er_row : v_row.x + es[j];
        const float lse = VEC ? dv[j].y : v_row.y, tt = VEC ? dv[j].z : v_row.z;
        alpha[j] = in[j] ? __expf((sc > 0.f ? sc : a.slope * sc) - lse) : 0.f;
        am[j] = sc > 0.f ? alpha[j] : a.slope * alpha[j];
        csum += in[j] ? am[j] * tt : 0.f;
      }
      auto add = [&](auto U) {
        constexpr int u = decltype(U)::value;
        if (VEC) {
          const float wa = Ht::template from_owner<u>(alpha);
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] = fmaf(wa, float(x[u][i]), acc[i]);
        }
        const float wm = Ht::template from_owner<u>(am);
#pragma unroll
        for (int i = 0; i < 8; ++i) wacc[i] = fmaf(wm, float(x[u][i]), wacc[i]);
      };
      add(std::integral_constant<int, 0>{});
      add(std::integral_constant<int, 1>{});
      add(std::integral_constant<int, 2>{});
      add(std::integral_constant<int, 3>{});
      add(std::integral_constant<int, 4>{});
      add(std::integral_constant<int, 5>{});
      add(std::integral_constant<int, 6>{});
      add(std::integral_constant<int, 7>{});
    }
  }
  float d = 0.f;
  if (active) {
#pragma unroll
    for (int i = 0; i < 8; ++i) d = fmaf(wacc[i], float(ur[i]), d);
  }
  float ds = head_sum1(d, LH) - Ht::sum(csum);
  if (w.whole) {
    ds = across_groups_sum<L>(ds);
    if (VEC) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = across_groups_sum<L>(acc[i]);
    }
    if (g) return;
  }
  if (!active || w.row < 0) return;
  if (w.slot < 0) bwd_row_store<VEC>(a, row, f0, head, leader, acc, ds);
  else bwd_stage_store<VEC>(a, w.slot, f0, head, leader, acc, ds);
}

// Follow-up kernel: sums the staged pieces of every row that has several, in order.
template <int L, bool VEC, bool MANY>
__global__ __launch_bounds__(kBlock) void gat_bwd_finish_kernel(GatBwdArgs a, const int4_t* __restrict__ split, int n_split, int per_wave) {
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
  __shared__ float s_sum[kWavesPerBlock][L][9];
  __shared__ int s_n;
  if (MANY) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
  }
  int4_t q = {0, 0, 0, 0};  // row, first slot, pieces, block
  if (g < per_wave && i0 + g < n_split) q = split[i0 + g];
  if (MANY && q[2] > kMany && l == 0) s_row[atomicAdd(&s_n, 1)] = q;
  const int alone = per_wave > 1 ? 8 : 0;  // pieces that a lane group adds by itself
  // adds the pieces first, first + stride, ... < end, four of them in flight at a time
  auto take = [&](float (&acc)[8], float& ds, pos_t first, pos_t end, pos_t stride) {
    for (pos_t k0 = first; k0 < end; k0 += 4 * stride) {
      half8_t o[4];
      float d[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const pos_t k = k0 + u * stride;
        o[u] = half8_t(0);
        d[u] = 0.f;
        if (k < end) {
          if (VEC) o[u] = *reinterpret_cast<const half8_t*>(a.staging + int64_t(k) * a.stage_ld + f0c);
          d[u] = a.stage_ds[int64_t(k) * a.H + head];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (VEC) {
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] += float(o[u][i]);
        }
        ds += d[u];
      }
    }
  };
  if (q[2] > 0 && q[2] <= alone) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float ds = 0.f;
    take(acc, ds, q[1], q[1] + q[2], 1);
    GatBwdArgs b = a;
    b.enter_block(q[3]);
    if (active) bwd_row_store<VEC>(b, q[0], f0, head, leader, acc, ds);
  }
  for (int j = 0; j < per_wave; ++j) {
    const int n = __shfl(q[2], j * L);
    if (n <= alone || (MANY && n > kMany)) continue;
    const int rj = __shfl(q[0], j * L), first = __shfl(q[1], j * L), bj = __shfl(q[3], j * L);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float ds = 0.f;
    take(acc, ds, first + g, first + n, G);
    if (VEC) {
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = across_groups_sum<L>(acc[i]);
    }
    ds = across_groups_sum<L>(ds);
    GatBwdArgs b = a;
    b.enter_block(bj);
    if (g == 0 && active) bwd_row_store<VEC>(b, rj, f0, head, leader, acc, ds);
  }
  if (!MANY) return;
  __syncthreads();
  for (int j = 0; j < s_n; ++j) {  // the rows of many pieces, one after the other (in whatever order), by all waves
    const int4_t r = s_row[j];
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float ds = 0.f;
    take(acc, ds, pos_t(r[1]) + wave * G + g, pos_t(r[1]) + r[2], kWavesPerBlock * G);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const float v = across_groups_sum<L>(i < 8 ? acc[i] : ds);
      if (g == 0) s_sum[wave][l][i] = v;
    }
    __syncthreads();
    if (wave == j % kWavesPerBlock && g == 0 && active) {
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) v += s_sum[w][l][i];
        if (i < 8) acc[i] = v;
        else ds = v;
      }
      GatBwdArgs b = a;
      b.enter_block(r[3]);
      bwd_row_store<VEC>(b, r[0], f0, head, leader, acc, ds);
    }
    __syncthreads();
  }
}

// Column-blocked plans: adds the nb partial rows (fp16 vectors, fp32 ds sums) of every row.
template <int L, bool VEC>
__global__ __launch_bounds__(kBlock) void gat_bwd_block_sum_kernel(GatBwdArgs a, const half_t* __restrict__ part,
                                                                   int part_ld, const float* __restrict__ part_ds,
                                                                   int64_t ds_stride, int nb) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const int64_t r = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  if (r >= a.nrows || f0 >= a.F) return;
  const int LH = a.D / 8, head = head_of_lane(l, LH);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float ds = 0.f;
  for (int b = 0; b < nb; ++b) {
    if (VEC) {
      const half8_t o = *reinterpret_cast<const half8_t*>(part + (int64_t(b) * a.nrows + r) * part_ld + f0);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += float(o[i]);
    }
    ds += part_ds[b * ds_stride + r * a.H + head];
  }
  bwd_row_store<VEC>(a, r, f0, head, (l & (LH - 1)) == 0, acc, ds);
}

// Everything the passes need of single vertices, in one launch: er[j,h] = a_r[h].Vt[j,h] for every source vertex, and for every
// destination vertex vtab[i,h] = (a_l[h].U[i,h], lse[i,h], t[i,h] = <dOut[i,h], out[i,h]>, 0).  With the masked result and
// weight sum that the saving forward pass left (outm, csum), the gradient of the row-side score term is a per-vertex
// expression and is written here: d_el[i,h] = <dOut[i,h], outm[i,h]> - t[i,h] * csum[i,h].
struct VertexArgs {
  const half_t *U, *Vt, *a_l, *a_r, *dOut, *out, *outm;  // outm, csum, d_el: nullptr without the saved tensors
  int64_t ldu, ldv, lddo, ldo, ldom;
  const float *lse, *csum;
  int nrows, ncols, F, D, H;
  float4* vtab;
  float* er;
  half_t* d_el;
};

template <int L>
__global__ __launch_bounds__(kBlock) void gat_vtab_kernel(VertexArgs a) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int LH = a.D / 8;
  const int64_t v = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  auto load = [&](const half_t* p, int64_t ld) { return *reinterpret_cast<const half8_t*>(p + v * ld + f0c); };
  const bool dst = active && v < a.nrows, src = active && v < a.ncols;
  float el = 0.f, er = 0.f, p = 0.f, pm = 0.f;
  if (dst) {
    const half8_t x = load(a.dOut, a.lddo);
    el = dot8(*reinterpret_cast<const half8_t*>(a.a_l + f0c), load(a.U, a.ldu));
    p = dot8(x, load(a.out, a.ldo));
    if (a.outm) pm = dot8(x, load(a.outm, a.ldom));
  }
  if (src) er = dot8(*reinterpret_cast<const half8_t*>(a.a_r + f0c), load(a.Vt, a.ldv));
  el = head_sum1(el, LH);
  er = head_sum1(er, LH);
  p = head_sum1(p, LH);
  if (a.outm) pm = head_sum1(pm, LH);
  if ((l & (LH - 1)) == 0) {
    const int64_t k = v * a.H + head_of_lane(l, LH);
    if (src) a.er[k] = er;
    if (dst) {
      a.vtab[k] = make_float4(el, a.lse[k], p, 0.f);
      if (a.outm) a.d_el[k] = half_t(pm - p * a.csum[k]);
    }
  }
}

template <int L, bool NEAR, bool VEC>
static void launch_bwd_tasks_l(int lh, unsigned waves, hipStream_t s, const GatBwdArgs& a, const TaskView& v, int ncols) {
  with_round<L, NEAR>(v, [&](auto most) {
    constexpr int M = decltype(most)::value;
    if (lh == 1) gat_bwd_task_kernel<L, NEAR, VEC, 1, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else if (lh == 2) gat_bwd_task_kernel<L, NEAR, VEC, L < 2 ? L : 2, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else if (lh == 4) gat_bwd_task_kernel<L, NEAR, VEC, L < 4 ? L : 4, M><<<waves, kWave, 0, s>>>(a, v, ncols);
    else gat_bwd_task_kernel<L, NEAR, VEC, L < 8 ? L : 8, M><<<waves, kWave, 0, s>>>(a, v, ncols);
  });
}

template <bool NEAR, bool VEC>
static void launch_bwd_tasks(int L, int lh, unsigned waves, hipStream_t s, const GatBwdArgs& a, const TaskView& v, int ncols) {
  switch (L) {
    case 1: launch_bwd_tasks_l<1, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    case 2: launch_bwd_tasks_l<2, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    case 4: launch_bwd_tasks_l<4, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    case 8: launch_bwd_tasks_l<8, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    case 16: launch_bwd_tasks_l<16, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    case 32: launch_bwd_tasks_l<32, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
    default: launch_bwd_tasks_l<64, NEAR, VEC>(lh, waves, s, a, v, ncols); break;
  }
}

template <int L, bool VEC>
static void launch_bwd_finish_l(dim3 grid, int per_wave, hipStream_t s, const GatBwdArgs& a, const TaskView& v) {
  if (many_pieces(v, kWave / L)) gat_bwd_finish_kernel<L, VEC, true><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
  else gat_bwd_finish_kernel<L, VEC, false><<<grid, kBlock, 0, s>>>(a, v.split, v.n_split, per_wave);
}

template <bool VEC>
static void launch_bwd_finish(int L, hipStream_t s, const GatBwdArgs& a, const TaskView& v) {
  const int per_wave = finish_rows_per_wave(v.n_split, v.n_slots, kWave / L);
  const dim3 grid(unsigned(ceil_div(v.n_split, int64_t(kWavesPerBlock) * per_wave)));
  switch (L) {
    case 1: launch_bwd_finish_l<1, VEC>(grid, per_wave, s, a, v); break;
    case 2: launch_bwd_finish_l<2, VEC>(grid, per_wave, s, a, v); break;
    case 4: launch_bwd_finish_l<4, VEC>(grid, per_wave, s, a, v); break;
    case 8: launch_bwd_finish_l<8, VEC>(grid, per_wave, s, a, v); break;
    case 16: launch_bwd_finish_l<16, VEC>(grid, per_wave, s, a, v); break;
    case 32: launch_bwd_finish_l<32, VEC>(grid, per_wave, s, a, v); break;
    default: launch_bwd_finish_l<64, VEC>(grid, per_wave, s, a, v); break;
  }
}

template <bool VEC>
static void launch_bwd_block_sum(int L, dim3 grid, hipStream_t s, const GatBwdArgs& a, const half_t* part, int part_ld,
                                 const float* part_ds, int64_t ds_stride, int nb) {
  switch (L) {
    case 1: gat_bwd_block_sum_kernel<1, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    case 2: gat_bwd_block_sum_kernel<2, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    case 4: gat_bwd_block_sum_kernel<4, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    case 8: gat_bwd_block_sum_kernel<8, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    case 16: gat_bwd_block_sum_kernel<16, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    case 32: gat_bwd_block_sum_kernel<32, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
    default: gat_bwd_block_sum_kernel<64, VEC><<<grid, kBlock, 0, s>>>(a, part, part_ld, part_ds, ds_stride, nb); break;
  }
}

static void launch_vtab(int L, dim3 grid, hipStream_t s, const VertexArgs& a) {
  switch (L) {
    case 1: gat_vtab_kernel<1><<<grid, kBlock, 0, s>>>(a); break;
    case 2: gat_vtab_kernel<2><<<grid, kBlock, 0, s>>>(a); break;
    case 4: gat_vtab_kernel<4><<<grid, kBlock, 0, s>>>(a); break;
    case 8: gat_vtab_kernel<8><<<grid, kBlock, 0, s>>>(a); break;
    case 16: gat_vtab_kernel<16><<<grid, kBlock, 0, s>>>(a); break;
    case 32: gat_vtab_kernel<32><<<grid, kBlock, 0, s>>>(a); break;
    default: gat_vtab_kernel<64><<<grid, kBlock, 0, s>>>(a); break;
  }
}

// one pass (row tasks t of plan q, follow-up)
template <bool VEC>
static hgnn_status run_bwd_tasks(const hgnn_plan* q, const hgnn_row_tasks* t, GatBwdArgs a, int ncols, hipStream_t s) {
  a.staging = reinterpret_cast<half_t*>(t->staging);
  a.stage_ds = t->stage_mz;
  a.stage_ld = q->max_F;
  const int L = pow2_at_least(a.F / 8), lh = a.D / 8;
  TaskView v = task_view(t, kWave / L, at_ranges(t, kRangesAttention, int64_t(ncols) * a.F * 2, q->l2_bytes), comes_back(false, int64_t(ncols) * a.ldx * 2, q->llc_bytes));
  v.longer = long_rounds(t->nb, q->nrows, t->nnz, q->S, kWave / L, 8);
  const int waves = v.first_wave[t->nb];
  if (waves > 0) {
    if (near_table(ncols, a.ldx)) launch_bwd_tasks<true, VEC>(L, lh, unsigned(waves), s, a, v, ncols);
    else launch_bwd_tasks<false, VEC>(L, lh, unsigned(waves), s, a, v, ncols);
    HGNN_LAUNCH_CHECK("gat_bwd_task_kernel");
  }
  if (v.n_split > 0) {
    launch_bwd_finish<VEC>(L, s, a, v);
    HGNN_LAUNCH_CHECK("gat_bwd_finish_kernel");
  }
  return HGNN_OK;
}

// a pass over graph gg with plan q (column-blocked or not)
template <bool VEC>
static hgnn_status run_bwd_pass(const hgnn_plan* q, const hgnn_csr* gg, GatBwdArgs a, hipStream_t s) {
  if (q->nb <= 1) return run_bwd_tasks<VEC>(q, q->tasks, a, gg->ncols, s);
  q = walked_cut(q, false);
  const size_t V = size_t(q->nrows);
  const int64_t ds_stride = int64_t(V) * q->max_H * 2;
  const int L = pow2_at_least(a.F / 8);
  {
    // all blocks in one launch: waves numbered block after block and dispatched in that order
    GatBwdArgs ab = a;
    ab.col = q->bcol;
    ab.Y = reinterpret_cast<half_t*>(q->bstage);
    ab.ldy = q->max_F;
    ab.dsum = nullptr;
    ab.dsum_f32 = q->bsum;
    ab.y_stride = int64_t(V) * q->max_F;
    ab.ds_stride = ds_stride;
    const hgnn_status st = run_bwd_tasks<VEC>(q, q->btasks, ab, gg->ncols, s);
    if (st != HGNN_OK) return st;
  }
  launch_bwd_block_sum<VEC>(L, dim3(unsigned(ceil_div(gg->nrows, int64_t(kWavesPerBlock) * (kWave / L)))), s, a,
                            reinterpret_cast<const half_t*>(q->bstage), q->max_F, q->bsum, ds_stride, q->nb);
  HGNN_LAUNCH_CHECK("gat_bwd_block_sum_kernel");
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

// out_masked / csum: what hgnn_gat_forward_fused_save left (then d_el is a per-vertex expression and the pass over g
// is not needed), or nullptr
static hgnn_status gat_backward_impl(const char* who, const hgnn_csr* g, const hgnn_plan* p, const hgnn_csr* gt,
                                     const hgnn_plan* pt, int32_t H, int32_t D, const hgnn_half* U, int64_t ldu,
                                     const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l, const hgnn_half* a_r,
                                     float neg_slope, const hgnn_half* out, int64_t ldo, const float* lse,
                                     const hgnn_half* out_masked, int64_t ldom, const float* csum, const hgnn_half* dOut,
                                     int64_t lddo, hgnn_half* dV, int64_t lddv, hgnn_half* d_el, hgnn_half* d_er,
                                     void* stream) {
  clear_error();
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  st = check_csr_args(gt, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr && pt != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: plan p was built for another graph than g", who);
  HGNN_REQUIRE(pt->nrows == gt->nrows && pt->ncols == gt->ncols && pt->nnz == gt->nnz, HGNN_EINVAL,
               "%s: plan pt was built for another graph than gt", who);
  HGNN_REQUIRE(gt->nrows == g->ncols && gt->ncols == g->nrows && gt->nnz == g->nnz, HGNN_EINVAL,
               "%s: gt is not the transpose of g", who);
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EUNSUPPORTED, "%s: g must not carry an edge-id map", who);
  HGNN_REQUIRE(H >= 1 && D >= 1 && int64_t(H) * D <= 512, HGNN_EINVAL, "%s: H = %d, D = %d out of range", who, H, D);
  const int F = H * D;
  HGNN_REQUIRE(H <= p->max_H && F <= p->max_F && H <= pt->max_H && F <= pt->max_F, HGNN_EINVAL,
               "%s: H = %d / F = %d exceed a plan's max_H / max_F", who, H, F);
  HGNN_REQUIRE(ldu >= F && ldv >= F && ldo >= F && lddo >= F && lddv >= F, HGNN_EINVAL,
               "%s: leading dimension smaller than F", who);
  if (g->nrows == 0 && g->ncols == 0) return HGNN_OK;
  HGNN_REQUIRE(U && Vt && a_l && a_r && out && lse && dOut && dV && d_el && d_er, HGNN_EINVAL, "%s: NULL argument", who);
  HGNN_REQUIRE(ldo % 8 == 0 && lddo % 8 == 0 && lddv % 8 == 0 && aligned16(out) && aligned16(dOut) && aligned16(dV),
               HGNN_EUNSUPPORTED, "%s: needs ld %% 8 == 0 and 16-byte aligned out, dOut, dV", who);
  const bool saved = out_masked != nullptr;
  HGNN_REQUIRE(!saved || (csum != nullptr && ldom >= F), HGNN_EINVAL, "%s: out_masked needs csum and ldom >= F", who);
  HGNN_REQUIRE(!saved || (ldom % 8 == 0 && aligned16(out_masked)), HGNN_EUNSUPPORTED,
               "%s: needs ldom %% 8 == 0 and a 16-byte aligned out_masked", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // per-vertex scalars in plan p's scratch: er, and (el, lse, t) packed per destination vertex
  st = gat_check(p, H, D, U, ldu, Vt, ldv, a_l, a_r, who);
  if (st != HGNN_OK) return st;
  const int L = pow2_at_least(F / 8), G = kWave / L;
  float* er = p->vscratch + size_t(g->nrows) * H;
  float4* vtab = reinterpret_cast<float4*>(p->vtab);
  {
    VertexArgs q{};
    auto h = [](const hgnn_half* x) { return reinterpret_cast<const half_t*>(x); };
    q.U = h(U), q.Vt = h(Vt), q.a_l = h(a_l), q.a_r = h(a_r), q.dOut = h(dOut), q.out = h(out), q.outm = h(out_masked);
    q.ldu = ldu, q.ldv = ldv, q.lddo = lddo, q.ldo = ldo, q.ldom = ldom;
    q.lse = lse, q.csum = csum;
    q.nrows = g->nrows, q.ncols = g->ncols, q.F = F, q.D = D, q.H = H;
    q.vtab = vtab, q.er = er, q.d_el = reinterpret_cast<half_t*>(d_el);
    const int nv = g->nrows > g->ncols ? g->nrows : g->ncols;
    launch_vtab(L, dim3(unsigned(ceil_div(nv, int64_t(kWavesPerBlock) * G))), s, q);
    HGNN_LAUNCH_CHECK("gat_vtab_kernel");
  }
  GatBwdArgs a{};
  a.F = F;
  a.H = H;
  a.D = D;
  a.slope = neg_slope;
  a.vtab = vtab;
  a.er = er;
  // transposed pass: rows j (sources), gathers dOut_i; dV_j and d_er_j
  if (gt->nrows > 0) {
    GatBwdArgs t = a;
    t.col = gt->col;
    t.nrows = gt->nrows;
    t.X = reinterpret_cast<const half_t*>(dOut);
    t.ldx = lddo;
    t.R = reinterpret_cast<const half_t*>(Vt);
    t.ldr = ldv;
    t.Y = reinterpret_cast<half_t*>(dV);
    t.ldy = lddv;
    t.dsum = reinterpret_cast<half_t*>(d_er);
    st = run_bwd_pass<true>(pt, gt, t, s);
    if (st != HGNN_OK) return st;
  }
  // forward pass: rows i (destinations), gathers h_j; d_el_i only (already written above from the saved tensors)
  if (g->nrows > 0 && !saved) {
    GatBwdArgs f = a;
    f.col = g->col;
    f.nrows = g->nrows;
    f.X = reinterpret_cast<const half_t*>(Vt);
    f.ldx = ldv;
    f.R = reinterpret_cast<const half_t*>(dOut);
    f.ldr = lddo;
    f.dsum = reinterpret_cast<half_t*>(d_el);
    st = run_bwd_pass<false>(p, g, f, s);
    if (st != HGNN_OK) return st;
  }
  return HGNN_OK;
}

extern "C" hgnn_status hgnn_gat_backward_fused(const hgnn_csr* g, const hgnn_plan* p, const hgnn_csr* gt,
                                               const hgnn_plan* pt, int32_t H, int32_t D, const hgnn_half* U, int64_t ldu,
                                               const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l, const hgnn_half* a_r,
                                               float neg_slope, const hgnn_half* out, int64_t ldo, const float* lse,
                                               const hgnn_half* dOut, int64_t lddo, hgnn_half* dV, int64_t lddv,
                                               hgnn_half* d_el, hgnn_half* d_er, void* stream) {
  return gat_backward_impl("hgnn_gat_backward_fused", g, p, gt, pt, H, D, U, ldu, Vt, ldv, a_l, a_r, neg_slope, out, ldo, lse,
                           nullptr, 0, nullptr, dOut, lddo, dV, lddv, d_el, d_er, stream);
}

extern "C" hgnn_status hgnn_gat_backward_fused_saved(const hgnn_csr* g, const hgnn_plan* p, const hgnn_csr* gt,
                                                     const hgnn_plan* pt, int32_t H, int32_t D, const hgnn_half* U,
                                                     int64_t ldu, const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l,
                                                     const hgnn_half* a_r, float neg_slope, const hgnn_half* out, int64_t ldo,
                                                     const float* lse, const hgnn_half* out_masked, int64_t ldom,
                                                     const float* csum, const hgnn_half* dOut, int64_t lddo, hgnn_half* dV,
                                                     int64_t lddv, hgnn_half* d_el, hgnn_half* d_er, void* stream) {
  const char* who = "hgnn_gat_backward_fused_saved";
  if (out_masked == nullptr || csum == nullptr) {
    clear_error();
    return fail(HGNN_EINVAL, "%s: out_masked and csum are required", who);
  }
  return gat_backward_impl(who, g, p, gt, pt, H, D, U, ldu, Vt, ldv, a_l, a_r, neg_slope, out, ldo, lse, out_masked, ldom, csum,
                           dOut, lddo, dV, lddv, d_el, d_er, stream);
}

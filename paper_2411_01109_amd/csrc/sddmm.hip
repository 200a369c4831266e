// fp16 SDDMM for gfx950 (paper sections 2.1.2 and 5.1): per non-zero, a reduction along the
// feature dimension of the row vertex's and the column vertex's vectors.
//
// Over a plan's row tasks a lane group stays inside one row: that row's vector is in registers, every lane loads 16 bytes (8
// halves) of the column vertices' rows -- the wide per-lane load of section 5.1.3 -- eight non-zeros at a time, and the
// eight partial dot products are summed by halves across the lanes of a head.  Results are collected in LDS and written
// back coalesced.  The vector-width study of section 6.3.1 runs the same kernel with 4 or 2 halves per lane and load.
#include "task.h"

namespace hgnn {

struct SddmmArgs {
  const int* rowptr;
  const int* col;
  const int* erow;  // COO row ids from the caller, or nullptr (then the row is searched in rowptr)
  const int* seg_lo;
  const int* seg_hi;
  const half_t* U;
  const half_t* Vt;
  const half_t* a_l;
  const half_t* a_r;
  half_t* out;
  const float* lse;  // [nrows][H] or nullptr; when set the edge score kernel writes exp(score - lse[row]) = alpha
  float* el;  // [nrows][H] fp32 scratch (factorised GAT score)
  float* er;  // [ncols][H]
  int64_t ldu, ldv, nnz, nseg;
  int nrows, ncols;
  int H, D, F, S;
  float slope;
  const int* delta;  // column blocks: slot = position in the block + delta[block][row], else nullptr: slot = position
};

constexpr int kTile = 256;  // non-zeros per wave in the kernels that run without a plan

// DOT over row tasks: out[k,h] = <U[row, h], Vt[col k, h]>.  MASK: one head whose length is not a multiple of 8 -- the group's
// lanes cover the padded row pitch and the elements past D are forced to zero on both operands (whatever the padding
// columns hold).  VW = halves per lane and load: 8, or 4 / 2 for the vector-width study (a row then takes more lanes, a wave holds
// fewer rows).  RS = min(lanes per head, 8).  Bound: the gathers (a row of 128 bytes is one request to the L2s).  Against
// the walk over equal runs of non-zeros, whose row changes took most of its steps through a slow path: 114 M non-zeros, one
// head of 64 in blocks: 1.06 -> 0.92 ms; 5.5 M, four heads of 16: the same (58 us); on power-law graphs of 20 to 31 M, where the
// gathers miss the L2s and the results of a row no longer fill lines with their neighbours', 1 to 6 % slower (31 M: one head of
// 64 338 -> 350 us, four of 16 391 -> 393).
// Rows of 32 bytes keep to five waves a SIMD: with six, which their registers allow, tables beyond an L2 are fetched more often: uniform, 200 000 vertices, 1 M
// non-zeros 17.4 / 19.6 us, 2.4 M 31.6 / 35.9 (power law, where most gathers hit, 26.3 / 25.8).
template <int L, bool NEAR, bool MASK, int RS, int VW, int MOST>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(RS <= 2 ? 5 : 6, NEAR && !MASK && L == 2 && RS == 2 && VW == 8 ? 5 : 8))) void sddmm_task_kernel(SddmmArgs a, TaskView v) {
  constexpr int G = kWave / L;
  typedef _Float16 hv_t __attribute__((ext_vector_type(VW)));
  typedef Round<L, MOST> Rd;
  typedef HeadTile<RS> Ht;
  __shared__ __align__(16) int s_handles[G * Rd::PITCH];
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const int g = lane / L, l = lane % L;
  const int f0 = VW * l;
  const bool active = f0 < a.F;
  const int f0c = active ? f0 : 0;
  const int LH = MASK ? L : a.D / VW;       // lanes per head (power of two)
  const int head = MASK ? 0 : head_of_lane(active ? l : 0, LH);
  const int nvalid = active ? a.F - f0 : 0; // MASK: elements of this lane's vector that exist
  auto masked = [&](hv_t x) -> hv_t {
    if (MASK) {
#pragma unroll
      for (int i = 0; i < VW; ++i) x[i] = i < nvalid ? x[i] : half_t(0);
    }
    return x;
  };
  auto dot_of = [](const hv_t& p, const hv_t& q) -> float {
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < VW; ++i) d = fmaf(float(p[i]), float(q[i]), d);
    return d;
  };
  const TaskWave w = task_enter<L, Rd::R>(v, blockIdx.x, g);
  int* const s_hnd = s_handles + g * Rd::PITCH;
  half_t* const s_out = reinterpret_cast<half_t*>(smem) + g * (Rd::R * a.H);  // [G][R * H]
  const RowTable<NEAR> table(a.Vt, a.ncols, a.ldv, f0c);
  const int row = w.row >= 0 ? w.row : 0;
  const hv_t ur = masked(*reinterpret_cast<const hv_t*>(a.U + int64_t(row) * a.ldu + f0c));
  const int64_t shift = a.delta ? int64_t(a.delta[int64_t(w.block) * a.nrows + row]) - w.first : 0;
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
      hv_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = table.template row<VW>(h8[u]);
      float d[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) d[u] = dot_of(ur, masked(x[u]));
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
      if (MASK || active) {
#pragma unroll
        for (int j = 0; j < Ht::NS; ++j) s_out[(q + j * RS + edge) * a.H + head] = half_t(s[j]);
      }
    }
    wave_sync();
    const int nout = n * a.H;
    half_t* dst = a.out + (int64_t(k) + shift) * a.H;
    for (int j = 4 * l; j < nout; j += 4 * L) {
      if (j + 4 <= nout) {
        __builtin_memcpy(dst + j, __builtin_assume_aligned(s_out + j, 8), 8);
      } else {
        for (int i = j; i < nout; ++i) dst[i] = s_out[i];
      }
    }
  }
}

// Without a plan: tiles of kTile non-zeros, row ids from the caller's COO array.
// SCORE = false: out = <U[i,h], Vt[j,h]>.  SCORE = true: out = LeakyReLU(<a_l[h],U[i,h]> + <a_r[h],Vt[j,h]>).
template <int L, bool SCORE>
__global__ __launch_bounds__(kBlock) void sddmm_edge_kernel(SddmmArgs a) {
  constexpr int G = kWave / L;
  constexpr int C = kTile / G;  // consecutive non-zeros per group
  constexpr int U_ = 4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < a.F;
  const int LH = a.D / 8;  // lanes per head (power of two)
  const int head = active ? l / LH : 0;
  half_t* s_out = reinterpret_cast<half_t*>(smem) + size_t(wave) * kTile * a.H;
  const int64_t e0 = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * kTile;
  const int n = e0 < a.nnz ? int(a.nnz - e0 < kTile ? a.nnz - e0 : kTile) : 0;
  half8_t al = half8_t(0), ar = half8_t(0);
  if (SCORE && active) {
    al = *reinterpret_cast<const half8_t*>(a.a_l + f0);
    ar = *reinterpret_cast<const half8_t*>(a.a_r + f0);
  }
  const int c0 = g * C < n ? g * C : n;
  const int c1 = c0 + C < n ? c0 + C : n;
  for (int i = c0; i < c1; i += U_) {
    half8_t u[U_], v[U_];
#pragma unroll
    for (int q = 0; q < U_; ++q) {
      u[q] = half8_t(0);
      v[q] = half8_t(0);
      if (i + q < c1 && active) {
        const int64_t k = e0 + i + q;
        const int r = a.erow ? a.erow[k] : row_of_edge(a.rowptr, a.nrows, k);
        u[q] = *reinterpret_cast<const half8_t*>(a.U + int64_t(r) * a.ldu + f0);
        v[q] = *reinterpret_cast<const half8_t*>(a.Vt + int64_t(a.col[k]) * a.ldv + f0);
      }
    }
#pragma unroll
    for (int q = 0; q < U_; ++q) {
      float p = SCORE ? dot8(al, u[q]) + dot8(ar, v[q]) : dot8(u[q], v[q]);
      for (int off = 1; off < LH; off <<= 1) p += __shfl_xor(p, off);
      if (SCORE) p = p > 0.f ? p : a.slope * p;
      if (i + q < c1 && active && (l % LH) == 0) s_out[(i + q) * a.H + head] = half_t(p);
    }
  }
  wave_sync();
  for (int j = lane; j < n * a.H; j += kWave) a.out[e0 * a.H + j] = s_out[j];
}

// Scalar path: one thread per (non-zero, head).
template <bool SCORE>
__global__ __launch_bounds__(kBlock) void sddmm_scalar_kernel(SddmmArgs a) {
  const int64_t idx = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= a.nnz * a.H) return;
  const int64_t k = idx / a.H;
  const int h = int(idx % a.H);
  const int r = a.erow ? a.erow[k] : row_of_edge(a.rowptr, a.nrows, k);
  const half_t* u = a.U + int64_t(r) * a.ldu + h * a.D;
  const half_t* v = a.Vt + int64_t(a.col[k]) * a.ldv + h * a.D;
  float p = 0.f;
  if (SCORE) {
    for (int d = 0; d < a.D; ++d) p = fmaf(float(a.a_l[h * a.D + d]), float(u[d]), p);
    for (int d = 0; d < a.D; ++d) p = fmaf(float(a.a_r[h * a.D + d]), float(v[d]), p);
    p = p > 0.f ? p : a.slope * p;
  } else {
    for (int d = 0; d < a.D; ++d) p = fmaf(float(u[d]), float(v[d]), p);
  }
  a.out[idx] = half_t(p);
}

// Factorised GAT score, step 1: proj[v,h] = <avec[h], feat[v,h]> for every vertex, fp32, on both sides (one launch: where
// they are the same features a row comes from memory once, 262 144 rows of 64 halves 8.6 + 8.6 -> 11.5 us).
struct ProjSide {
  const half_t* feat;
  int64_t ld;
  int nv;  // 0: this side is not wanted
  const half_t* avec;
  float* proj;
};

template <int L>
__global__ __launch_bounds__(kBlock) void vertex_proj_kernel(ProjSide u, ProjSide w, int F, int D, int H) {
  constexpr int G = kWave / L;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int g = lane / L, l = lane % L;
  const int f0 = 8 * l;
  const bool active = f0 < F;
  const int LH = D / 8;
  const int64_t v = (int64_t(blockIdx.x) * kWavesPerBlock + wave) * G + g;
  const bool inu = active && v < u.nv, inw = active && v < w.nv;
  float p = 0.f, q = 0.f;
  if (inu) p = dot8(*reinterpret_cast<const half8_t*>(u.avec + f0), *reinterpret_cast<const half8_t*>(u.feat + v * u.ld + f0));
  if (inw) q = dot8(*reinterpret_cast<const half8_t*>(w.avec + f0), *reinterpret_cast<const half8_t*>(w.feat + v * w.ld + f0));
  for (int off = 1; off < LH; off <<= 1) {
    p += __shfl_xor(p, off);
    q += __shfl_xor(q, off);
  }
  if ((l & (LH - 1)) != 0) return;
  const int head = head_of_lane(l, LH);
  if (inu) u.proj[v * H + head] = p;
  if (inw) w.proj[v * H + head] = q;
}

// step 2, one plan segment per wave: e[k,h] = LeakyReLU(el[row k, h] + er[col k, h]); row ids
// come from the offset array (staged in LDS), so the only per-edge stream read is the column id.  Bound by the chain ids ->
// er and offsets -> rows -> el: the ids and er of 256 non-zeros go out before the rows are staged, el of all of them together
// (one step of a wave after the other, behind the rows: 5.5 M non-zeros x 4 heads 43.9 us, now 41.0; the lines of er at 3.6 clocks each
// in a compute unit are 32).
template <int HT>
__global__ __launch_bounds__(kBlock) void edge_score_seg_kernel(SddmmArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int S = a.S;
  const int per = seg_slots_per_lane(S), spad = kWave * per;
  int* s_row = reinterpret_cast<int*>(smem) + size_t(wave) * spad;
  const int64_t seg = int64_t(blockIdx.x) * kWavesPerBlock + wave;
  if (seg >= a.nseg) return;
  const int64_t e0 = seg * S;
  const int n = int(a.nnz - e0 < S ? a.nnz - e0 : S);
  const int row_lo = a.seg_lo[seg], row_hi = a.seg_hi[seg];
  if (HT == 0) {  // any head count: one output element per lane and step
    seg_stage_rows(s_row, lane, per, row_lo, row_hi, a.rowptr, e0, [] {});
    const int tot = n * a.H;
    for (int j = lane; j < tot; j += kWave) {
      const int k = j / a.H, h = j - k * a.H;
      float s = a.el[int64_t(s_row[k]) * a.H + h] + a.er[int64_t(a.col[e0 + k]) * a.H + h];
      s = s > 0.f ? s : a.slope * s;
      if (a.lse) s = __expf(s - a.lse[int64_t(s_row[k]) * a.H + h]);
      a.out[e0 * a.H + j] = half_t(s);
    }
    return;
  }
  // H in {1,2,4,8}: a lane produces 8 consecutive outputs (8/H non-zeros) and stores them as 16 bytes, IT times over
  constexpr int H = HT > 0 ? HT : 1;
  constexpr int EPL = 8 / H, STEP = kWave * EPL, IT = STEP < 256 ? 256 / STEP : 1;
  typedef float fv_t __attribute__((ext_vector_type(H)));
  typedef int iv_t __attribute__((ext_vector_type(EPL < 4 ? EPL : 4)));
  constexpr int W = EPL < 4 ? EPL : 4;  // ids a load
  const int* const ids = a.col + e0;
  half_t* dst = a.out + e0 * H;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(dst) & 15u) == 0, ids_ok = (reinterpret_cast<uintptr_t>(ids) & 15u) == 0;
  for (int k0 = 0; k0 < n; k0 += IT * STEP) {
    fv_t vr[IT * EPL];
    auto right = [&] {
      int cols[IT * EPL];
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int kb = k0 + i * STEP + lane * EPL;
        if (ids_ok && kb + EPL <= n) {
#pragma unroll
          for (int v = 0; v < EPL / W; ++v) {
            const iv_t c = *reinterpret_cast<const iv_t*>(ids + kb + W * v);
#pragma unroll
            for (int q = 0; q < W; ++q) cols[i * EPL + W * v + q] = c[q];
          }
        } else {
#pragma unroll
          for (int e = 0; e < EPL; ++e) cols[i * EPL + e] = ids[kb + e < n ? kb + e : n - 1];
        }
      }
#pragma unroll
      for (int e = 0; e < IT * EPL; ++e) vr[e] = *reinterpret_cast<const fv_t*>(a.er + int64_t(cols[e]) * H);
    };
    if (k0 == 0) seg_stage_rows(s_row, lane, per, row_lo, row_hi, a.rowptr, e0, right);
    else right();
    int rows[IT * EPL];
    fv_t vl[IT * EPL];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const int k = k0 + i * STEP + lane * EPL + e;
        rows[i * EPL + e] = s_row[k < n ? k : n - 1];
      }
    }
#pragma unroll
    for (int e = 0; e < IT * EPL; ++e) vl[e] = *reinterpret_cast<const fv_t*>(a.el + int64_t(rows[e]) * H);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int kb = k0 + i * STEP + lane * EPL;
      half8_t o = half8_t(0);
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
          float s = vl[i * EPL + e][h] + vr[i * EPL + e][h];
          s = s > 0.f ? s : a.slope * s;
          if (a.lse) s = __expf(s - a.lse[int64_t(rows[i * EPL + e]) * H + h]);
          o[e * H + h] = half_t(s);
        }
      }
      if (vec_ok && kb + EPL <= n) {
        *reinterpret_cast<half8_t*>(dst + kb * H) = o;
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (kb * H + q < n * H) dst[kb * H + q] = o[q];
      }
    }
  }
}

template <bool SCORE>
static void launch_edge(int L, dim3 grid, size_t lds, hipStream_t s, const SddmmArgs& a) {
  switch (L) {
    case 1: sddmm_edge_kernel<1, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    case 2: sddmm_edge_kernel<2, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    case 4: sddmm_edge_kernel<4, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    case 8: sddmm_edge_kernel<8, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    case 16: sddmm_edge_kernel<16, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    case 32: sddmm_edge_kernel<32, SCORE><<<grid, kBlock, lds, s>>>(a); break;
    default: sddmm_edge_kernel<64, SCORE><<<grid, kBlock, lds, s>>>(a); break;
  }
}

template <int L, bool NEAR, int VW>
static void launch_dot_tasks_l(int lh, bool mask, unsigned waves, hipStream_t s, const SddmmArgs& a, const TaskView& v) {
  with_round<L, NEAR && VW == 8>(v, [&](auto most) {
    constexpr int M = decltype(most)::value;
    const size_t lds = size_t(kWave / L) * size_t(Round<L, M>::R) * size_t(a.H) * sizeof(half_t);  // results
    if constexpr (VW == 8) {
      if (mask) {
        sddmm_task_kernel<L, NEAR, true, L < 8 ? L : 8, VW, M><<<waves, kWave, lds, s>>>(a, v);
        return;
      }
      if (lh == 1) {
        sddmm_task_kernel<L, NEAR, false, 1, VW, M><<<waves, kWave, lds, s>>>(a, v);
        return;
      }
    }
    if (lh == 2) sddmm_task_kernel<L, NEAR, false, L < 2 ? L : 2, VW, M><<<waves, kWave, lds, s>>>(a, v);
    else if (lh == 4) sddmm_task_kernel<L, NEAR, false, L < 4 ? L : 4, VW, M><<<waves, kWave, lds, s>>>(a, v);
    else sddmm_task_kernel<L, NEAR, false, L < 8 ? L : 8, VW, M><<<waves, kWave, lds, s>>>(a, v);
  });
}

template <bool NEAR, int VW>
static void launch_dot_tasks(int L, int lh, bool mask, unsigned waves, hipStream_t s, const SddmmArgs& a, const TaskView& v) {
  switch (L) {
    case 1: launch_dot_tasks_l<1, NEAR, VW>(lh, mask, waves, s, a, v); break;
    case 2: launch_dot_tasks_l<2, NEAR, VW>(lh, mask, waves, s, a, v); break;
    case 4: launch_dot_tasks_l<4, NEAR, VW>(lh, mask, waves, s, a, v); break;
    case 8: launch_dot_tasks_l<8, NEAR, VW>(lh, mask, waves, s, a, v); break;
    case 16: launch_dot_tasks_l<16, NEAR, VW>(lh, mask, waves, s, a, v); break;
    case 32: launch_dot_tasks_l<32, NEAR, VW>(lh, mask, waves, s, a, v); break;
    default: launch_dot_tasks_l<64, NEAR, VW>(lh, mask, waves, s, a, v); break;
  }
}

template <int VW>
static void launch_dot(bool near, int L, int lh, bool mask, unsigned waves, hipStream_t s, const SddmmArgs& a, const TaskView& v) {
  if (near) launch_dot_tasks<true, VW>(L, lh, mask, waves, s, a, v);
  else launch_dot_tasks<false, VW>(L, lh, mask, waves, s, a, v);
}

static void launch_proj(int L, dim3 grid, hipStream_t s, const ProjSide& u, const ProjSide& w, int F, int D, int H) {
  switch (L) {
    case 1: vertex_proj_kernel<1><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    case 2: vertex_proj_kernel<2><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    case 4: vertex_proj_kernel<4><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    case 8: vertex_proj_kernel<8><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    case 16: vertex_proj_kernel<16><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    case 32: vertex_proj_kernel<32><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
    default: vertex_proj_kernel<64><<<grid, kBlock, 0, s>>>(u, w, F, D, H); break;
  }
}

static hgnn_status launch_edge_score(const SddmmArgs& a, int64_t seg_blocks, hipStream_t s) {
  const int spad = kWave * 4 * ((a.S + 255) / 256);
  const size_t lds = size_t(spad) * sizeof(int) * kWavesPerBlock;
  const dim3 gs{unsigned(seg_blocks > 0 ? seg_blocks : 1), 1u, 1u};
  switch (a.H) {
    case 1: edge_score_seg_kernel<1><<<gs, kBlock, lds, s>>>(a); break;
    case 2: edge_score_seg_kernel<2><<<gs, kBlock, lds, s>>>(a); break;
    case 4: edge_score_seg_kernel<4><<<gs, kBlock, lds, s>>>(a); break;
    case 8: edge_score_seg_kernel<8><<<gs, kBlock, lds, s>>>(a); break;
    default: edge_score_seg_kernel<0><<<gs, kBlock, lds, s>>>(a); break;
  }
  HGNN_LAUNCH_CHECK("edge_score_seg_kernel");
  return HGNN_OK;
}

hgnn_status gat_check(const hgnn_plan* p, int H, int D, const hgnn_half* U, int64_t ldu, const hgnn_half* Vt, int64_t ldv,
                      const hgnn_half* a_l, const hgnn_half* a_r, const char* who) {
  const int F = H * D, LH = D / 8;
  // Vt == nullptr: only the row side is wanted
  HGNN_REQUIRE(D % 8 == 0 && (LH & (LH - 1)) == 0 && F <= 512 && ldu % 8 == 0 && ldv % 8 == 0 && aligned16(U) &&
                   aligned16(Vt) && aligned16(a_l) && aligned16(a_r),
               HGNN_EUNSUPPORTED,
               "%s: the per-vertex projection needs D = 8 * 2^k, H * D <= 512, ld %% 8 == 0 and 16-byte aligned U, Vt, a_l, a_r",
               who);
  HGNN_REQUIRE(H <= p->max_H, HGNN_EINVAL, "%s: H = %d exceeds the plan's max_H = %d", who, H, p->max_H);
  return HGNN_OK;
}

hgnn_status gat_project(const hgnn_plan* p, const hgnn_csr* g, int H, int D, const hgnn_half* U, int64_t ldu,
                        const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l, const hgnn_half* a_r, hipStream_t s,
                        const char* who) {
  const hgnn_status st = gat_check(p, H, D, U, ldu, Vt, ldv, a_l, a_r, who);
  if (st != HGNN_OK) return st;
  const int F = H * D;
  const int L = pow2_at_least(F / 8), G = kWave / L;
  float* el = p->vscratch;
  float* er = p->vscratch + size_t(g->nrows) * H;
  const ProjSide u{reinterpret_cast<const half_t*>(U), ldu, g->nrows, reinterpret_cast<const half_t*>(a_l), el};
  const ProjSide w{reinterpret_cast<const half_t*>(Vt), ldv, Vt ? g->ncols : 0, reinterpret_cast<const half_t*>(a_r), er};
  launch_proj(L, dim3(unsigned(ceil_div(std::max(u.nv, w.nv), int64_t(kWavesPerBlock) * G))), s, u, w, F, D, H);
  HGNN_LAUNCH_CHECK("vertex_proj_kernel");
  return HGNN_OK;
}

}  // namespace hgnn

using namespace hgnn;

extern "C" hgnn_status hgnn_sddmm(const hgnn_csr* g, const hgnn_plan* p, hgnn_sddmm_op op, int32_t H, int32_t D,
                                  const hgnn_half* U, int64_t ldu, const hgnn_half* Vt, int64_t ldv,
                                  const hgnn_half* a_l, const hgnn_half* a_r, float neg_slope, hgnn_half* out,
                                  void* stream) {
  clear_error();
  hgnn_status st = check_csr_args(g, "hgnn_sddmm");
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(op == HGNN_SDDMM_DOT || op == HGNN_SDDMM_GAT_SCORE, HGNN_EINVAL, "hgnn_sddmm: unknown op %d", int(op));
  HGNN_REQUIRE(H >= 1 && D >= 1, HGNN_EINVAL, "hgnn_sddmm: H = %d, D = %d must be positive", H, D);
  const int64_t F64 = int64_t(H) * D;
  HGNN_REQUIRE(F64 <= (1 << 20), HGNN_EINVAL, "hgnn_sddmm: H * D too large");
  const int F = int(F64);
  HGNN_REQUIRE(F % 2 == 0, HGNN_EINVAL, "hgnn_sddmm: F = H*D = %d is odd; pad the feature length to the next even number", F);
  HGNN_REQUIRE(ldu >= F && ldv >= F && ldu % 2 == 0 && ldv % 2 == 0, HGNN_EINVAL, "hgnn_sddmm: bad leading dimension");
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EUNSUPPORTED, "hgnn_sddmm: an edge-id map is not supported here");
  if (g->nnz == 0) return HGNN_OK;
  HGNN_REQUIRE(U && Vt && out, HGNN_EINVAL, "hgnn_sddmm: U, Vt or out is NULL");
  const bool score = op == HGNN_SDDMM_GAT_SCORE;
  HGNN_REQUIRE(!score || (a_l && a_r), HGNN_EINVAL, "hgnn_sddmm: GAT_SCORE needs a_l and a_r");
  if (p)
    HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
                 "hgnn_sddmm: the plan was built for another graph");
  hipStream_t s = static_cast<hipStream_t>(stream);
  SddmmArgs a{};
  a.rowptr = g->rowptr;
  a.col = g->col;
  a.erow = g->row;
  a.U = reinterpret_cast<const half_t*>(U);
  a.Vt = reinterpret_cast<const half_t*>(Vt);
  a.a_l = reinterpret_cast<const half_t*>(a_l);
  a.a_r = reinterpret_cast<const half_t*>(a_r);
  a.out = reinterpret_cast<half_t*>(out);
  a.ldu = ldu;
  a.ldv = ldv;
  a.nnz = g->nnz;
  a.nrows = g->nrows;
  a.ncols = g->ncols;
  a.H = H;
  a.D = D;
  a.F = F;
  a.slope = neg_slope;
  if (p) {
    a.seg_lo = p->seg_row_lo;
    a.seg_hi = p->seg_row_hi;
    a.nseg = p->nseg;
    a.S = p->S;
  }
  const int LH = D / 8;
  const bool wide = F <= 512 && ldu % 8 == 0 && ldv % 8 == 0 && aligned16(U) && aligned16(Vt);
  const bool vec = wide && D % 8 == 0 && (LH & (LH - 1)) == 0 && (!score || (aligned16(a_l) && aligned16(a_r)));
  // one head of any even length: 16-byte loads up to the padded pitch, the tail masked (DOT over a plan only)
  const bool masked = wide && !vec && !score && H == 1 && p != nullptr;
  const int L = (vec || masked) ? pow2_at_least((F + 7) / 8) : 0;
  const int64_t seg_blocks = p ? ceil_div(p->nseg, kWavesPerBlock) : 0;

  if (vec && score && p && H <= p->max_H) {
    // project every vertex once, then one add per (edge, head)
    hgnn_status st2 = gat_project(p, g, H, D, U, ldu, Vt, ldv, a_l, a_r, s, "hgnn_sddmm");
    if (st2 != HGNN_OK) return st2;
    a.el = p->vscratch;
    a.er = p->vscratch + size_t(g->nrows) * H;
    if (H == 1 && p->ns > 0 && p->slice_scores) return slice_edge_score(p, g, a.el, a.er, nullptr, neg_slope, out, s);
    return launch_edge_score(a, seg_blocks, s);
  }
  if ((vec || masked) && !score && p) {
    // halves per lane: the plan's setting, when the shape allows a narrower load than 16 bytes
    const int vw = p->vec_halves, lh = D / vw;
    if (vw != 8)
      HGNN_REQUIRE(vec && F <= kWave * vw && D % vw == 0 && (lh & (lh - 1)) == 0, HGNN_EUNSUPPORTED,
                   "hgnn_sddmm: %d halves per lane needs F <= %d and D / %d a power of two", vw, kWave * vw, vw);
    // column-blocked plan: block after block, so that the gathered slice of Vt stays cache resident (a plan built over an
    // edge-id map maps its blocks to that map's slots)
    const hgnn_row_tasks* t = p->tasks;
    if (p->nb > 1 && !p->block_eid) {
      p = walked_cut(p, true);
      t = p->btasks;
      a.col = p->bcol;
      a.delta = p->bdelta;
    }
    const int lanes = pow2_at_least((F + vw - 1) / vw);
    TaskView v = task_view(t, kWave / lanes, at_ranges(t, kRangesDot, int64_t(g->ncols) * F * 2, p->l2_bytes), comes_back(false, int64_t(g->ncols) * ldv * 2, p->llc_bytes), false);
    v.longer = long_rounds(t->nb, p->nrows, t->nnz, p->S, kWave / lanes, 4 + 2 * H);
    const int waves = v.first_wave[t->nb];
    if (waves > 0) {
      const bool near = near_table(g->ncols, ldv);
      if (vw == 8) launch_dot<8>(near, lanes, lh, masked, unsigned(waves), s, a, v);
      else if (vw == 4) launch_dot<4>(near, lanes, lh, false, unsigned(waves), s, a, v);
      else launch_dot<2>(near, lanes, lh, false, unsigned(waves), s, a, v);
      HGNN_LAUNCH_CHECK("sddmm_task_kernel");
    }
    return HGNN_OK;
  }
  const size_t lds_tile = size_t(kTile) * H * sizeof(hgnn_half) * kWavesPerBlock;
  if (vec && lds_tile <= 65536) {
    dim3 grid(unsigned(ceil_div(g->nnz, int64_t(kTile) * kWavesPerBlock)));
    if (score) launch_edge<true>(L, grid, lds_tile, s, a);
    else launch_edge<false>(L, grid, lds_tile, s, a);
    HGNN_LAUNCH_CHECK("sddmm_edge_kernel");
    return HGNN_OK;
  }
  dim3 grid(unsigned(ceil_div(g->nnz * H, kBlock)));
  if (score) sddmm_scalar_kernel<true><<<grid, kBlock, 0, s>>>(a);
  else sddmm_scalar_kernel<false><<<grid, kBlock, 0, s>>>(a);
  HGNN_LAUNCH_CHECK("sddmm_scalar_kernel");
  return HGNN_OK;
}

extern "C" hgnn_status hgnn_gat_alpha(const hgnn_csr* g, const hgnn_plan* p, int32_t H, int32_t D, const hgnn_half* U,
                                      int64_t ldu, const hgnn_half* Vt, int64_t ldv, const hgnn_half* a_l,
                                      const hgnn_half* a_r, float neg_slope, const float* lse, hgnn_half* alpha,
                                      void* stream) {
  clear_error();
  const char* who = "hgnn_gat_alpha";
  hgnn_status st = check_csr_args(g, who);
  if (st != HGNN_OK) return st;
  HGNN_REQUIRE(p != nullptr, HGNN_EINVAL, "%s: plan is NULL", who);
  HGNN_REQUIRE(p->nrows == g->nrows && p->ncols == g->ncols && p->nnz == g->nnz, HGNN_EINVAL,
               "%s: the plan was built for another graph", who);
  HGNN_REQUIRE(g->eid == nullptr, HGNN_EUNSUPPORTED, "%s: an edge-id map is not supported here", who);
  HGNN_REQUIRE(H >= 1 && D >= 1 && int64_t(H) * D <= 512, HGNN_EINVAL, "%s: H = %d, D = %d out of range", who, H, D);
  if (g->nnz == 0) return HGNN_OK;
  HGNN_REQUIRE(U && Vt && a_l && a_r && lse && alpha, HGNN_EINVAL, "%s: NULL argument", who);
  hipStream_t s = static_cast<hipStream_t>(stream);
  st = gat_project(p, g, H, D, U, ldu, Vt, ldv, a_l, a_r, s, who);
  if (st != HGNN_OK) return st;
  SddmmArgs a{};
  a.rowptr = g->rowptr;
  a.col = g->col;
  a.out = reinterpret_cast<half_t*>(alpha);
  a.nnz = g->nnz;
  a.nrows = g->nrows;
  a.ncols = g->ncols;
  a.H = H;
  a.D = D;
  a.F = H * D;
  a.slope = neg_slope;
  a.seg_lo = p->seg_row_lo;
  a.seg_hi = p->seg_row_hi;
  a.nseg = p->nseg;
  a.S = p->S;
  a.el = p->vscratch;
  a.er = p->vscratch + size_t(g->nrows) * H;
  a.lse = lse;
  if (H == 1 && p->ns > 0 && p->slice_scores) return slice_edge_score(p, g, a.el, a.er, lse, neg_slope, alpha, s);
  return launch_edge_score(a, ceil_div(p->nseg, kWavesPerBlock), s);
}

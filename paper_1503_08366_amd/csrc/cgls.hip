// Indirect projection (Section 3.5): each ADMM iteration projects onto the
// graph by CGLS on the reduced least-squares problem
//     x = argmin ||x - c||^2 + ||A^ x - d||^2     ([A^; I] x ~ [d; c]),
// started from the half step x_h, with no Gram matrix and no factorisation.
//
// Per iteration (after the prox step, which also sets x = x_h):
//   C0   row pass     t = A^ x_h         -> r1 = d - t, primal residual sums
//   C1   column pass  A^T [r1, nu_h]     -> s = A^T r1 + c - x, dual residual sums
//   then CG steps j = 0, 1, ..., cap - 1, three launches each:
//   KA   row pass     q_j = A^ s_j + beta q_{j-1}  (= A^ p_j), r1 -= alpha_{j-1} q_{j-1},
//                     ||q_j||^2 sums; the step runs only while ||s_j|| > thr
//   KB   column pass  A^T [r1, q_j] split partials
//   KC   finish       p_j = s_j + beta p_{j-1}, x += alpha_j p_j,
//                     s_{j+1} = A^T r1 - alpha_j A^T q_j + c - x
//   and a last KA (j = cap) that only applies the pending r1 update.
// alpha_j = ||s_j||^2 / (||q_j||^2 + ||p_j||^2), beta = ||s_j||^2 / ||s_{j-1}||^2,
// with ||p_j||^2 = ||s_j||^2 + 2 beta s_j^T p_{j-1} + beta^2 ||p_{j-1}||^2 (the
// expansion of ||s_j + beta p_{j-1}||^2, whose terms the previous finish
// summed), so every scalar is known at the start of the launch that needs it.
// The projection leaves x~ = c - x, y~ = r1, y = d - r1 (the prox step reads
// them in that form).  The tolerance is thr = cg_tol * eps_dual / rho: the
// final normal residual s equals x~ + A^T y~, which enters the next dual
// residual multiplied by rho.
//
// float32 A with m >= n and rows of at most 2048 entries: C0 with C1, and KA with
// KB, are one launch each that reads A once (cg_one_pass_body): what the column
// pass needs of row i (r1_i and nu_i or q_i) is known as soon as row i's product
// is, so the row is used for both while it is in registers.
//
// Every launch of a step decides from the same partial sums whether the step
// runs, so the sequence of launches is fixed (it can be captured once) while
// the work stops as soon as the tolerance is met.
#include "cgls.hpp"
#include "gemv_launch.hpp"

namespace pogs {

template <typename T>
__global__ __launch_bounds__(kBlock) void cg_first_finish_kernel(IterArgs<T> p, int splits, int ncolp) {
  if (!cg_first_enter<T>(p)) return;
  EpiCgFirst<T> e{p};
  __shared__ GemvFinishLds lds;
  gemv_t_finish_body<2, EpiCgFirst<T>>(hw_block(), p.n, splits, p.part, ncolp, e, lds);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void cg_finish_kernel(IterArgs<T> p, int j, int splits, int ncolp) {
  EpiCgStep<T> e;
  if (!cg_step_enter<T>(p, j, &e)) return;
  __shared__ GemvFinishLds lds;
  gemv_t_finish_body<2, EpiCgStep<T>>(hw_block(), p.n, splits, p.part, ncolp, e, lds);
}

// One pass over A for both products of a CG step (or, FIRST, of the passes that
// start a projection): the layout of tall_one_pass_body -- a wave takes a
// contiguous run of rows, a row's NC pieces are in registers, the next row's
// loads are in flight, inputs and outputs of 64 rows at a time live in the
// lanes -- with one product per row and float64 column sums throughout.
//   FIRST: t = A x_h, r1 = d - t, (t - y_h)^2; column sums A^T [r1, nu_h]
//   else:  q = A s + beta q', r1 -= alpha' q' (q', alpha' of step j - 1), q^2;
//          column sums A^T [r1, q]
// HBM bound; 20000 x 1000: the step 37.5 -> 24.2 us.  The 2 x 4 NC float64 sums per
// lane leave one workgroup of 8 waves per CU, and rows of at most 1024 entries
// (64 sums of NC = 8 spill: 65 us at 20000 x 2000 against 59.4 in two passes).
template <int NC, bool NT, bool FIRST>
__device__ __forceinline__ void cg_one_pass_body(const IterArgs<float> &p, int j, int cap, int ncolp) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int NW = kOnePassThreads / kWave, CH = 64 * NC;
  constexpr int CPT = (CH + kOnePassThreads - 1) / kOnePassThreads;
  static_assert(NW <= kCgWaves, "scratch of the prologues");
  __shared__ float xs[256 * NC];
  __shared__ double red[NW][2][256 * NC];
  __shared__ double bs[NW];
  const bool stopped = p.ctrl->st[p.par].done != 0;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const int W = gridDim.x * NW;
  const int gw = __builtin_amdgcn_readfirstlane(blockIdx.x * NW + w);
  const int m = p.m, n = p.n, ld = p.ld;
  const float *A = p.A;
  const float *vec = FIRST ? p.x : p.sv;  // context vectors, 16-byte aligned
  f4 stg[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int idx = 4 * (threadIdx.x + kOnePassThreads * k);
    if (idx < 256 * NC) {
      if (idx + 3 < n) {
        stg[k] = *reinterpret_cast<const f4 *>(vec + idx);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) stg[k][c] = idx + c < n ? vec[idx + c] : 0.f;
      }
    }
  }
  const int rq = m / W, rr = m % W;
  const int nrows = rq + (gw < rr ? 1 : 0), row0 = gw * rq + min(gw, rr);
  int cofs[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) cofs[u] = min(4 * lane + 256 * u, ld - 4);
  auto load = [&](f4 *dst, int r) {
    const float *rp = A + (size_t)r * ld;
#pragma unroll
    for (int u = 0; u < NC; ++u) dst[u] = mat_load<NT>(reinterpret_cast<const f4 *>(rp + cofs[u]));
  };
  f4 a0[NC], a1[NC];
  if (nrows > 0) load(a0, row0);
  // FIRST: d, y_h, nu_h; else q', r1
  float b0 = 0.f, b1 = 0.f, b2 = 0.f;
  auto load_inputs = [&](int i0) {
    if (lane < min(kWave, nrows - i0)) {
      const int i = row0 + i0 + lane;
      b0 = FIRST ? p.dy[i] : p.qv[i];
      b1 = FIRST ? p.yh[i] : p.yt[i];
      if (FIRST) b2 = p.nu[i];
    }
  };
  load_inputs(0);
  if (stopped) return;
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int idx = 4 * (threadIdx.x + kOnePassThreads * k);
    if (idx < 256 * NC) *reinterpret_cast<f4 *>(&xs[idx]) = stg[k];
  }
  double alpha_prev = 0.0, beta = 0.0;
  if constexpr (!FIRST) {
    EpiCgRows<float> e;
    if (!cg_rows_enter<float>(p, j, cap, &e)) return;
    alpha_prev = e.alpha_prev;
    beta = e.beta;
  }
  const bool has_prev = j > 0;
  __syncthreads();

  double acc[2][NC][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[r][u][k] = 0.0;
  double sq = 0.0;
  float o_r = 0.f, o_q = 0.f;
  auto bcast = [](float v, int t) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t)); };
  auto row = [&](const f4 *a, int t) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const f4 x = *reinterpret_cast<const f4 *>(&xs[4 * lane + 256 * u]);
#pragma unroll
      for (int k = 0; k < 4; ++k) s = fma((double)a[u][k], (double)x[k], s);
    }
    s = wave_sum_dpp(s);
    float r1, w1;
    if constexpr (FIRST) {
      r1 = (float)((double)bcast(b0, t) - s);
      w1 = bcast(b2, t);
      const double r = s - (double)bcast(b1, t);
      sq += r * r;
    } else {
      r1 = bcast(b1, t);
      double qn = s;
      if (has_prev) {
        const double qo = (double)bcast(b0, t);
        r1 = (float)((double)r1 - alpha_prev * qo);
        qn = s + beta * qo;
      }
      w1 = (float)qn;
      sq += (double)w1 * (double)w1;
    }
    if (lane == t) {
      o_r = r1;
      o_q = w1;
    }
    const double d0 = (double)r1, d1 = (double)w1;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double e = (double)a[u][k];
        acc[0][u][k] = fma(e, d0, acc[0][u][k]);
        acc[1][u][k] = fma(e, d1, acc[1][u][k]);
      }
    }
  };
  for (int i0 = 0; i0 < nrows; i0 += kWave) {
    const int cnt = min(kWave, nrows - i0), mine = row0 + i0 + lane;
    if (i0 > 0) load_inputs(i0);
    for (int t = 0; t < cnt; t += 2) {
      const int i = i0 + t;
      if (i + 1 < nrows) load(a1, row0 + i + 1);
      row(a0, t);
      if (t + 1 >= cnt) break;
      if (i + 2 < nrows) load(a0, row0 + i + 2);
      row(a1, t + 1);
    }
    if (lane < cnt) {
      if (FIRST || has_prev) p.yt[mine] = o_r;
      if (!FIRST) p.qv[mine] = o_q;
    }
  }
  // the workgroup's column sums, the waves added in order
  if (lane == 0) bs[w] = sq;  // the same in every lane
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) red[w][r][4 * lane + 256 * u + k] = acc[r][u][k];
  __syncthreads();
  for (int c = threadIdx.x; c < ncolp; c += kOnePassThreads)
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      double v = 0.0;
#pragma unroll
      for (int k = 0; k < NW; ++k) v += red[k][r][c];
      p.part[(size_t)(blockIdx.x * 2 + r) * ncolp + c] = v;
    }
  if (threadIdx.x == 0) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) v += bs[k];
    (FIRST ? p.s_pri : p.s_qq)[blockIdx.x] = v;
  }
}

template <int NC, bool NT, bool FIRST>
__global__ __launch_bounds__(kOnePassThreads) void cg_one_pass_kernel(IterArgs<float> p, int j, int cap, int ncolp) {
  cg_one_pass_body<NC, NT, FIRST>(p, j, cap, ncolp);
}

// The same for rows of 1025 to 2048 entries: four waves share a row (thread t of
// a half workgroup has columns 4 t + 1024 u), so a lane holds 16 float64 sums, four
// rows at a time are in flight and their products meet in LDS once per group,
// as in equil_sweep_body; the two halves of a workgroup take alternate groups and
// add their column sums in LDS.  20000 x 2000: the step 59.4 -> 38.3
// us (the pass 34 us: 160 MB at 4.7 TB/s).  Two workgroups per CU (128 registers, 20 of
// them spilled, twice the partial sums) measured 49.0.
constexpr int kCgGroup = 4;
template <bool NT, bool FIRST>
__global__ __launch_bounds__(kOnePassThreads) void cg_group_pass_kernel(IterArgs<float> p, int j, int cap, int ncolp) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int R = kCgGroup, U = 2, HALF = kOnePassThreads / 2, HW = HALF / kWave;
  __shared__ double red[2][2][R][HW];  // [turn parity][half][row][wave]
  __shared__ double cs[2048];
  __shared__ double bs[2];
  if (p.ctrl->st[p.par].done != 0) return;
  const int t = threadIdx.x % HALF, half = __builtin_amdgcn_readfirstlane(threadIdx.x / HALF);
  const int lane = t & (kWave - 1), w = t >> 6;
  const int m = p.m, n = p.n, ld = p.ld;
  const int r0 = (int)((int64_t)m * blockIdx.x / gridDim.x), r1 = (int)((int64_t)m * (blockIdx.x + 1) / gridDim.x);
  const float *vec = FIRST ? p.x : p.sv;
  f4 a[R][U], v[U];
  float b0 = 0.f, b1 = 0.f, b2 = 0.f;  // the row's own inputs, row i in lane i of each wave
  auto load = [&](int i0) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int row = min(i0 + i, r1 - 1);  // past the end: the last row again, not added
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = min(4 * t + 1024 * u, ld - 4);  // past ld: the last piece again, times zeros
        a[i][u] = mat_load<NT>(reinterpret_cast<const f4 *>(p.A + (size_t)row * ld + c));
      }
    }
    const int mine = min(i0 + (lane & (R - 1)), r1 - 1);
    b0 = FIRST ? p.dy[mine] : p.qv[mine];
    b1 = FIRST ? p.yh[mine] : p.yt[mine];
    if (FIRST) b2 = p.nu[mine];
  };
  auto bcast = [](float x, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l)); };
  const int first = r0 + half * R;
  if (first < r1) load(first);
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = 4 * t + 1024 * u + k;
      v[u][k] = c < n ? vec[c] : 0.f;
    }
  double alpha_prev = 0.0, beta = 0.0;
  if constexpr (!FIRST) {
    EpiCgRows<float> e;
    if (!cg_rows_enter<float>(p, j, cap, &e)) return;
    alpha_prev = e.alpha_prev;
    beta = e.beta;
  }
  const bool has_prev = j > 0;
  double acc[2][U][4];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[0][u][k] = acc[1][u][k] = 0.0;
  double sq = 0.0;
  const int turns = (r1 - r0 + 2 * R - 1) / (2 * R);  // the same for both halves: a barrier per turn
  for (int g = 0; g < turns; ++g) {
    const int i0 = first + g * 2 * R;
    // the rows and the vector stay float32 in their registers: kept widened
    // from one use to the next they would spill
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" : "+v"(v[u]));
    double s[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      double z = 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) z = fma((double)a[i][u][k], (double)v[u][k], z);
      s[i] = z;
      __builtin_amdgcn_sched_barrier(0);
    }
    const double z = wave_sum4(s[0], s[1], s[2], s[3]);  // rows 0, 2, 1, 3 in the lanes' rows of 16
    if ((lane & 15) == 0) red[g & 1][half][((lane >> 4) & 1) * 2 + (lane >> 5)][w] = z;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const double *q = red[g & 1][half][i];
      const double x = (q[0] + q[1]) + (q[2] + q[3]);
      const bool live = i0 + i < r1;
      float o0, o1;
      if constexpr (FIRST) {
        o0 = (float)((double)bcast(b0, i) - x);
        o1 = bcast(b2, i);
        const double r = x - (double)bcast(b1, i);
        sq += live ? r * r : 0.0;
      } else {
        o0 = bcast(b1, i);
        double qn = x;
        if (has_prev) {
          const double qo = (double)bcast(b0, i);
          o0 = (float)((double)o0 - alpha_prev * qo);
          qn = x + beta * qo;
        }
        o1 = (float)qn;
        sq += live ? (double)o1 * (double)o1 : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(a[i][u]));
      if (t == i && live) {
        if (FIRST || has_prev) p.yt[i0 + i] = o0;
        if (!FIRST) p.qv[i0 + i] = o1;
      }
      const double d0 = live ? (double)o0 : 0.0, d1 = live ? (double)o1 : 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double e = (double)a[i][u][k];
          acc[0][u][k] = fma(e, d0, acc[0][u][k]);
          acc[1][u][k] = fma(e, d1, acc[1][u][k]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i0 + 2 * R < r1) load(i0 + 2 * R);
  }
  if (t == 0) bs[half] = sq;  // the same in every thread of the half
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    __syncthreads();
    if (half)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) cs[4 * t + 1024 * u + k] = acc[r][u][k];
    __syncthreads();
    if (!half)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int c = 4 * t + 1024 * u + k;
          if (c < ncolp) p.part[(size_t)(blockIdx.x * 2 + r) * ncolp + c] = acc[r][u][k] + cs[c];
        }
  }
  if (threadIdx.x == 0) (FIRST ? p.s_pri : p.s_qq)[blockIdx.x] = bs[0] + bs[1];
}

template <bool NT, bool FIRST>
static void launch_cg_one_pass_nt(const IterArgs<float> &p, int j, int cap, int ncolp, hipStream_t s) {
  const dim3 grid((unsigned)p.cg_blocks), block(kOnePassThreads);
  if (p.ld <= 256) hipLaunchKernelGGL((cg_one_pass_kernel<1, NT, FIRST>), grid, block, 0, s, p, j, cap, ncolp);
  else if (p.ld <= 512) hipLaunchKernelGGL((cg_one_pass_kernel<2, NT, FIRST>), grid, block, 0, s, p, j, cap, ncolp);
  else if (p.ld <= 1024) hipLaunchKernelGGL((cg_one_pass_kernel<4, NT, FIRST>), grid, block, 0, s, p, j, cap, ncolp);
  else hipLaunchKernelGGL((cg_group_pass_kernel<NT, FIRST>), grid, block, 0, s, p, j, cap, ncolp);
}
template <bool FIRST>
static void launch_cg_one_pass(const IterArgs<float> &p, int j, int cap, int ncolp, hipStream_t s) {
  if (p.nt_rows) launch_cg_one_pass_nt<true, FIRST>(p, j, cap, ncolp, s);
  else launch_cg_one_pass_nt<false, FIRST>(p, j, cap, ncolp, s);
}

template <int NC, bool NT>
__global__ __launch_bounds__(kBlock) void cg_rows_f32_kernel(IterArgs<float> p, int j, int cap) {
  EpiCgRows<float> e;
  if (!cg_rows_enter<float>(p, j, cap, &e)) return;
  gemv_n_rows_body<1, NC, EpiCgRows<float>, NT>(hw_block(), p.A, p.m, p.n, p.ld, p.sv, p.sv, e);
}

template <typename T, int LPR, int RPT, bool NT>
__global__ __launch_bounds__(kBlock) void cg_rows_lds_kernel(IterArgs<T> p, int j, int cap) {
  EpiCgRows<T> e;
  if (!cg_rows_enter<T>(p, j, cap, &e)) return;
  __shared__ GemvNLds<T, 1> lds;
  gemv_n_body<T, T, 1, false, LPR, RPT, EpiCgRows<T>, NT>(hw_block(), p.A, p.m, p.n, p.ld, p.sv, p.sv, e, lds);
}

template <typename T, bool NT> static void launch_cg_rows_nt(const IterArgs<T> &p, int j, int cap, hipStream_t s) {
  const GemvNShape sh = gemv_n_shape(p.m, p.n, p.ld, sizeof(T));
  const dim3 grid(sh.grid), block(kBlock);
  if constexpr (sizeof(T) == 4) {
    switch (sh.variant) {
      case GEMV_N_ROWS1: hipLaunchKernelGGL((cg_rows_f32_kernel<1, NT>), grid, block, 0, s, p, j, cap); return;
      case GEMV_N_ROWS2: hipLaunchKernelGGL((cg_rows_f32_kernel<2, NT>), grid, block, 0, s, p, j, cap); return;
      case GEMV_N_ROWS4: hipLaunchKernelGGL((cg_rows_f32_kernel<4, NT>), grid, block, 0, s, p, j, cap); return;
      case GEMV_N_ROWS8: hipLaunchKernelGGL((cg_rows_f32_kernel<8, NT>), grid, block, 0, s, p, j, cap); return;
      default: break;
    }
  }
  switch (sh.variant) {
    case GEMV_N_L64R4: hipLaunchKernelGGL((cg_rows_lds_kernel<T, 64, 4, NT>), grid, block, 0, s, p, j, cap); break;
    case GEMV_N_L64R1: hipLaunchKernelGGL((cg_rows_lds_kernel<T, 64, 1, NT>), grid, block, 0, s, p, j, cap); break;
    case GEMV_N_L16R4: hipLaunchKernelGGL((cg_rows_lds_kernel<T, 16, 4, NT>), grid, block, 0, s, p, j, cap); break;
    default: hipLaunchKernelGGL((cg_rows_lds_kernel<T, 16, 1, NT>), grid, block, 0, s, p, j, cap); break;
  }
}

template <typename T> static void launch_cg_rows(const IterArgs<T> &p, int j, int cap, hipStream_t s) {
  if (p.nt_rows) launch_cg_rows_nt<T, true>(p, j, cap, s);
  else launch_cg_rows_nt<T, false>(p, j, cap, s);
}

template <typename T> static void launch_first(const IterArgs<T> &p, int splits, int rps, int ncolp, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (p.cg_blocks) {
      launch_cg_one_pass<true>(p, 0, 0, ncolp, s);
      hipLaunchKernelGGL(cg_first_finish_kernel<T>, dim3(cdiv(p.n, kFinishCols)), dim3(kBlock), 0, s, p, p.cg_blocks,
                         ncolp);
      return;
    }
  }
  EpiCgStart<T> e0{{p}};
  gemv_n<T, T, 1>(p.A, p.m, p.n, p.ld, p.x, p.x, e0, s, p.nt_rows);
  const int tiles = (int)cdiv(p.n, gemv_t_tile(sizeof(T)));
  EpiBase<T> eb{p};
  if (p.nt_cols)
    hipLaunchKernelGGL((gemv_t_kernel<T, T, 2, false, EpiBase<T>, true>), dim3(tiles, splits), dim3(kBlock), 0, s, p.A,
                       p.m, p.n, p.ld, (const T *)p.yt, (const T *)p.nu, rps, p.part, ncolp, eb);
  else
    hipLaunchKernelGGL((gemv_t_kernel<T, T, 2, false, EpiBase<T>, false>), dim3(tiles, splits), dim3(kBlock), 0, s,
                       p.A, p.m, p.n, p.ld, (const T *)p.yt, (const T *)p.nu, rps, p.part, ncolp, eb);
  hipLaunchKernelGGL(cg_first_finish_kernel<T>, dim3(cdiv(p.n, kFinishCols)), dim3(kBlock), 0, s, p, splits, ncolp);
}

template <typename T> static void launch_step(const IterArgs<T> &p, int j, int cap, int splits, int rps, int ncolp,
                                              hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (p.cg_blocks) {
      launch_cg_one_pass<false>(p, j, cap, ncolp, s);
      hipLaunchKernelGGL(cg_finish_kernel<T>, dim3(cdiv(p.n, kFinishCols)), dim3(kBlock), 0, s, p, j, p.cg_blocks,
                         ncolp);
      return;
    }
  }
  launch_cg_rows<T>(p, j, cap, s);
  const int tiles = (int)cdiv(p.n, gemv_t_tile(sizeof(T)));
  EpiCgSkip<T> ek{p};
  if (p.nt_cols)
    hipLaunchKernelGGL((gemv_t_kernel<T, T, 2, false, EpiCgSkip<T>, true>), dim3(tiles, splits), dim3(kBlock), 0, s,
                       p.A, p.m, p.n, p.ld, (const T *)p.yt, (const T *)p.qv, rps, p.part, ncolp, ek);
  else
    hipLaunchKernelGGL((gemv_t_kernel<T, T, 2, false, EpiCgSkip<T>, false>), dim3(tiles, splits), dim3(kBlock), 0, s,
                       p.A, p.m, p.n, p.ld, (const T *)p.yt, (const T *)p.qv, rps, p.part, ncolp, ek);
  hipLaunchKernelGGL(cg_finish_kernel<T>, dim3(cdiv(p.n, kFinishCols)), dim3(kBlock), 0, s, p, j, splits, ncolp);
}

template <typename T>
void launch_iteration_cg(const IterArgs<T> &p, int splits, int rps, int ncolp, int cap, hipStream_t s) {
  hipLaunchKernelGGL(prox_cg_kernel<T>, dim3(p.n_smu + p.n_syh), dim3(kBlock), 0, s, p);
  launch_first<T>(p, splits, rps, ncolp, s);
  for (int j = 0; j < cap; ++j) launch_step<T>(p, j, cap, splits, rps, ncolp, s);
  if constexpr (sizeof(T) == 4) {
    if (p.cg_blocks) return launch_cg_one_pass<false>(p, cap, cap, ncolp, s);
  }
  launch_cg_rows<T>(p, cap, cap, s);
}

template <typename T>
void launch_iteration_cg_part(const IterArgs<T> &p, int which, int splits, int rps, int ncolp, hipStream_t s) {
  if (which == 0) hipLaunchKernelGGL(prox_cg_kernel<T>, dim3(p.n_smu + p.n_syh), dim3(kBlock), 0, s, p);
  else if (which == 1) launch_first<T>(p, splits, rps, ncolp, s);
  else launch_step<T>(p, 0, 1 << 30, splits, rps, ncolp, s);
}

template <typename T> void launch_prox_cg(const IterArgs<T> &p, hipStream_t s) {
  hipLaunchKernelGGL(prox_cg_kernel<T>, dim3(p.n_smu + p.n_syh), dim3(kBlock), 0, s, p);
}

template <typename T> void launch_cg_from_state(const IterArgs<T> &p, hipStream_t s) {
  hipLaunchKernelGGL(cg_from_state_kernel<T>, dim3(cdiv(p.n + p.m, kBlock)), dim3(kBlock), 0, s, p);
}

template void launch_iteration_cg<float>(const IterArgs<float> &, int, int, int, int, hipStream_t);
template void launch_iteration_cg<double>(const IterArgs<double> &, int, int, int, int, hipStream_t);
template void launch_iteration_cg_part<float>(const IterArgs<float> &, int, int, int, int, hipStream_t);
template void launch_iteration_cg_part<double>(const IterArgs<double> &, int, int, int, int, hipStream_t);
template void launch_prox_cg<float>(const IterArgs<float> &, hipStream_t);
template void launch_prox_cg<double>(const IterArgs<double> &, hipStream_t);
template void launch_cg_from_state<float>(const IterArgs<float> &, hipStream_t);
template void launch_cg_from_state<double>(const IterArgs<double> &, hipStream_t);

}  // namespace pogs

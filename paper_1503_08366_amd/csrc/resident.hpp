// Resident solve (direct projection, residual stopping): a chunk of iterations
// in one launch of G workgroups that stay on the GPU together and exchange
// vectors through memory instead of ending a kernel per step.
//
// The matrix is taken with its longer side as rows: M = A^ (m >= n) or its
// transpose (m < n), L x q.  Workgroup g owns R consecutive rows of M (the
// "long" side: y for m >= n, x for m < n) with their vectors and function
// parameters, and nc consecutive columns (the "short" side) with theirs and
// the matching rows of K^{-1}, which it keeps in LDS; so does it with its rows
// of M where they fit.  One iteration:
//   short stage  the column sums of M^T [., .] (m >= n: [d, nu_h], m < n: [c, x_h])
//                arrive; half step of the own columns, right-hand side of the
//                reduced system and residual (Section 3.5);       -> exchange 2
//   solve        own rows of K^{-1} rhs;                          -> exchange 3
//   long stage   M times the solution and the half step: the projected
//                iterate, scaled dual and residual of the own rows, then the
//                next iteration's half step of those rows and their share of
//                the column sums;                                 -> exchange 1
//   control      stopping test and Algorithm 3, the same in every workgroup.
// The next half step on the long side needs the rho that Algorithm 3 picks
// after this iteration, of whose inputs only the long side's own residual is
// still open; it is predicted from the previous iteration's, and where the rule
// then picks another rho the half step and its column sums are formed again.
//
// Exchanges.  Every 8-byte word carries 32 bits of data and the exchange's
// number in the other 32, written and read with relaxed device-scope atomics,
// so a word is its own arrival flag: a reader polls the words it needs, no
// fence and no cache write-back is involved, and an exchange costs one trip
// through memory (MI355X, 512 threads per workgroup: 1.1 us at 32 workgroups, 1.6 at
// 128, 1.9 at 256, against 2.1-3.8 us with a counter or flag barrier between
// plain stores and loads and 3-4 us for the end of one kernel and the start of
// the next).  Reuse of a buffer is safe without a further barrier: every
// workgroup reads exchange 1 from every other one, so a workgroup that has
// passed exchange 1 of an iteration knows that all have read exchanges 2 and
// 3 of the iteration before (they published exchange 1 afterwards); exchange 1
// itself alternates between two buffers, and is overwritten only after
// another exchange 1 that needed every reader's words.
// Every wait is bounded.  Until a workgroup has seen words of this launch from
// all others, some may not be on the GPU yet: other streams' kernels hold their
// CUs, or will not leave any.  It waits kResArrive polls (about 7 ms) for them.
// Under a stream of 0.9 ms kernels a 1.2 ms solve takes 4.6 ms so, where one launch
// per step took 109; behind 120 ms kernels, or with half the CUs masked off, the
// wait is lost, and with a bound of kResSpin (0.7 s, now the bound once all have
// arrived) such a solve took 570 and 766 ms.  A workgroup that gives up sets
// ctrl->res_failed and ends; the others, and those that start later, see that
// and end too, and the host solves again with one launch per step.
#pragma once

#include "iter.hpp"

namespace pogs {

constexpr int kResThreads = 512;
typedef unsigned long long ResWord;

// What the host reads after a launch (pinned memory).
struct ResHost {
  CtrlState st;
  unsigned e1, e2;  // numbers of the last exchanges
  int failed;       // a workgroup gave up waiting
};

template <typename T> struct ResArgs {
  int L, q, ld, G, nc, wide;  // ld: row stride of M and of K^{-1} (q rounded up to 64)
  const T *M, *Kinv;
  FnDev<T> fl, fs;            // long- and short-side functions
  T *lv, *lvt, *lh, *ldu, *lp;  // long side: iterate, scaled dual, half step, its dual, projection input
  T *sv, *svt, *sh, *sdu;       // short side
  Ctrl *ctrl;
  ResHost *host;              // pinned: the state after the launch, for the host's check
  ResWord *x1[2], *x2, *x3;   // exchange buffers
  int first, iters;           // first launch of a solve; iterations per launch
  unsigned polls;             // bound of a wait until all workgroups have arrived (0: it gives up before its first wait)
};

// Words of the exchange buffers: 1 (each of two): per reader, writer and own
// column of the reader two float64 sums, and per writer two residual sums; 2:
// per writer its entries of two short vectors and its residual sums; 3: the
// entries of one short vector.  A workgroup's words of an exchange lie together
// and one wave stores them.
template <typename T> inline size_t res_words1(int G, int nc) { return (size_t)G * G * nc * 4 + (size_t)G * 4; }
template <typename T> inline size_t res_words2(int G, int nc) { return (size_t)G * (2 * nc * (sizeof(T) / 4) + 4); }
template <typename T> inline size_t res_words3(int G, int nc) { return (size_t)G * nc * (sizeof(T) / 4); }

// Waves of a workgroup, pieces of 16 bytes per lane and row (NC), rows of M
// (RPW) and of K^{-1} (KR) per wave: all of them in registers for the launch.
constexpr int kResWaves = kResThreads / kWave;
template <typename T, int NC, int RPW> struct ResShape {
  static constexpr int VN = Vec16<T>::N;
  static constexpr int LD = kWave * VN * NC;  // columns the lanes cover
  static constexpr int KR = NC >= 4 ? 1 : 2;
  static constexpr int rows = kResWaves * RPW, cols = kResWaves * KR;  // per workgroup, at most
  // LDS: three vectors, the waves' column sums (then the arriving ones), the residual sums
  static constexpr int vec = 0, red = 3 * LD * (int)sizeof(T);
  static constexpr size_t red_bytes(int G) {
    return std::max<size_t>((size_t)kResWaves * 2 * LD * 8, (size_t)G * cols * 16);
  }
  static constexpr size_t lds_bytes(int G) { return red + red_bytes(G) + (size_t)2 * G * 8; }
};

__device__ __forceinline__ void res_put(ResWord *p, unsigned tag, unsigned v) {
  __hip_atomic_store(p, ((ResWord)tag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_put(ResWord *p, unsigned tag, float v) { res_put(p, tag, __float_as_uint(v)); }
__device__ __forceinline__ void res_put(ResWord *p, unsigned tag, double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  res_put(p, tag, (unsigned)b);
  res_put(p + 1, tag, (unsigned)(b >> 32));
}
__device__ __forceinline__ ResWord res_get(const ResWord *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ctrl->res_failed, set and seen while a launch runs.
__device__ __forceinline__ int res_gave_up(const Ctrl *c) {
  return __hip_atomic_load(&c->res_failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words src(i), i < n, with the given tag into LDS dst(i).  Every thread loads
// up to U words at once and tries again until all of them carry the tag, at
// most `polls` times and not after another workgroup has given up.
template <int U, class Src, class Dst>
__device__ __forceinline__ void res_gather(int n, unsigned tag, unsigned polls, const Ctrl *ctrl, int *bad, Src src,
                                           Dst dst) {
  for (int b = threadIdx.x; b < n; b += U * kResThreads) {
    ResWord x[U];
    unsigned spin = 0;
    for (;;) {
      unsigned miss = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (b + u * kResThreads < n) x[u] = res_get(src(b + u * kResThreads));
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (b + u * kResThreads < n) miss |= (unsigned)(x[u] >> 32) ^ tag;
      if (!miss) break;
      if (++spin > polls || ((spin & 63) == 0 && (*(volatile int *)bad || res_gave_up(ctrl)))) {
        *(volatile int *)bad = 1;
        break;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b + u * kResThreads < n) *dst(b + u * kResThreads) = (unsigned)x[u];
  }
}

__device__ __forceinline__ double lane_value(double v, int l) {  // l uniform
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// One function element and the vectors of its row or column.
template <typename T> struct ResElem {
  int fh;
  T fa, fb, fc, fd, fe;
  T v, vt;     // iterate and scaled dual
  T h, du, p;  // half step, its dual, projection input
  __device__ __forceinline__ void load_fn(const FnDev<T> &F, int i) {
    fh = F.h[i];
    fa = F.a[i];
    fb = F.b[i];
    fc = F.c[i];
    fd = F.d[i];
    fe = F.e[i];
  }
  __device__ __forceinline__ HalfStep<T> step(T rho, T resc, T alpha) const {
    return half_step<T>(fh, fa, fb, fc, fd, fe, v, vt, rho, resc, alpha);
  }
};

// Wave w of workgroup g has rows 8 RPW g + w RPW + i (i < RPW) of M and rows
// g nc + w + 8 k (k < KR, w + 8 k < nc) of K^{-1}; lane i < RPW (k < KR) of the wave works on
// the vectors and function parameters (in LDS) of its row i (column k), so a
// wave takes its rows from the products to the half step and the column sums
// alone.
template <typename T, int NC, int RPW>
__device__ __forceinline__ void resident_body(const ResArgs<T> &p, char *smem) {
  using S = ResShape<T, NC, RPW>;
  using V = typename Vec16<T>::type;
  constexpr int VN = S::VN, W = sizeof(T) / 4, KR = S::KR, LD = S::LD, NW = kResWaves;
  __shared__ double scal[4];  // long residual and norm, short residual and norm (squared)
  __shared__ double bs[2][NW];
  __shared__ double dots[NW][2][RPW + (RPW & 1)];
  __shared__ ResElem<T> le[NW][RPW], se[NW][KR];
  __shared__ T out[2][S::cols];  // what the next exchange takes from the own columns
  __shared__ int bad;
  __shared__ unsigned none;
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = blockIdx.x, G = p.G, ld = p.ld, q = p.q;
  const int nc = p.nc;  // <= S::cols
  const float inv_nc = 1.0f / (float)nc;
  const bool wide = p.wide != 0;
  const int r0 = g * S::rows + w * RPW, c0 = g * nc + w;  // the wave's first row and column
  T *vec0 = (T *)(smem + S::vec), *vec1 = vec0 + LD, *vecr = vec1 + LD;
  double *red = (double *)(smem + S::red);
  double *sums = (double *)(smem + S::red + S::red_bytes(G));

  CtrlState st = p.ctrl->st[0];  // every thread runs the control step on its own copy
  if (t == 0) bad = 0;
  auto fail = [&]() {
    if (t == 0) {
      __hip_atomic_store(&p.ctrl->res_failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      p.host->failed = 1;
    }
  };
  if (p.polls == 0 || res_gave_up(p.ctrl)) return fail();
  if (st.done) return;
  const CtrlParams qc = ctrl_params(p.ctrl);
  const double eps_abs = qc.eps_abs, eps_rel = qc.eps_rel;
  const T alpha = (T)qc.alpha;
  unsigned e1 = p.ctrl->res_e1, e2 = p.ctrl->res_e2;

  // the wave's rows; rows past L and pieces past ld are zero
  V a[RPW][NC], kin[KR][NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    const int c = (lane + kWave * u) * VN;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
      a[i][u] = c < ld && r0 + i < p.L ? *reinterpret_cast<const V *>(p.M + (size_t)(r0 + i) * ld + c) : V{};
#pragma unroll
    for (int k = 0; k < KR; ++k)
      kin[k][u] = c < ld && w + NW * k < nc && c0 + NW * k < q
                      ? *reinterpret_cast<const V *>(p.Kinv + (size_t)(c0 + NW * k) * ld + c) : V{};
  }
  for (int i = t; i < 3 * LD; i += kResThreads) vec0[i] = T(0);  // entries past q stay zero
  if (t < 2 * S::cols) out[t / S::cols][t % S::cols] = T(0);
  ResElem<T> &l = le[w][lane < RPW ? lane : 0], &s = se[w][lane < KR ? lane : 0];
  T nh = T(0), ndu = T(0), np = T(0);
  const bool lmine = lane < RPW && r0 + lane < p.L, smine = lane < KR && w + NW * lane < nc && c0 + NW * lane < q;
  const int li = lmine ? r0 + lane : 0, si = smine ? c0 + NW * lane : 0;
  if (lmine) {
    l.load_fn(p.fl, li);
    l.v = p.lv[li];
    l.vt = p.lvt[li];
    l.h = p.lh[li];
    l.du = p.ldu[li];
    l.p = p.lp[li];
  }
  if (smine) {
    s.load_fn(p.fs, si);
    s.v = p.sv[si];
    s.vt = p.svt[si];
  }
  // products of the wave's RR rows x (in registers) with one or two LDS
  // vectors: lane i gets the sums of row i
  auto products = [&](auto &x, auto rows_c, const T *v0, const T *v1, double &o0, double &o1) {
    constexpr int RR = decltype(rows_c)::value, RE = RR + (RR & 1);
    double s0[RE], s1[RE];
#pragma unroll
    for (int i = 0; i < RE; ++i) s0[i] = s1[i] = 0.0;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const V y0 = *reinterpret_cast<const V *>(v0 + (lane + kWave * u) * VN);
      V y1 = V{};
      if (v1) y1 = *reinterpret_cast<const V *>(v1 + (lane + kWave * u) * VN);
#pragma unroll
      for (int k = 0; k < VN; ++k) {
        const double d0 = (double)y0[k], d1 = (double)y1[k];
#pragma unroll
        for (int i = 0; i < RR; ++i) {
          const double e = (double)x[i][u][k];
          s0[i] = fma(e, d0, s0[i]);
          if (v1) s1[i] = fma(e, d1, s1[i]);
        }
      }
    }
    // four sums at a time; lanes 0, 32 (16, 48) have those of row i (i + 1)
#pragma unroll
    for (int i = 0; i < RE; i += 2) {
      const double z = wave_sum4(s0[i], s1[i], s0[i + 1], s1[i + 1]);
      if ((lane & 15) == 0) dots[w][lane >> 5][i + ((lane >> 4) & 1)] = z;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int i = lane < RR ? lane : 0;
    o0 = dots[w][0][i];
    o1 = dots[w][1][i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  // sum of G float64 pairs in `sums` ([pair][2]) into scal[at], scal[at + 1] (waves 0 and 1)
  auto sum_pairs = [&](int at) {
    if (w < 2) {
      double v = 0.0;
      for (int i = lane; i < G; i += kWave) v += sums[2 * i + w];
      v = wave_sum_dpp(v);
      if (lane == 0) scal[at + w] = v;
    }
  };
  // the waves' sums of two values, for total() after the next barrier
  auto wave_sums = [&](double x, double y) {
    const double z = row16_sum_dpp(merge_sum16(merge_sum32(x, y), 0.0));
    if (lane == 0) bs[0][w] = z;
    if (lane == 32) bs[1][w] = z;
  };
  // word i (0..3) of the two totals, the waves added in order
  auto total = [&](int i) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) v += bs[i >> 1][k];
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (unsigned)(i & 1 ? b >> 32 : b);
  };

  // Each turn of the loop forms a half step of the long side and its column
  // sums (unless an earlier launch did), then runs the control step of the
  // iteration whose residuals came with them (fresh), and the next iteration
  // up to the long side's new iterate.  A turn that is not fresh follows the
  // start of a solve or a rho that was not the predicted one.
  bool publish = p.first != 0, fresh = false;
  double rho = st.rho, resc = st.rescale;  // of the half step to form
  double res2 = 0.0, lnorm2 = 0.0, r_s = 0.0, eps_s = 0.0, eps_l = 0.0;
  int it = 0;
  unsigned polls = p.polls;
  for (;;) {
    // float32 rows stay float32 in their registers: without this the compiler
    // widens them all ahead of the loop, twice the registers
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int u = 0; u < NC; ++u) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) asm volatile("" : "+v"(a[i][u]));
#pragma unroll
        for (int k = 0; k < KR; ++k) asm volatile("" : "+v"(kin[k][u]));
      }
    }
    const size_t n1 = (size_t)G * nc * 4;  // words of exchange 1 per reader
    if (publish) {
      // ---- half step of the own rows, their share of M^T [d, n] ---------------
      double norm2 = 0.0;
      if (lmine) {
        const HalfStep<T> hs = l.step((T)rho, (T)resc, alpha);
        nh = hs.h;
        ndu = hs.dual;
        np = hs.proj_in;
        norm2 = wide ? (double)ndu * (double)ndu : (double)nh * (double)nh;
      }
      ++e1;
      ResWord *x1 = p.x1[e1 & 1];
      const double dd = (double)np, dn = (double)(wide ? nh : ndu);
      double d[RPW], n[RPW];
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        d[i] = lane_value(dd, i);
        n[i] = lane_value(dn, i);
      }
#pragma unroll
      for (int u = 0; u < NC; ++u) {
        double a0[VN], a1[VN];
#pragma unroll
        for (int k = 0; k < VN; ++k) a0[k] = a1[k] = 0.0;
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
          for (int k = 0; k < VN; ++k) {
            const double e = (double)a[i][u][k];
            a0[k] = fma(e, d[i], a0[k]);
            a1[k] = fma(e, n[i], a1[k]);
          }
        double *o = red + (size_t)w * LD + (lane + kWave * u) * VN;
#pragma unroll
        for (int k = 0; k < VN; ++k) {
          o[k] = a0[k];
          o[(size_t)NW * LD + k] = a1[k];
        }
      }
      wave_sums(res2, norm2);
      __syncthreads();
      if (t < 4) res_put(x1 + (size_t)G * n1 + (size_t)g * 4 + t, e1, total(t));
      // the waves' sums added in wave order; they stay where wave 0's were
      double *red1 = red + (size_t)NW * LD;
      for (int c = t; c < LD; c += kResThreads) {
        double v0 = 0.0, v1 = 0.0;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
          v0 += red[(size_t)k * LD + c];
          v1 += red1[(size_t)k * LD + c];
        }
        red[c] = v0;
        red1[c] = v1;
      }
      __syncthreads();
      // word by word, in the order they lie in memory: 64 lanes fill whole lines
      // (8-byte words at a stride of 32 bytes cost twice the time: 125
      // workgroups, q = 1000: 5.2 -> 2.8 us for the exchange)
      {
        const unsigned *z0 = (const unsigned *)red, *z1 = (const unsigned *)red1;
        ResWord *to = x1 + (size_t)g * nc * 4;
        const int hop = (G - 1) * nc * 4;  // from one reader's words to the next's
        for (int i = t; i < (int)n1; i += kResThreads) {
          const int c = i >> 2, o = (int)(((float)c + 0.5f) * inv_nc);  // c / nc (exact: c < 2^20)
          unsigned v = 0;  // columns past q: zeros
          if (c < LD) v = ((i & 2) ? z1 : z0)[2 * c + (i & 1)];
          res_put(to + (size_t)o * hop + i, e1, v);
        }
      }
      __syncthreads();  // red is free again
    }
    // ---- exchange 1 -------------------------------------------------------------
    {
      const ResWord *own = p.x1[e1 & 1] + (size_t)g * n1, *tail = p.x1[e1 & 1] + (size_t)G * n1 - n1;
      unsigned *r32 = (unsigned *)red, *s32 = (unsigned *)sums - n1;
      res_gather<8>((int)n1 + 4 * G, e1, polls, p.ctrl, &bad, [&](int i) { return (i < (int)n1 ? own : tail) + i; },
                    [&](int i) { return (i < (int)n1 ? r32 : s32) + i; });
    }
    __syncthreads();
    if (bad) return fail();
    sum_pairs(0);
    // the wave's 2 KR column sums: a group of lanes per sum
    double cw = 0.0, cs = 0.0;
    {
      constexpr int NV = 2 * KR, LPV = kWave / NV;
      const int v = lane / LPV, at = 2 * (w + NW * (v >> 1)) + (v & 1);
      double z = 0.0;
      for (int i = lane % LPV; i < G; i += LPV) z += red[(size_t)i * 2 * nc + at];
      z = row16_sum_dpp(z);
      if (LPV == 32) z = swap_pair_sum16(z);
#pragma unroll
      for (int k = 0; k < KR; ++k) {
        const double zw = lane_value(z, 2 * k * LPV), zs = lane_value(z, (2 * k + 1) * LPV);
        if (lane == k) {
          cw = zw;
          cs = zs;
        }
      }
    }
    __syncthreads();
    // ---- control ------------------------------------------------------------------
    if (fresh) {
      const double r_l = sqrt(scal[0]);
      if (wide) control_decide(qc, st, r_s, eps_s, r_l, eps_l);
      else control_decide(qc, st, r_l, eps_l, r_s, eps_s);
      if (st.done) break;
      fresh = false;
      if (st.rho != rho) {  // the same in every workgroup
        rho = st.rho;
        resc = st.rescale;
        res2 = 0.0;
        continue;
      }
    }
    if (publish && lmine) {
      l.h = nh;
      l.du = ndu;
      l.p = np;
    }
    if (it++ == p.iters) break;
    lnorm2 = scal[1];
    // ---- short stage --------------------------------------------------------------
    ++e2;
    double sres2 = 0.0, snorm2 = 0.0;
    if (smine) {
      const HalfStep<T> hs = s.step((T)st.rho, (T)st.rescale, alpha);
      s.h = hs.h;
      s.du = hs.dual;
      s.p = hs.proj_in;
      // m < n: rhs = A c - d, A x_h - y_h; m >= n: rhs = c + A^T d, A^T nu_h + mu_h
      const T rhs = wide ? (T)(cw - (double)s.p) : (T)((double)s.p + cw);
      const double r = wide ? cs - (double)s.h : cs + (double)s.du;
      const double o = wide ? (double)s.h : (double)s.du;
      sres2 = r * r;
      snorm2 = o * o;
      out[0][w + NW * lane] = rhs;
      out[1][w + NW * lane] = wide ? s.du : s.h;
    }
    wave_sums(sres2, snorm2);
    __syncthreads();
    const int nw = nc * W, ch = 2 * nw + 4;  // words of a vector's own entries, of exchange 2
    if (t < ch)
      res_put(p.x2 + (size_t)g * ch + t, e2,
              t < 2 * nw ? ((const unsigned *)out[t < nw ? 0 : 1])[t < nw ? t : t - nw] : total(t - 2 * nw));
    {
      const float inv_ch = 1.0f / (float)ch;
      unsigned *vr = (unsigned *)vecr, *v1 = (unsigned *)vec1, *s32 = (unsigned *)sums;
      res_gather<8>(G * ch, e2, polls, p.ctrl, &bad, [&](int i) { return p.x2 + i; },
                    [&](int i) {
                      const int o = (int)(((float)i + 0.5f) * inv_ch), k = i - o * ch;
                      const int e = o * nw + (k < nw ? k : k - nw);  // word of the vector
                      unsigned *d = k < nw ? vr + e : v1 + e;
                      d = e < LD * W ? d : &none;  // columns past the rows' pieces
                      return k < 2 * nw ? d : s32 + o * 4 + (k - 2 * nw);
                    });
    }
    __syncthreads();
    if (bad) return fail();
    polls = kResSpin;  // every workgroup is here
    // ---- solve ----------------------------------------------------------------------
    sum_pairs(2);
    double x0, x1;
    products(kin, std::integral_constant<int, KR>{}, vecr, nullptr, x0, x1);
    if (smine) {
      s.v = wide ? (T)((double)s.p + x0) : (T)x0;
      s.vt = s.p - s.v;
      out[0][w + NW * lane] = wide ? s.vt : s.v;
    }
    __syncthreads();
    if (t < nw) res_put(p.x3 + (size_t)g * nw + t, e2, ((const unsigned *)out[0])[t]);
    // Algorithm 3's prediction: the short side's residual and both tolerances of
    // this iteration, the previous iteration's test of the long side's residual
    r_s = sqrt(scal[2]);
    eps_s = eps_abs + eps_rel * sqrt(scal[3]);
    eps_l = eps_abs + eps_rel * sqrt(lnorm2);
    rho = st.rho;
    resc = 1.0;
    if (qc.adaptive) {
      const bool pri_ok = wide ? r_s < eps_s : st.r_pri < st.eps_pri;
      const bool dual_ok = wide ? st.r_dual < st.eps_dual : r_s < eps_s;
      if (dual_ok && qc.tau * st.k > st.l) rho = qc.delta * st.rho;
      else if (pri_ok && qc.tau * st.k > st.u) rho = st.rho / qc.delta;
      if (rho != st.rho) resc = st.rho / rho;
    }
    {
      unsigned *v0 = (unsigned *)vec0;
      res_gather<4>(q * W, e2, polls, p.ctrl, &bad, [&](int i) { return p.x3 + i; }, [&](int i) { return v0 + i; });
    }
    __syncthreads();
    if (bad) return fail();
    // ---- long stage -------------------------------------------------------------------
    products(a, std::integral_constant<int, RPW>{}, vec0, vec1, x0, x1);
    res2 = 0.0;
    if (lmine) {
      // m < n: x = c + A^T y~, A^T nu_h + mu_h; m >= n: y = A x, A x_h - y_h
      l.v = wide ? (T)((double)l.p + x0) : (T)x0;
      const double r = wide ? x1 + (double)l.du : x1 - (double)l.h;
      l.vt = l.p - l.v;
      res2 = r * r;
    }
    publish = fresh = true;
  }

  if (lmine) {
    p.lh[li] = l.h;
    p.ldu[li] = l.du;
    p.lp[li] = l.p;
    p.lv[li] = l.v;
    p.lvt[li] = l.vt;
  }
  if (smine) {
    p.sh[si] = s.h;
    p.sdu[si] = s.du;
    p.sv[si] = s.v;
    p.svt[si] = s.vt;
  }
  if (g == 0 && t == 0) {
    p.ctrl->st[0] = st;
    p.ctrl->res_e1 = e1;
    p.ctrl->res_e2 = e2;
    p.host->st = st;
    p.host->e1 = e1;
    p.host->e2 = e2;
  }
}

}  // namespace pogs

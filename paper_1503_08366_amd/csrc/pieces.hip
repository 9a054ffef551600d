// Passes over a large sparse float32 matrix kept in pieces: split by columns
// into segments of at most kPcSeg, so that the part of the vector a segment
// multiplies is in the workgroup's LDS and every gather is an LDS read.
//
// A row pass that gathers from L2 ran at 130 G gathers/s on gfx950 (245 us for
// the 32 M entries of a 2000000 x 200000 matrix, and no faster with more rows
// in flight): each 4-byte gather moves a 128-byte line through a CU's L1, while
// the entries themselves need 50 us of HBM.
//
// Measured, 2000000 x 200000, 16 entries a row: A^ s 245 -> 70 us, A^T r1 255
// -> 79 (the entries, row bounds and partial sums are 255 and 250 MB), a CG step
// 500 -> 180, a Lasso 336 -> 132 ms.  Of a pass, adding up the products takes
// about 12 us, refilling the segments 5, the gathers 2.  Two groups of entries on
// the way: 1 and 3 are 1 and 6 % slower (3 runs out of registers).  The bounds of
// the rows are 16 bits each from their block's: as 32-bit ones they were 50 MB of
// a pass, and a step 189 us.
//
// A workgroup (16 waves, one per CU: the segment takes most of the LDS) owns
// up to kPcTile rows; a wave takes 64 of them at a time, one per lane, for each
// segment in turn.  The entries of 64 rows in one segment are contiguous, so
// the wave loads them with 16-byte loads, 4 per lane, multiplies each by its
// element of the segment and lays the float64 products out in LDS, where each
// lane then adds up its own row's.  The rows' sums stay in registers over the
// segments.  The next 64 rows' entries are loaded before these are added up.
//
// A^ (more rows than columns): a workgroup goes through all segments and ends
// with the rows' epilogue.  A^T: few long rows, so its segments are dealt to
// kPcGroups workgroups per row range, whose float64 sums a finish kernel adds in
// order.  The column index inside a segment takes 16 bits: 6 bytes per entry
// instead of 8.
#include "cgls.hpp"

namespace pogs {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned short u4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
// memory that no kernel writes while it is read: uniform loads go to scalar registers
#define KernelConst __attribute__((address_space(4)))

constexpr int kPcThreads = kPcWaves * 64;
constexpr int kPcChunk = 256;  // entries a wave handles at once, 4 per lane
constexpr int kPcSegLoads = (kPcSeg + 4 * kPcThreads - 1) / (4 * kPcThreads);
constexpr int kPcAhead = 2;    // groups of 64 rows whose entries are on the way
constexpr int kPcWg = 256;     // workgroups of a launch that fill the GPU

struct PcLds {
  float v[kPcSeg];
  double prod[kPcWaves][kPcChunk + 4];  // the sums read up to 3 past their last product
};

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// acc[g] = row (first row of the tile) + (16 g + wave) 64 + lane times the
// vector, over the segments sg0 .. sg1 - 1; src(i) returns elements i .. i + 3.
template <class Src>
__device__ __forceinline__ void pieces_body(const SpPieces &A, int tile, int sg0, int sg1, const Src &src, PcLds &lds,
                                            double (&acc)[kPcRpl]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = tile * A.tile, r1 = min(A.rows, r0 + A.tile);
  double *pw = lds.prod[w];
#pragma unroll
  for (int g = 0; g < kPcRpl; ++g) acc[g] = 0.0;
  for (int sg = sg0; sg < sg1; ++sg) {
    const int c0 = sg * A.seg, len = min(A.seg, A.cols - c0);
    const KernelConst int *base = (const KernelConst int *)(uintptr_t)(A.base + (size_t)sg * A.blocks);
    const uint16_t *off = A.off + (size_t)sg * A.blocks * 64;
    f4 st[kPcSegLoads];
#pragma unroll
    for (int u = 0; u < kPcSegLoads; ++u) {
      const int t = (u * kPcThreads + threadIdx.x) * 4;
      if (t < len) st[u] = src(c0 + t);
    }
    // where a block's entries begin and end, and every row's from there; a lane's
    // entries end where the next lane's begin (blocks past the tile repeat its last)
    int begin[kPcRpl], ends[kPcRpl], lo[kPcRpl];
#pragma unroll
    for (int g = 0; g < kPcRpl; ++g) {
      const int b = min(r0 + (g * kPcWaves + w) * 64, r1 - 1) >> 6;
      begin[g] = base[b];
      ends[g] = base[b + 1];
      lo[g] = off[b * 64 + lane];
    }
    __syncthreads();  // the last segment has been read
#pragma unroll
    for (int u = 0; u < kPcSegLoads; ++u) {
      const int t = (u * kPcThreads + threadIdx.x) * 4;
      if (t < len) *reinterpret_cast<f4 *>(lds.v + t) = st[u];
    }
    f4 a[kPcAhead + 1];
    u4 j[kPcAhead + 1];
    auto load = [&](int k, int ke, f4 &av, u4 &jv) {
      const int kk = k + 4 * lane;
      av = f4{0.f, 0.f, 0.f, 0.f};
      jv = u4{0, 0, 0, 0};
      if (kk < ke) {
        av = *reinterpret_cast<const f4 *>(A.va + kk);
        jv = *reinterpret_cast<const u4 *>(A.ci + kk);
      }
    };
    auto first = [&](int g) { return begin[g] & ~3; };
#pragma unroll
    for (int g = 0; g < kPcAhead; ++g) load(first(g), ends[g], a[g], j[g]);
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kPcRpl; ++g) {
      if (r0 + (g * kPcWaves + w) * 64 >= r1) break;
      constexpr int R = kPcAhead + 1;
      if (g + kPcAhead < kPcRpl) load(first(g + kPcAhead), ends[g + kPcAhead], a[(g + kPcAhead) % R], j[(g + kPcAhead) % R]);
      const int kb = first(g), ke = ends[g];
      const int next = __shfl_down(lo[g], 1);
      const int from = begin[g] + lo[g], hi = lane == 63 ? ke : begin[g] + next;
      f4 av = a[g % R];
      u4 jv = j[g % R];
      double s = 0.0;
      for (int k = kb;;) {
        d2 p0, p1;
        p0.x = (double)av.x * (double)lds.v[jv.x];
        p0.y = (double)av.y * (double)lds.v[jv.y];
        p1.x = (double)av.z * (double)lds.v[jv.z];
        p1.y = (double)av.w * (double)lds.v[jv.w];
        reinterpret_cast<d2 *>(pw)[2 * lane] = p0;
        reinterpret_cast<d2 *>(pw)[2 * lane + 1] = p1;
        wave_lds_order();
        const int q1 = min(hi - k, kPcChunk);
        for (int q = max(from - k, 0); q < q1; q += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double t = pw[q + u];
            if (q + u < q1) s += t;
          }
        }
        wave_lds_order();
        k += kPcChunk;
        if (k >= ke) break;
        load(k, ke, av, jv);
      }
      acc[g] += s;
    }
  }
}

// fn(row, sum) for every row of the tile that this lane holds
template <class F> __device__ __forceinline__ void pieces_rows(const SpPieces &A, int tile, const double (&acc)[kPcRpl],
                                                               const F &fn) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = tile * A.tile, r1 = min(A.rows, r0 + A.tile);
#pragma unroll
  for (int g = 0; g < kPcRpl; ++g) {
    const int row = r0 + (g * kPcWaves + w) * 64 + lane;
    if (row < r1) fn(row, acc[g]);
  }
}

struct SrcVec {
  const float *v;
  __device__ f4 operator()(int i) const { return *reinterpret_cast<const f4 *>(v + i); }
};
template <class Epi>
__device__ __forceinline__ void pieces_rows_pass(const SpPieces &A, const float *v, const Epi &e, PcLds &lds) {
  __shared__ double bs[kPcWaves];
  double acc[kPcRpl], contrib = 0.0;
  pieces_body(A, blockIdx.x, 0, A.nseg, SrcVec{v}, lds, acc);
  pieces_rows(A, blockIdx.x, acc, [&](int row, double s) { contrib += e.row(row, s, 0.0); });
  const double t = block_sum(contrib, bs);
  if (threadIdx.x == 0) e.block_done(blockIdx.x, t);
}

// t = A^ x_h, r1 = d - t
__global__ __launch_bounds__(kPcThreads) void pc_start_kernel(IterArgs<float> p) {
  __shared__ PcLds lds;
  EpiCgStart<float> e{{p}};
  if (e.skip()) return;
  pieces_rows_pass(p.pa, p.x, e, lds);
}

// q_j = A^ s_j + beta q_{j-1}
struct EpiPcRows {
  IterArgs<float> p;
  double beta;
  int has_prev;
  __device__ double row(int i, double as, double) const {
    const float qt = (float)(has_prev ? as + beta * (double)p.qv[i] : as);
    p.qv[i] = qt;
    return (double)qt * (double)qt;
  }
  __device__ void block_done(int b, double v) const { p.s_qq[b] = v; }
};

__global__ __launch_bounds__(kPcThreads) void pc_rows_kernel(IterArgs<float> p, int j, int cap) {
  __shared__ PcLds lds;
  EpiCgRows<float> e;
  if (!cg_rows_enter<float, false>(p, j, cap, &e)) return;
  pieces_rows_pass(p.pa, p.sv, EpiPcRows{p, e.beta, e.has_prev}, lds);
}

// alpha_j, and r1 -= alpha_j q_j.  In the pass over A^T, where every row range's
// workgroups would do it again as they fill their segments, it cost 34 us of
// that pass's 121; here it takes 10 and the pass finds alpha_j decided.
__global__ __launch_bounds__(kBlock) void pc_residual_kernel(IterArgs<float> p, int j) {
  EpiCgStep<float> e;
  if (!cg_step_enter<float>(p, j, &e)) return;
  for (int i = (blockIdx.x * kBlock + threadIdx.x) * 4; i < p.m; i += gridDim.x * kBlock * 4) {
    f4 r = *reinterpret_cast<const f4 *>(p.yt + i);
    const f4 q = *reinterpret_cast<const f4 *>(p.qv + i);
#pragma unroll
    for (int u = 0; u < 4; ++u) r[u] = (float)((double)r[u] - e.alpha * (double)q[u]);
    *reinterpret_cast<f4 *>(p.yt + i) = r;
  }
}

// Partial sums of A^T v.  Workgroups whose index differs by a multiple of
// `groups` (8, as the XCDs) take the same segments, so an XCD's L2 serves a
// segment to all of them.
template <class Src>
__device__ __forceinline__ void pieces_cols_pass(const SpPieces &A, const Src &src, int rhs, double *part, int ncolp,
                                                 PcLds &lds) {
  const int grp = blockIdx.x % A.groups, tile = blockIdx.x / A.groups;
  const int per = (A.nseg + A.groups - 1) / A.groups;
  const int sg0 = min(A.nseg, grp * per), sg1 = min(A.nseg, sg0 + per);
  double acc[kPcRpl];
  pieces_body(A, tile, sg0, sg1, src, lds, acc);
  double *o = part + (size_t)(rhs * A.groups + grp) * ncolp;
  pieces_rows(A, tile, acc, [&](int row, double s) { o[row] = s; });
}

// A^T r1 (blockIdx.y = 0) and A^T nu_h (1)
__global__ __launch_bounds__(kPcThreads) void pc_first_kernel(IterArgs<float> p, int ncolp) {
  __shared__ PcLds lds;
  if (p.ctrl->st[p.par].done) return;
  pieces_cols_pass(p.pat, SrcVec{blockIdx.y ? p.nu : p.yt}, blockIdx.y, p.part, ncolp, lds);
}

// A^T r1 after the update of step j
__global__ __launch_bounds__(kPcThreads) void pc_step_kernel(IterArgs<float> p, int ncolp) {
  __shared__ PcLds lds;
  if ((p.ctrl->st[p.par].done != 0) | (p.ctrl->cg.stop >= 0)) return;
  pieces_cols_pass(p.pat, SrcVec{p.yt}, 0, p.part, ncolp, lds);
}

template <int NRHS, class Epi>
__device__ __forceinline__ void pieces_finish(const IterArgs<float> &p, int ncolp, const Epi &e) {
  __shared__ double bs[kBlock / kWave];
  const int col = blockIdx.x * kBlock + threadIdx.x;
  Sum2 c{0.0, 0.0};
  if (col < p.n) {
    // every partial of the column loaded before the first is added
    double v[NRHS][kPcGroups], s[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
#pragma unroll
      for (int g = 0; g < kPcGroups; ++g) v[r][g] = p.part[(size_t)(r * kPcGroups + g) * ncolp + col];
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
#pragma unroll
      for (int g = 0; g < kPcGroups; ++g) s[r] += v[r][g];
    c = e.column(col, s[0], s[1]);
  }
  const double a = block_sum(c.a, bs), b = block_sum(c.b, bs);
  if (threadIdx.x == 0) e.tile_done(blockIdx.x, a, b);
}

__global__ __launch_bounds__(kBlock) void pc_first_finish_kernel(IterArgs<float> p, int ncolp) {
  if (!cg_first_enter<float>(p)) return;
  pieces_finish<2>(p, ncolp, EpiCgFirst<float>{p});
}

// alpha_j is stored and in r1 already (the second sum is 0).
__global__ __launch_bounds__(kBlock) void pc_step_finish_kernel(IterArgs<float> p, int j, int ncolp) {
  const Ctrl &q = *p.ctrl;
  if ((q.st[p.par].done != 0) | (q.cg.stop >= 0)) return;
  const double beta = j > 0 ? q.cg.gamma[j & 1] / q.cg.gamma[(j - 1) & 1] : 0.0;
  pieces_finish<1>(p, ncolp, EpiCgStep<float>{p, q.cg.alpha, beta, j > 0 ? 1 : 0, (j + 1) & 1});
}

// ---- building the pieces -----------------------------------------------------
// Rows of the source of up to kPcLongRow entries are walked by one lane each, one
// dependent read and write of a counter per entry; longer ones 64 entries at a
// time, to be counted by all waves of a workgroup, to be moved by one wave in
// order, so a piece keeps the source's order.  With lanes alone a full column of
// 2000000 x 200000, one row of A^T, took 0.65 s in each of the two kernels.
constexpr int kPcLongRow = 1024;
constexpr int kPcCountThreads = 1024;

template <class F> __device__ __forceinline__ void pc_row(const Csr<float> &A, int r, const F &fn) {
  for (int s = 0; s < A.nseg; ++s) {
    const int *rp = A.rp + (size_t)s * A.rows + r;
    fn(rp[0], rp[1]);
  }
}
__device__ __forceinline__ int pc_row_length(const Csr<float> &A, int r) {
  int len = 0;
  if (r < A.rows) pc_row(A, r, [&](int k0, int k1) { len += k1 - k0; });
  return len;
}
// 64 entries, c the column of this lane's or -1: fn(segment, lanes in it), by segment.
template <class F> __device__ __forceinline__ void pc_segments(const SpPieces &P, int c, const F &fn) {
  const int sg = c < 0 ? -1 : c / P.seg;
  for (unsigned long long left = __ballot(sg >= 0); left;) {
    const int one = __builtin_amdgcn_readlane(sg, __builtin_ctzll(left));
    const unsigned long long mask = __ballot(sg == one);
    fn(one, mask);
    left &= ~mask;
  }
}

// Also the longest row (rows of up to kPcLongRow entries count as none).
__global__ __launch_bounds__(kPcCountThreads) void pc_count_kernel(Csr<float> A, SpPieces P, int *cnt, PcStats *st) {
  constexpr int NW = kPcCountThreads / 64;
  __shared__ unsigned long long longs[NW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = blockIdx.x * kPcCountThreads, r = r0 + threadIdx.x;
  const int len = pc_row_length(A, r);
  if (r < A.rows && len <= kPcLongRow)
    pc_row(A, r, [&](int k0, int k1) {
      for (int k = k0; k < k1; ++k) ++cnt[(size_t)(A.ci[k] / P.seg) * P.rows + r];
    });
  if (len > kPcLongRow) atomicMax(&st->longest, len);
  const unsigned long long mine = __ballot(len > kPcLongRow);
  if (lane == 0) longs[w] = mine;
  __syncthreads();
  for (int v = 0; v < NW; ++v)
    for (unsigned long long rows = longs[v]; rows; rows &= rows - 1) {
      const int row = r0 + 64 * v + __builtin_ctzll(rows);
      int have = -1, n = 0;  // n more entries in segment `have`
      auto add = [&]() {
        if (n && lane == 0) atomicAdd(cnt + (size_t)have * P.rows + row, n);
      };
      pc_row(A, row, [&](int k0, int k1) {
        for (int64_t k = (int64_t)k0 + 64 * w; k < k1; k += kPcCountThreads)
          pc_segments(P, k + lane < k1 ? A.ci[k + lane] : -1, [&](int sg, unsigned long long mask) {
            if (sg != have) {
              add();
              have = sg;
              n = 0;
            }
            n += __popcll(mask);
          });
      });
      add();
    }
}

__global__ __launch_bounds__(kBlock) void pc_scatter_kernel(Csr<float> A, SpPieces P, int *cur) {
  const int r = blockIdx.x * kBlock + threadIdx.x, lane = threadIdx.x & 63;
  const int len = pc_row_length(A, r);
  auto put = [&](int64_t k, int sg, int to) {
    P.va[to] = A.va[k];
    P.ci[to] = (uint16_t)(A.ci[k] - sg * P.seg);
  };
  if (r < A.rows && len <= kPcLongRow)
    pc_row(A, r, [&](int k0, int k1) {
      for (int k = k0; k < k1; ++k) {
        const int sg = A.ci[k] / P.seg;
        put(k, sg, cur[(size_t)sg * P.rows + r]++);
      }
    });
  for (unsigned long long rows = __ballot(len > kPcLongRow); rows; rows &= rows - 1) {
    const int row = r - lane + __builtin_ctzll(rows);
    int have = -1, at = 0;  // the next entry in segment `have` goes to `at`
    pc_row(A, row, [&](int k0, int k1) {
      constexpr int U = 4;  // groups of 64 on the way
      for (int64_t k = k0; k < k1; k += 64 * U) {
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = k + 64 * u + lane < k1 ? A.ci[k + 64 * u + lane] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u)
          pc_segments(P, c[u], [&](int sg, unsigned long long mask) {
            if (sg != have) {
              if (lane == 0) {
                if (have >= 0) cur[(size_t)have * P.rows + row] = at;
                at = cur[(size_t)sg * P.rows + row];
              }
              have = sg;
              at = __builtin_amdgcn_readfirstlane(at);
            }
            if (mask >> lane & 1) put(k + 64 * u + lane, sg, at + __popcll(mask & ((1ull << lane) - 1)));
            at += __popcll(mask);
          });
      }
    });
  }
}

constexpr int kScanPer = 8, kScanBlock = kBlock * kScanPer;

__global__ __launch_bounds__(kBlock) void pc_block_sums_kernel(const int *v, int64_t len, int *sums) {
  __shared__ int red[kBlock];
  int t = 0;
  for (int u = 0; u < kScanPer; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kScanBlock + u * kBlock + threadIdx.x;
    if (i < len) t += v[i];
  }
  red[threadIdx.x] = t;
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = red[0];
}

// Exclusive prefix sums of `mine` over the workgroup; *total: their sum.
__device__ inline int block_prefix(int mine, int *total) {
  __shared__ int sc[2][kBlock];
  int b = 0;
  sc[0][threadIdx.x] = mine;
  __syncthreads();
  for (int o = 1; o < kBlock; o *= 2, b ^= 1) {
    sc[b ^ 1][threadIdx.x] = sc[b][threadIdx.x] + ((int)threadIdx.x >= o ? sc[b][threadIdx.x - o] : 0);
    __syncthreads();
  }
  const int incl = sc[b][threadIdx.x];
  *total = sc[b][kBlock - 1];
  __syncthreads();
  return incl - mine;
}

__global__ __launch_bounds__(kBlock) void pc_scan_sums_kernel(int *sums, int64_t len) {
  int carry = 0;
  for (int64_t i0 = 0; i0 < len; i0 += kBlock) {
    const int64_t i = i0 + threadIdx.x;
    int total;
    const int at = block_prefix(i < len ? sums[i] : 0, &total);
    if (i < len) sums[i] = carry + at;
    carry += total;
  }
}

__global__ __launch_bounds__(kBlock) void pc_scan_kernel(int *v, int *copy, int64_t len, const int *sums, int nnz) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanPer;
  int x[kScanPer], t = 0, total;
  for (int u = 0; u < kScanPer; ++u) {
    x[u] = i0 + u < len ? v[i0 + u] : 0;
    t += x[u];
  }
  int at = sums[blockIdx.x] + block_prefix(t, &total);
  for (int u = 0; u < kScanPer; ++u)
    if (i0 + u < len) {
      v[i0 + u] = copy[i0 + u] = at;
      at += x[u];
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) v[len] = nnz;
}

// base and off from the rows' beginnings rp.
__global__ __launch_bounds__(kBlock) void pc_bounds_kernel(const int *rp, SpPieces P, int nnz, PcStats *st) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, per = (int64_t)P.blocks * 64;
  if (i >= per * P.nseg) return;
  const int *seg = rp + (i / per) * P.rows;
  const int r = (int)(i % per), b0 = r & ~63, b1 = min(b0 + 64, P.rows);
  const int len = seg[b1] - seg[b0];
  P.off[i] = (uint16_t)(r < P.rows ? seg[r] - seg[b0] : len);
  if (r == b0) {
    P.base[i >> 6] = seg[b0];
    if (len > 0xffff) st->too_long = 1;
  }
  if (i == 0) P.base[(size_t)P.blocks * P.nseg] = nnz;
}

// What a wave does with 64 rows of a segment takes the longest row's share of each
// chunk, added up by one lane (kPcAddNs an entry, in fours), and the chunks after the
// first, whose loads are waited for (kPcChunkNs each).  cost[seg blocks + b]: that sum.
constexpr float kPcAddNs = 45.f, kPcChunkNs = 1100.f;
__global__ __launch_bounds__(kBlock) void pc_cost_kernel(SpPieces P, float *cost) {
  const int lane = threadIdx.x & 63;
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
  if (i >= (int64_t)P.blocks * P.nseg) return;
  const int begin = P.base[i], ke = P.base[i + 1], lo = P.off[i * 64 + lane];
  const int next = __shfl_down(lo, 1), from = begin + lo, hi = lane == 63 ? ke : begin + next;
  int adds = 0, chunks = 0;
  for (int k = begin & ~3; k < ke; k += kPcChunk, ++chunks) {
    int run = max(0, min(hi - k, kPcChunk) - max(from - k, 0));
    for (int o = 32; o > 0; o >>= 1) run = max(run, __shfl_xor(run, o));
    adds += (run + 3) & ~3;
  }
  if (lane == 0) cost[i] = kPcAddNs * (float)adds + kPcChunkNs * (float)max(chunks - 1, 0);
}

// The longest workgroup: a barrier per segment, each wave its blocks of the tile.
__global__ __launch_bounds__(64) void pc_worst_kernel(SpPieces P, const float *cost, PcStats *st) {
  const int grp = blockIdx.x % P.groups, tile = blockIdx.x / P.groups, w = threadIdx.x & 15, g0 = threadIdx.x >> 4;
  const int per = (P.nseg + P.groups - 1) / P.groups;
  const int sg0 = min(P.nseg, grp * per), sg1 = min(P.nseg, sg0 + per);
  const int r0 = tile * P.tile, r1 = min(P.rows, r0 + P.tile);
  float t = 0.f;
  for (int sg = sg0; sg < sg1; ++sg) {
    float v = 0.f;
    for (int g = g0; g < kPcRpl; g += 4) {
      const int row = r0 + (g * kPcWaves + w) * 64;
      if (row < r1) v += cost[(size_t)sg * P.blocks + (row >> 6)];
    }
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    for (int o = 8; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    t += v;
  }
  if (threadIdx.x == 0) atomicMax((unsigned *)&st->worst_ns, __float_as_uint(t));  // not negative: ordered as its bits
}

__global__ __launch_bounds__(kPcPad) void pc_pad_kernel(SpPieces P, int64_t nnz) {
  P.va[nnz + threadIdx.x] = 0.f;
  P.ci[nnz + threadIdx.x] = 0;
}
__global__ __launch_bounds__(kBlock) void pc_zero_kernel(int *v, int64_t len) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < len; i += (int64_t)gridDim.x * kBlock) v[i] = 0;
}

}  // namespace

// Where the pieces are faster (CG step of the plain passes -> in pieces, us):
//  - at least a million entries, so that the pass is bound by them:
//    200000 x 50000, 6 a row: 31.6 -> 29.1; 2000000 x 200000, 16 a row: 500 -> 180;
//  - at least 6 of a workgroup's 16 waves with rows of their own:
//    100000 x 25000, 10 a row (7 and 12 waves): 31.1 -> 26.5;
//    100000 x 10000, 20 a row (7 and 5): 40.7 -> 41.6;
//  - at least one entry per row and segment, or the row bounds outweigh them:
//    500000 x 125000, 9 a row (2.3): 84.7 -> 49.7;
//    1000000 x 250000, 6 a row (0.75): 95.7 -> 94.9 and the first pass 103 -> 125;
// and where pieces_pay says so.
bool pieces_shape(int64_t rows, int64_t cols, int64_t nnz, int groups, SpPieces *P) {
  *P = SpPieces{};
  int64_t nseg = round_up(cdiv(cols, (int64_t)kPcSeg), groups);
  const int64_t seg = round_up(cdiv(cols, nseg), 64);
  nseg = cdiv(cols, seg);
  const int64_t wgs = kPcWg / groups, rounds = cdiv(rows, wgs * kPcTile);
  if (nnz < ((int64_t)1 << 20) || rows < wgs * 64 * 6 || nnz < rows * nseg) return false;
  if (rows >= (1LL << 30) || cols >= (1LL << 30) || (rows + 63) * nseg >= (1LL << 31) - 1 || nnz >= (1LL << 31) - kPcPad - 1) return false;
  P->rows = (int)rows;
  P->blocks = (int)cdiv(rows, (int64_t)64);
  P->cols = (int)cols;
  P->seg = (int)seg;
  P->nseg = (int)nseg;
  P->tile = (int)round_up(cdiv(rows, wgs * rounds), 64);
  P->tiles = (int)cdiv(rows, (int64_t)P->tile);
  P->groups = groups;
  return true;
}

// A row belongs to one lane, so dense rows, long rows and rows of unlike lengths
// side by side leave most lanes of a wave, or most workgroups, without work: the
// pass takes what its longest workgroup takes (pc_cost_kernel, from the matrix's own
// bounds), or its entries' loads.  The plain passes give a row lpr lanes and
// deal rows out evenly; they take their entries' gathers, or the longest row's
// chain of them (an estimate that is low where many rows are long).  CG steps, us, plain /
// pieces -> chosen:
//    200000 x 20000, 24 entries a row 68 / 50, 48: 121 / 117, 100: 272 / 368, 200: 502 / 1202
//      -> pieces up to 48;
//    1000000 x 20000, 32 a row 463 / 299, 64: 893 / 867 with 1000 / 1428 for the
//      first pass (A^T twice) -> pieces at 32: A^T counts 1.2 times;
//    column frequencies 1 / (rank + 100), frequent ones side by side, 300000 x 30000
//      105 / 1976, 2000000 x 200000 2253 / 12006 -> plain; the same columns
//      in random order 120 / 125 and 2400 / 736 -> pieces for the larger;
//    rows sorted by length 1 / (rank + 1000), 2000000 x 200000: 730 / 26996 -> plain;
//    a full column, 300000 x 30000 (64 lanes a row) 2150 / 1731 -> plain, 500000 x
//      125000 11545 / 2868, 2000000 x 200000 56100 / 11730 (16 lanes) -> pieces.
bool pieces_pay(const PcStats &a, const PcStats &at, int lpr, int lprt, int64_t nnz) {
  if (a.too_long || at.too_long) return false;
  constexpr double kLoadNs = 0.0025, kGatherNs = 0.007, kChainNs = 440.0;  // per entry, entry, turn of a row's lanes
  auto pieces = [&](const PcStats &s) { return std::max(kLoadNs * (double)nnz, (double)s.worst_ns); };
  auto plain = [&](const PcStats &s, int l) { return std::max(kGatherNs * (double)nnz, kChainNs * (double)s.longest / l); };
  return pieces(a) + 1.2 * pieces(at) < plain(a, lpr) + plain(at, lprt);
}

int64_t pieces_sums(const SpPieces &P) { return cdiv((int64_t)P.rows * P.nseg, (int64_t)kScanBlock); }

void count_pieces(const Csr<float> &A, const SpPieces &P, int64_t nnz, int *rp, int *cur, int *sums, float *cost,
                  PcStats *st, hipStream_t s) {
  const int64_t len = (int64_t)P.rows * P.nseg, blocks = pieces_sums(P);
  const dim3 b(kBlock);
  hipLaunchKernelGGL(pc_zero_kernel, dim3(1024), b, 0, s, rp, len + 1);
  hipLaunchKernelGGL(pc_count_kernel, dim3(cdiv(A.rows, kPcCountThreads)), dim3(kPcCountThreads), 0, s, A, P, rp, st);
  hipLaunchKernelGGL(pc_block_sums_kernel, dim3(blocks), b, 0, s, (const int *)rp, len, sums);
  hipLaunchKernelGGL(pc_scan_sums_kernel, dim3(1), b, 0, s, sums, blocks);
  hipLaunchKernelGGL(pc_scan_kernel, dim3(blocks), b, 0, s, rp, cur, len, (const int *)sums, (int)nnz);
  const dim3 per_row(cdiv((int64_t)P.blocks * 64 * P.nseg, (int64_t)kBlock));
  hipLaunchKernelGGL(pc_bounds_kernel, per_row, b, 0, s, (const int *)rp, P, (int)nnz, st);
  hipLaunchKernelGGL(pc_cost_kernel, per_row, b, 0, s, P, cost);
  hipLaunchKernelGGL(pc_worst_kernel, dim3(P.tiles * P.groups), dim3(64), 0, s, P, (const float *)cost, st);
}

void fill_pieces(const Csr<float> &A, const SpPieces &P, int64_t nnz, int *cur, hipStream_t s) {
  hipLaunchKernelGGL(pc_scatter_kernel, dim3(cdiv(A.rows, kBlock)), dim3(kBlock), 0, s, A, P, cur);
  hipLaunchKernelGGL(pc_pad_kernel, dim3(1), dim3(kPcPad), 0, s, P, nnz);
}

int pieces_finish_blocks(int n) { return (int)cdiv(n, kBlock); }

void launch_pc_first(const IterArgs<float> &p, int ncolp, hipStream_t s) {
  hipLaunchKernelGGL(pc_start_kernel, dim3(p.pa.tiles), dim3(kPcThreads), 0, s, p);
  hipLaunchKernelGGL(pc_first_kernel, dim3(p.pat.tiles * p.pat.groups, 2), dim3(kPcThreads), 0, s, p, ncolp);
  hipLaunchKernelGGL(pc_first_finish_kernel, dim3(pieces_finish_blocks(p.n)), dim3(kBlock), 0, s, p, ncolp);
}

void launch_pc_rows(const IterArgs<float> &p, int j, int cap, hipStream_t s) {
  hipLaunchKernelGGL(pc_rows_kernel, dim3(p.pa.tiles), dim3(kPcThreads), 0, s, p, j, cap);
}

void launch_pc_step(const IterArgs<float> &p, int j, int cap, int ncolp, hipStream_t s) {
  launch_pc_rows(p, j, cap, s);
  hipLaunchKernelGGL(pc_residual_kernel, dim3(std::min<int64_t>(512, cdiv(p.m, 4 * kBlock))), dim3(kBlock), 0, s, p, j);
  hipLaunchKernelGGL(pc_step_kernel, dim3(p.pat.tiles * p.pat.groups), dim3(kPcThreads), 0, s, p, ncolp);
  hipLaunchKernelGGL(pc_step_finish_kernel, dim3(pieces_finish_blocks(p.n)), dim3(kBlock), 0, s, p, j, ncolp);
}

}  // namespace pogs

// Launches of the resident solve (resident.hpp) and the rule for the shapes
// that take it.
#include "resident.hpp"

#include <atomic>

namespace pogs {

template <typename T, int NC, int RPW>
__global__ __launch_bounds__(kResThreads) void resident_kernel(ResArgs<T> p) {
  extern __shared__ __align__(16) char smem[];
  resident_body<T, NC, RPW>(p, smem);
}

// The kernels: 16-byte pieces per lane and row, rows per wave.  A wave keeps at
// most 20 pieces of M per lane (80 registers of the 256 that two waves per SIMD
// leave each); a workgroup has a CU to itself.
#define POGS_RES_SHAPES_F32(X) X(1, 4) X(1, 10) X(1, 20) X(2, 4) X(2, 10) X(4, 2) X(4, 5)
#define POGS_RES_SHAPES_F64(X) X(1, 4) X(1, 10) X(1, 16) X(2, 4) X(2, 8) X(4, 2) X(4, 4) X(6, 3) X(8, 2)

int res_capacity() {
  static std::atomic<int> cus{0};  // the same for every device of a process
  int n = cus.load(std::memory_order_relaxed), dev = 0;
  if (!n) {
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      n = 0;
    cus.store(n, std::memory_order_relaxed);
  }
  return std::min(n, 256);
}

// Streams restricted to some CUs never run resident launches: two of them can
// overlap, so what fits together is not known, and waiting it out takes 7 ms of
// a 2 ms solve (8000 x 1000 on half the CUs: 9.0 ms, with one launch per step 2.1).
bool res_all_cus(hipStream_t s) {
  uint32_t mask[32] = {};
  if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  int n = 0;
  for (uint32_t w : mask) n += __builtin_popcount(w);
  return n >= res_capacity();
}

// Shapes taken: those whose rows fit the registers of the CUs (20 MB of matrix at
// half the CUs, 40 MB at all of them) and have up to 1024 entries.  The registers
// would hold longer ones (2000 x 2000 float32 is 16 MB), but the eight waves' float64
// column sums of a workgroup take 16 bytes an entry and wave of LDS
// (ResShape::red_bytes), 128 of its 160 KB at 1024.  Of the
// kernels for a row length the first that needs at most 128 workgroups, else the
// one with the most rows: fewer, fuller workgroups cost rows per wave, more of
// them cost exchange words (us per iteration, one launch per step / RPW and G:
// 1999 x 503 f32 29.7 / 13.3 at 10 rows and 25 workgroups, 11.4 at 4 and 63;
// 1000 x 1000 27.0 / 15.5 at 5 and 25, 13.5 at 2 and 125; 4000 x 1000 28.0 / 15.7 at
// 5 and 100, 16.4 at 2 and 250).  It is taken wherever it fits: from 23.0 -> 9.1
// at 100 x 50 to 31.1 -> 15.5 at 20000 x 450 and 31.2 -> 17.4 at 8000 x 1000.
ResGeom res_geometry(int64_t m, int64_t n, int es) {
  constexpr int64_t kTarget = 128;
  ResGeom r;
  const int64_t L = std::max(m, n), q = std::min(m, n), ld = round_up(q, 64), most = res_capacity();
  const int64_t lanes = kWave * (16 / es);  // elements one piece per lane covers
  auto consider = [&](int pieces, int rpw, int cols) {
    if (lanes * pieces < ld || (r.G && (r.pieces < pieces || r.G <= kTarget))) return;
    const int64_t G = std::max(cdiv(L, (int64_t)kResWaves * rpw), cdiv(q, (int64_t)cols));
    if (G > most) return;
    r.G = (int)G;
    r.pieces = pieces;
    r.rpw = rpw;
    r.nc = (int)cdiv(q, G);
  };
#define POGS_RES_TRY(NC, RPW) consider(NC, RPW, es == 4 ? ResShape<float, NC, RPW>::cols : ResShape<double, NC, RPW>::cols);
  if (es == 4) {
    POGS_RES_SHAPES_F32(POGS_RES_TRY)
  } else {
    POGS_RES_SHAPES_F64(POGS_RES_TRY)
  }
#undef POGS_RES_TRY
  return r;
}

size_t res_exchange_bytes(const ResGeom &r, int es) {
  const size_t w = es == 4 ? 2 * res_words1<float>(r.G, r.nc) + res_words2<float>(r.G, r.nc) + res_words3<float>(r.G, r.nc)
                           : 2 * res_words1<double>(r.G, r.nc) + res_words2<double>(r.G, r.nc) + res_words3<double>(r.G, r.nc);
  return w * sizeof(ResWord);
}

template <typename T, int NC, int RPW> static int launch_res(const ResArgs<T> &a, hipStream_t s) {
  const int lds = (int)ResShape<T, NC, RPW>::lds_bytes(a.G);
  if (lds > 64 * 1024)
    POGS_HIP_TRY(hipFuncSetAttribute((const void *)resident_kernel<T, NC, RPW>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
  hipLaunchKernelGGL((resident_kernel<T, NC, RPW>), dim3(a.G), dim3(kResThreads), lds, s, a);
  POGS_HIP_TRY(hipGetLastError());
  return POGS_OK;
}

template <typename T>
int launch_resident(const IterArgs<T> &p, const ResGeom &r, const T *M, void *xbuf, ResHost *host, int first, int iters,
                    unsigned polls, hipStream_t s) {
  const bool wide = p.m < p.n;
  ResArgs<T> a{};
  a.L = wide ? p.n : p.m;
  a.q = p.q;
  a.ld = p.ldk;
  a.G = r.G;
  a.nc = r.nc;
  a.wide = wide ? 1 : 0;
  a.M = M;
  a.Kinv = p.Kinv;
  a.fl = wide ? p.g : p.f;
  a.fs = wide ? p.f : p.g;
  a.lv = wide ? p.x : p.y;
  a.lvt = wide ? p.xt : p.yt;
  a.lh = wide ? p.xh : p.yh;
  a.ldu = wide ? p.mu : p.nu;
  a.lp = wide ? p.cx : p.dy;
  a.sv = wide ? p.y : p.x;
  a.svt = wide ? p.yt : p.xt;
  a.sh = wide ? p.yh : p.xh;
  a.sdu = wide ? p.nu : p.mu;
  a.ctrl = p.ctrl;
  a.host = host;
  ResWord *x = (ResWord *)xbuf;
  a.x1[0] = x;
  a.x1[1] = a.x1[0] + res_words1<T>(r.G, r.nc);
  a.x2 = a.x1[1] + res_words1<T>(r.G, r.nc);
  a.x3 = a.x2 + res_words2<T>(r.G, r.nc);
  a.first = first;
  a.iters = iters;
  a.polls = polls;
#define POGS_RES_LAUNCH(NC, RPW) \
  if (r.pieces == NC && r.rpw == RPW) return launch_res<T, NC, RPW>(a, s);
  if constexpr (sizeof(T) == 4) {
    POGS_RES_SHAPES_F32(POGS_RES_LAUNCH)
  } else {
    POGS_RES_SHAPES_F64(POGS_RES_LAUNCH)
  }
#undef POGS_RES_LAUNCH
  return POGS_EDEVICE;
}

template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *A, int m, int n, int ld, T *At, int ldt) {
  __shared__ T tile[64][65];
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64, tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int k = ty; k < 64; k += 4)
    tile[k][tx] = r0 + k < m && c0 + tx < n ? A[(size_t)(r0 + k) * ld + c0 + tx] : T(0);
  __syncthreads();
  for (int k = ty; k < 64; k += 4)
    if (c0 + k < n) At[(size_t)(c0 + k) * ldt + r0 + tx] = tile[tx][k];  // r0 + tx < ldt = m rounded up to 64
}

template <typename T> void launch_transpose(const T *A, int m, int n, int ld, T *At, int ldt, hipStream_t s) {
  hipLaunchKernelGGL(transpose_kernel<T>, dim3(cdiv(m, 64), cdiv(n, 64)), dim3(256), 0, s, A, m, n, ld, At, ldt);
}

#define POGS_INST(T)                                                                                              \
  template int launch_resident<T>(const IterArgs<T> &, const ResGeom &, const T *, void *, ResHost *, int, int,   \
                                  unsigned, hipStream_t);                                                         \
  template void launch_transpose<T>(const T *, int, int, int, T *, int, hipStream_t);
POGS_INST(float)
POGS_INST(double)
#undef POGS_INST

}  // namespace pogs

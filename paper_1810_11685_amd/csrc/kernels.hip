// Launch side of the row and column passes (device code in passes.hpp, one
// translation unit per compile-time line length in passes<length>.hip) and the
// small kernels around them: sensor data, sound-speed gradient, reductions,
// output check.
#include "passes.hpp"
#include "passes_len.hpp"

#include <map>
#include <mutex>

namespace qpat {

// ---------------------------------------------------------------- sensor data
__global__ void combine_kernel(const Item* __restrict__ items, const IO* __restrict__ io) {
  const Medium& M = items[blockIdx.y].m;
  const float* part = items[blockIdx.y].w.part;
  float* out = io[blockIdx.y].out;
  const int total = M.nt * M.ns;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x)
    out[i] = part[2 * i] + part[2 * i + 1];
}

// Residual samples in sensor-tap order, rtap[m][e] = r[m][s(e)] for the 2 ns
// taps e (the adjoint row passes read one contiguous run per tile).  Written
// into the vector's sensor-partial buffer, which the adjoint does not use.
__global__ void tap_order_kernel(const Item* __restrict__ items, const IO* __restrict__ io) {
  const Medium& M = items[blockIdx.y].m;
  float* dst = items[blockIdx.y].w.part;
  const float* r = io[blockIdx.y].in;
  const int ntap = 2 * M.ns, total = M.nt * ntap;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int m = i / ntap, e = i - m * ntap;
    dst[i] = r[unsigned(m) * unsigned(M.ns) + M.taps[e].s];
  }
}

// ---------------------------------------------------------------- sound-speed gradient
// d<r, H_a p0>/dc = sum_m p*^m dp^m/dc (the equation-of-state part, gc) minus
// (2/c) p0 H_a^* r (the source of eq s1 scales as 1/c^2).
__global__ void __launch_bounds__(kBlock) grad_c_kernel(const float* __restrict__ c2, const float* __restrict__ p0,
                                                        const float* __restrict__ g0, const double* __restrict__ gc,
                                                        long long n, long long gc_stride, float* __restrict__ out) {
  const long long b = blockIdx.y;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const double c = sqrt(double(c2[i]));
    out[b * n + i] = float(gc[b * gc_stride + i] - 2.0 * double(p0[b * n + i]) * double(g0[b * n + i]) / c);
  }
}

// ---------------------------------------------------------------- reductions
__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__global__ void __launch_bounds__(kBlock) dot_partial(const float* __restrict__ a, const float* __restrict__ b,
                                                      int64_t n, double* __restrict__ partial) {
  __shared__ double red[kBlock / 64];
  double acc = 0.0;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    acc += double(a[i]) * double(b[i]);
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += red[w];
    partial[blockIdx.x] = s;
  }
}

__global__ void __launch_bounds__(kBlock) dot_final(const double* __restrict__ partial, int nblk,
                                                    double* __restrict__ out) {
  __shared__ double red[kBlock / 64];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) acc += partial[i];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) s += red[w];
    *out = s;
  }
}

// ---------------------------------------------------------------- launchers
// Launches pick the kernel instance for their row / column length (lengths
// with a compile-time plan): uniform launches by the plan's length, table
// launches by the length all their items share (`len`, 0 when they differ).
// The instances without a length: for table launches over several, which hold
// them all, and for uniform launches of the short ones (8 to 24).
template <int MODE>
static hipError_t launch_row_any(const Launch& L, bool uniform, int ntile, int chunk, int nblocks, int threads,
                                 size_t lds, int n, int flags, hipStream_t st) {
  const dim3 g(nblocks), t(threads);
  if (uniform) hipLaunchKernelGGL((row_kernel<MODE, true, 0>), g, t, lds, st, L, ntile, chunk, n, flags);
  else hipLaunchKernelGGL((row_kernel<MODE, false, 0>), g, t, lds, st, L, ntile, chunk, n, flags);
  return hipGetLastError();
}

hipError_t launch_row(int mode, const Launch& L, bool uniform, int len, bool tg, int ntile, int chunk, int nblocks,
                      int threads, size_t lds, int n, int flags, hipStream_t st) {
  if (tg && !uniform) return hipErrorInvalidValue;
  const LaunchKind kind = !uniform ? LK_TABLE : tg ? LK_UNIFORM_TG : LK_UNIFORM;
#define QPAT_LEN_CASE(N) \
  case N: return launch_row_len<N>(mode, kind, L, ntile, chunk, nblocks, threads, lds, n, flags, st);
  switch (uniform ? L.m.nx : len) {
    QPAT_FOR_LENGTHS(QPAT_LEN_CASE)
    default: break;
  }
#undef QPAT_LEN_CASE
  if (tg) return hipErrorInvalidValue;  // global-twiddle instances exist for the lengths above only
#define QPAT_ROW_CASE(m) \
  case m: return launch_row_any<m>(L, uniform, ntile, chunk, nblocks, threads, lds, n, flags, st);
  switch (mode) {
    QPAT_ROW_CASE(RM_F1)
    QPAT_ROW_CASE(RM_F2)
    QPAT_ROW_CASE(RM_F2L)
    QPAT_ROW_CASE(RM_F3)
    QPAT_ROW_CASE(RM_A1)
    QPAT_ROW_CASE(RM_A1L)
    QPAT_ROW_CASE(RM_A2)
    QPAT_ROW_CASE(RM_A3)
    QPAT_ROW_CASE(RM_FWD1)
    QPAT_ROW_CASE(RM_INV1)
    QPAT_ROW_CASE(RM_F2L | RM_X)
    QPAT_ROW_CASE(RM_F3 | RM_X)
    QPAT_ROW_CASE(RM_A1 | RM_X)
    QPAT_ROW_CASE(RM_A1L | RM_X)
    default: return hipErrorInvalidValue;
  }
#undef QPAT_ROW_CASE
}

template <int CM>
static hipError_t launch_col_any(int mcode, const Launch& L, bool uniform, int ntile, int chunk, int nblocks,
                                 int threads, size_t lds, int n, hipStream_t st) {
  const dim3 g(nblocks), t(threads);
  if (uniform) hipLaunchKernelGGL((col_kernel<true, CM, 0>), g, t, lds, st, L, ntile, chunk, mcode, n);
  else hipLaunchKernelGGL((col_kernel<false, CM, 0>), g, t, lds, st, L, ntile, chunk, mcode, n);
  return hipGetLastError();
}

hipError_t launch_col(int cm, int mcode, const Launch& L, bool uniform, int len, bool tg, int ntile, int chunk,
                      int nblocks, int threads, size_t lds, int n, hipStream_t st) {
  if (tg && !uniform) return hipErrorInvalidValue;
  const LaunchKind kind = !uniform ? LK_TABLE : tg ? LK_UNIFORM_TG : LK_UNIFORM;
#define QPAT_LEN_CASE(N) \
  case N: return launch_col_len<N>(cm, kind, mcode, L, ntile, chunk, nblocks, threads, lds, n, st);
  switch (uniform ? L.m.ny : len) {
    QPAT_FOR_LENGTHS(QPAT_LEN_CASE)
    default: break;
  }
#undef QPAT_LEN_CASE
  if (tg) return hipErrorInvalidValue;
#define QPAT_COL_MODE(c) \
  case c: return launch_col_any<c>(mcode, L, uniform, ntile, chunk, nblocks, threads, lds, n, st);
  switch (cm) {
    QPAT_COL_MODE(CM_GRADP1)
    QPAT_COL_MODE(CM_GRADM2)
    QPAT_COL_MODE(CM_FRAC)
    QPAT_COL_MODE(CM_GRADP2)
    QPAT_COL_MODE(CM_DIVM)
    QPAT_COL_MODE(CM_APPLY)
    default: return hipErrorInvalidValue;
  }
#undef QPAT_COL_MODE
}

bool kernels_row_fused(int n, bool tg) {
#define QPAT_HAVE(N) if (n == N) return row_fused_len<N>(tg);
  QPAT_FOR_LENGTHS(QPAT_HAVE)
#undef QPAT_HAVE
  return false;
}

bool kernels_have_length(int n) {
#define QPAT_HAVE(N) if (n == N) return true;
  QPAT_FOR_LENGTHS(QPAT_HAVE)
#undef QPAT_HAVE
  return false;
}

// Let the pass kernels that grids of nx x ny can launch (their lengths' own
// instances and the all-length ones) use up to `bytes` of dynamic LDS.
template <typename K>
static hipError_t allow_fn(K* k, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(bytes));
}
template <int MODE>
static hipError_t allow_row(size_t bytes) {
  const hipError_t e = allow_fn(&row_kernel<MODE, false, 0>, bytes);
  return e != hipSuccess ? e : allow_fn(&row_kernel<MODE, true, 0>, bytes);
}
template <int CM>
static hipError_t allow_col(size_t bytes) {
  const hipError_t e = allow_fn(&col_kernel<false, CM, 0>, bytes);
  return e != hipSuccess ? e : allow_fn(&col_kernel<true, CM, 0>, bytes);
}

hipError_t kernels_allow_lds(int nx, int ny, size_t bytes) {
#define QPAT_ALLOW(N)                                            \
  if (nx == N) {                                                 \
    const hipError_t e = allow_lds_len<N>(false, bytes);         \
    if (e != hipSuccess) return e;                               \
  }                                                              \
  if (ny == N) {                                                 \
    const hipError_t e = allow_lds_len<N>(true, bytes);          \
    if (e != hipSuccess) return e;                               \
  }
  QPAT_FOR_LENGTHS(QPAT_ALLOW)
#undef QPAT_ALLOW
  const hipError_t es[] = {allow_row<RM_F1>(bytes),      allow_row<RM_F2>(bytes),     allow_row<RM_F2L>(bytes),
                           allow_row<RM_F3>(bytes),      allow_row<RM_A1>(bytes),     allow_row<RM_A1L>(bytes),
                           allow_row<RM_A2>(bytes),      allow_row<RM_A3>(bytes),     allow_row<RM_FWD1>(bytes),
                           allow_row<RM_INV1>(bytes),    allow_row<RM_F2L | RM_X>(bytes), allow_row<RM_F3 | RM_X>(bytes),
                           allow_row<RM_A1 | RM_X>(bytes), allow_row<RM_A1L | RM_X>(bytes),
                           allow_col<CM_GRADP1>(bytes), allow_col<CM_GRADM2>(bytes),
                           allow_col<CM_FRAC>(bytes),    allow_col<CM_GRADP2>(bytes), allow_col<CM_DIVM>(bytes),
                           allow_col<CM_APPLY>(bytes)};
  for (hipError_t e : es)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_combine(const Item* items, const IO* io, int nitems, int max_count, hipStream_t st) {
  int bx = (max_count + kBlock - 1) / kBlock;
  if (bx > 1024) bx = 1024;
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(combine_kernel, dim3(bx, nitems), dim3(kBlock), 0, st, items, io);
  return hipGetLastError();
}

hipError_t launch_tap_order(const Item* items, const IO* io, int nitems, int max_count, hipStream_t st) {
  int bx = (max_count + kBlock - 1) / kBlock;
  if (bx > 1024) bx = 1024;
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(tap_order_kernel, dim3(bx, nitems), dim3(kBlock), 0, st, items, io);
  return hipGetLastError();
}

hipError_t launch_grad_c(const float* c2, const float* p0, const float* g0, const double* gc, long long n,
                         int batch, long long gc_stride, float* out, hipStream_t st) {
  long long bx = (n + kBlock - 1) / kBlock;
  if (bx > 1024) bx = 1024;
  hipLaunchKernelGGL(grad_c_kernel, dim3(unsigned(bx), unsigned(batch)), dim3(kBlock), 0, st, c2, p0, g0, gc, n,
                     gc_stride, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- output check
// flag <- 1 if any of x[0 .. n) is NaN or infinite (every writer stores the
// same value, so no atomics are needed; the host clears the flag).
__global__ void __launch_bounds__(kBlock) finite_kernel(const float* __restrict__ x, int64_t n, int* flag) {
  bool bad = false;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
    bad |= !isfinite(x[i]);
  if (bad) *flag = 1;
}

hipError_t launch_finite(const float* x, int64_t n, int* flag, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t want = (n + kBlock - 1) / kBlock;
  const int nblk = int(want < 1024 ? want : 1024);
  hipLaunchKernelGGL(finite_kernel, dim3(nblk), dim3(kBlock), 0, st, x, n, flag);
  return hipGetLastError();
}

// Partial sums of qpat_dot_noalloc: a static array that every device the
// library runs on holds until the process ends, shared by all calls on that
// device.  Host code never passes the array's name to a kernel; it uses the
// device address looked up once per device below.
static __device__ __align__(256) double scratch[kDotBlocks];

hipError_t dot_scratch(double** ptr) {
  static std::mutex mu;
  static std::map<int, double*> addr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> g(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    double* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    it = addr.emplace(dev, p).first;
  }
  *ptr = it->second;
  return hipSuccess;
}

hipError_t launch_dot(const float* a, const float* b, int64_t n, double* partial, int nblk, double* out,
                      hipStream_t st) {
  hipLaunchKernelGGL(dot_partial, dim3(nblk), dim3(kBlock), 0, st, a, b, n, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(dot_final, dim3(1), dim3(kBlock), 0, st, partial, nblk, out);
  return hipGetLastError();
}

}  // namespace qpat

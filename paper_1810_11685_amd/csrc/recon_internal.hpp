// Internal interface of the TV priorconditioner kernels (recon.hip) and their
// host side (recon.cpp).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "cg_mg.hpp"

namespace qpat {

constexpr int kRedThreads = 256;  // threads per block of the TV / CG kernels
constexpr int kRedBlocks = 256;   // blocks per field (fixed: the reductions run in a fixed order)

// One level of the multigrid preconditioner of the CG solve, [batch][ny][nx]
// fields of fs values.  Level 0 is the grid itself (its diagonal term is the
// number gamma, its b the right-hand side); level l + 1 aggregates 2 x 2 blocks
// of level l.
struct MgLevel {
  int nx, ny, pitch;           // row stride of the operator's arrays
  size_t fs;
  int uniform;                 // the diagonal term is gamma everywhere
  double gamma;
  double *g, *wh, *wv, *dinv;  // operator: diagonal (gamma) term, edge weights, inverse diagonal
  double *b, *t;               // right-hand side, post-smoothed iterate
};

// That operator, for the solver of cg_mg.hpp.
struct TvOp {
  using Level = MgLevel;
  static constexpr int kArrays = 4;
  static __host__ __device__ double*& array(Level& L, int a) {
    return a == 0 ? L.g : a == 1 ? L.wh : a == 2 ? L.wv : L.dinv;
  }
  static __host__ __device__ double* array(const Level& L, int a) {
    return a == 0 ? L.g : a == 1 ? L.wh : a == 2 ? L.wv : L.dinv;
  }
  struct Coef {
    double g, e, w, n, s;
  };
  // diagonal term and edges of node (j, i); 0 where there is no neighbour
  static __device__ __forceinline__ Coef coef(const Level& L, size_t base, int i, int j) {
    const size_t k = base + size_t(j) * L.nx + i;
    const bool W = i > 0, S = j > 0;
    Coef C{L.uniform ? L.gamma : L.g[k], L.wh[k], L.wh[W ? k - 1 : k], L.wv[k], L.wv[S ? k - L.nx : k]};
    if (!W) C.w = 0.0;
    if (!S) C.s = 0.0;
    return C;
  }
  // at position k of arrays (m values each, rows of w) whose rings are 0
  static __device__ __forceinline__ Coef ringed(const double* a, int m, int k, int w) {
    const double *wh = a + m, *wv = wh + m;
    return Coef{a[k], wh[k], wh[k - 1], wv[k], wv[k - w]};
  }
  static __device__ __forceinline__ double product(const Coef& C, double c, double e, double w, double n, double s,
                                                   double, double) {
    return C.g * c + C.e * (c - e) + C.w * (c - w) + C.n * (c - n) + C.s * (c - s);
  }
  // coarse operator at node k: the aggregate's diagonal terms and the fine edges
  // between two aggregates (to the west and south also, for the diagonal)
  static __device__ __forceinline__ void coarsen(const Level& f, size_t bf, const Level& c, size_t bc, int k) {
    const int J = k / c.nx, I = k - J * c.nx, j0 = 2 * J, i0 = 2 * I;
    const size_t o = bc + size_t(J) * c.pitch + I;
    double g = 0.0;
    for (int j = j0; j < j0 + 2 && j < f.ny; ++j)
      for (int i = i0; i < i0 + 2 && i < f.nx; ++i) g += f.uniform ? f.gamma : f.g[bf + size_t(j) * f.pitch + i];
    auto column = [&](int i) {   // edges (j, i)-(j, i + 1) of the aggregate's rows
      double h = 0.0;
      for (int j = j0; j < j0 + 2 && j < f.ny; ++j) h += f.wh[bf + size_t(j) * f.pitch + i];
      return h;
    };
    auto row = [&](int j) {
      double v = 0.0;
      for (int i = i0; i < i0 + 2 && i < f.nx; ++i) v += f.wv[bf + size_t(j) * f.pitch + i];
      return v;
    };
    const double h = I + 1 < c.nx ? column(i0 + 1) : 0.0, v = J + 1 < c.ny ? row(j0 + 1) : 0.0;
    double d = g;
    if (I + 1 < c.nx) d += h;
    if (I > 0) d += column(i0 - 1);
    if (J + 1 < c.ny) d += v;
    if (J > 0) d += row(j0 - 1);
    c.g[o] = g;
    c.wh[o] = h;
    c.wv[o] = v;
    c.dinv[o] = 1.0 / d;
  }
};
using TvLevels = cgmg::Levels<TvOp>;

hipError_t launch_tv_weights(const float* x, int nx, int ny, int batch, double beta, double* wh, double* wv,
                             hipStream_t st);
hipError_t launch_tv_apply(const float* x, float* y, const double* wh, const double* wv, int nx, int ny, int batch,
                           double gamma, hipStream_t st);
hipError_t launch_tv_value(const float* x, int nx, int ny, int batch, double beta, double* part, hipStream_t st);
// Inverse diagonal of level 0 and operators of the others, for the levels' gamma.
hipError_t launch_mg_setup(const TvLevels& L, int batch, hipStream_t st);
hipError_t launch_cg_start(const float* rhs, const cgmg::Vectors& c, const TvLevels& L, hipStream_t st);
hipError_t launch_cg_iteration(const cgmg::Vectors& c, const TvLevels& L, int par, double tol2, hipStream_t st);
hipError_t launch_cg_finish(const cgmg::Vectors& c, float* out, size_t n, hipStream_t st);
hipError_t tv_allow_lds();
hipError_t launch_axpby(int64_t n, float a, const float* x, float b, float* y, hipStream_t st);

// PCG of Algorithm 4 with device scalars, `batch` fields of n values:
// out[f * ostride] = scale * a_f . b_f (FP64; part holds [batch][kRedBlocks]);
// live / done flags of iteration i; the alpha step; the beta direction update;
// x += sol for the flagged fields.
hipError_t launch_ld_dots(const float* a, const float* b, size_t n, int batch, double* part, double* out,
                          int ostride, double scale, hipStream_t st);
hipError_t launch_ld_live(int batch, const double* rz, int rzs, int i, int i_max, int i_m, double tol_in, int* done,
                          int* live, hipStream_t st);
hipError_t launch_ld_step(size_t n, int batch, const double* rz, int rzs, int i, const double* dhd, const int* live,
                          const float* d, const float* hd, float* sol, float* r, hipStream_t st);
hipError_t launch_ld_dir(size_t n, int batch, const double* rz, int rzs, int i, const int* live, const float* z,
                         float* d, hipStream_t st);
hipError_t launch_ld_add(size_t n, int batch, const int* flag, const float* sol, float* x, hipStream_t st);
// hsol += alpha_i jd per live data set, alpha_i = rz_i / dhd (the step of launch_ld_step on data vectors)
hipError_t launch_ld_data_step(size_t nd, int batch, const double* rz, int rzs, int i, const double* dhd,
                               const int* live, const float* jd, float* hsol, hipStream_t st);

}  // namespace qpat

// Internal structures of the optical operators (optical.hip, optical.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "cg_mg.hpp"

namespace qpat {

constexpr int kOptThreads = 256;  // threads per block of the optical kernels
constexpr int kOptBlocks = 256;   // most blocks per field (a fixed count per mesh: deterministic reductions)

// One level of the multigrid preconditioner of the CG solve, on the node
// grid ([batch][ny][nx] fields, fs values a field; level 0 is the mesh's
// (ny + 1) x (nx + 1) nodes, level l + 1 aggregates 2 x 2 nodes of level l).
// The operator is a symmetric 7-point stencil: diagonal and the couplings to
// the east, north and north-east neighbours (the mesh diagonals run south-west
// to north-east, and 2 x 2 aggregation keeps that pattern).  Level 0's b is the
// right-hand side.
struct OptLevel {
  int nx, ny, pitch;   // row stride of the stencil arrays
  size_t fs;
  double *sc, *se, *sn, *sd, *dinv;  // stencil and inverse diagonal
  double *b, *t;                     // right-hand side, post-smoothed iterate
};

// That stencil, for the solver of cg_mg.hpp.
struct OptOp {
  using Level = OptLevel;
  static constexpr int kArrays = 5;
  static __host__ __device__ double*& array(Level& L, int a) {
    return a == 0 ? L.sc : a == 1 ? L.se : a == 2 ? L.sn : a == 3 ? L.sd : L.dinv;
  }
  static __host__ __device__ double* array(const Level& L, int a) {
    return a == 0 ? L.sc : a == 1 ? L.se : a == 2 ? L.sn : a == 3 ? L.sd : L.dinv;
  }
  struct Coef {
    double c, e, w, n, s, ne, sw;
  };
  // couplings of node (j, i); 0 where there is no neighbour
  static __device__ __forceinline__ Coef coef(const Level& L, size_t base, int i, int j) {
    const size_t k = base + size_t(j) * L.nx + i;
    const bool W = i > 0, S = j > 0;
    Coef C{L.sc[k], L.se[k], L.se[W ? k - 1 : k], L.sn[k], L.sn[S ? k - L.nx : k], L.sd[k],
           L.sd[W && S ? k - L.nx - 1 : k]};
    if (!W) C.w = 0.0;
    if (!S) C.s = 0.0;
    if (!W || !S) C.sw = 0.0;
    return C;
  }
  // at position k of arrays (m values each, rows of w) whose rings are 0
  static __device__ __forceinline__ Coef ringed(const double* a, int m, int k, int w) {
    const double *se = a + m, *sn = se + m, *sd = sn + m;
    return Coef{a[k], se[k], se[k - 1], sn[k], sn[k - w], sd[k], sd[k - w - 1]};
  }
  static __device__ __forceinline__ double product(const Coef& C, double c, double e, double w, double n, double s,
                                                   double ne, double sw) {
    return C.c * c + C.e * e + C.w * w + C.n * n + C.s * s + C.ne * ne + C.sw * sw;
  }
  // Galerkin coarse stencil P^T A P of 2 x 2 aggregates: the diagonal sums the
  // aggregate's diagonal and twice its inner couplings; a coarse coupling sums
  // the fine couplings between two aggregates
  static __device__ __forceinline__ void coarsen(const Level& f, size_t bf, const Level& c, size_t bc, int k) {
    auto F = [&](const double* a, int j, int i) { return (j < f.ny && i < f.nx) ? a[bf + size_t(j) * f.pitch + i] : 0.0; };
    const int J = k / c.nx, I = k - J * c.nx, j = 2 * J, i = 2 * I;
    const size_t o = bc + size_t(J) * c.pitch + I;
    const double d = F(f.sc, j, i) + F(f.sc, j, i + 1) + F(f.sc, j + 1, i) + F(f.sc, j + 1, i + 1) +
                     2.0 * (F(f.se, j, i) + F(f.se, j + 1, i) + F(f.sn, j, i) + F(f.sn, j, i + 1) + F(f.sd, j, i));
    const bool east = I + 1 < c.nx, north = J + 1 < c.ny;
    c.sc[o] = d;
    c.se[o] = east ? F(f.se, j, i + 1) + F(f.se, j + 1, i + 1) + F(f.sd, j, i + 1) : 0.0;
    c.sn[o] = north ? F(f.sn, j + 1, i) + F(f.sn, j + 1, i + 1) + F(f.sd, j + 1, i) : 0.0;
    c.sd[o] = (east && north) ? F(f.sd, j + 1, i + 1) : 0.0;
    c.dinv[o] = 1.0 / d;
  }
};
using OptLevels = cgmg::Levels<OptOp>;

// Device state of up to `batch` optical problems on one mesh (FP64).
struct OptCg {
  int nx, ny, nn, ne, batch;
  int nblk;                    // blocks per field, min(kOptBlocks, ceil(nn / kOptThreads))
  double h;
  double *ka, *mu;             // [batch][ne] coefficients of the last forward solve
  double *ek, *em;             // [batch][ne] staged perturbations (J_o)
  double* phi;                 // [batch][nn] Phi0 of the last forward solve
  double* cur;                 // [batch][4] side currents
  cgmg::Vectors v;             // conjugate-gradient work; the right-hand side goes to v.r[1]
};

hipError_t opt_launch_set(const OptCg& c, const float* kappa, const float* mu, hipStream_t st);
hipError_t opt_launch_stage(const OptCg& c, const float* da, const float* dm, hipStream_t st);
hipError_t opt_launch_rhs(const OptCg& c, int mode, const double* cur, const float* Hin, hipStream_t st);
// Stencils of every level for the current coefficients (c.ka, c.mu).
hipError_t opt_launch_mg_setup(const OptCg& c, const OptLevels& L, hipStream_t st);
// x = 0, r and z for the right-hand side.
hipError_t opt_launch_cg_start(const OptCg& c, const OptLevels& L, hipStream_t st);
hipError_t opt_launch_cg_iteration(const OptCg& c, const OptLevels& L, int par, double tol2, hipStream_t st);
hipError_t opt_allow_lds();
hipError_t opt_launch_out(const OptCg& c, int mode, const float* Hin, float* o1, float* o2, hipStream_t st);
hipError_t opt_launch_pixels(const float* in, float* out, int npix, int batch, bool transpose, hipStream_t st);

}  // namespace qpat

// Conjugate gradients in FP64, preconditioned by one multigrid V-cycle, for a
// batch of symmetric stencil systems on [batch][ny][nx] node grids: the
// device code that the optical solve (optical.hip) and the TV priorconditioner
// (recon.hip) share.  Op names the stencil (its level type, coefficients and
// product).
//
// The V-cycle: levels of 2 x 2 node aggregates down to one node, with
// piecewise-constant prolongation P; on each level one damped Jacobi sweep
// from zero, x = om dinv b, the coarse right-hand side P^T (b - A x), the
// correction x' = x + P xc and a sweep t = x' + om dinv (b - A x'); the single
// node at the bottom is solved exactly.  x and x' are recomputed where they
// are needed, never stored.
//
// What an iteration costs is the number of launches in its chain and, on the
// finest level, the passes over memory.  So one iteration is
//   dir_q     p = z + beta p and q = A p of a tile, p.q
//   update    x += alpha p, r -= alpha q, r.r, and the level 1 right-hand side
//   restrict  level l -> l + 1 while the level is large
//   tail      all smaller levels, down and up, one workgroup a field, in LDS
//   post      level l + 1 -> l
//   post      of level 0: z, and r.z
// (513 x 513 nodes: 10 launches where a kernel per sweep, product and dot took
// 25; us an iteration of four fields, before -> now: optical 225 -> 93, TV
// 157 -> 75; 129 x 129: 87 -> 37, 89 -> 38.)  p and r alternate between two
// buffers, as a tile reads its neighbours' old values.
// Reductions run in a fixed order (one partial a block, every wave adds all of
// them), so that a field's result depends on neither the batch nor the run.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <vector>

namespace qpat {
namespace cgmg {

constexpr double kOmega = 0.8;      // damping of the Jacobi sweeps
constexpr int kMaxLevels = 32;
constexpr int kParts = 1024;        // most block partials per field

// The vectors and scalars of the solve, [batch][n] and [batch]
struct Vectors {
  int batch;
  double* x;
  double *p[2], *r[2];     // iteration k reads p[k % 2], r[k % 2] and writes the other
  double *q, *z;
  double *part_rz, *part_rr, *part_pq;   // [batch][kParts]
  double* rz;              // [2][batch]: iteration k reads rz[k % 2] and writes the other
  double *rr, *bb;         // r.r after the last iteration, r.r of the right-hand side (adjacent: rr[cap], bb[cap])
};

// ---------------------------------------------------------------- tiles
// A block of two waves works on a tile of 512 nodes, TX x 512 / TX: thread (x, y)
// on column x, rows 4 y .. 4 y + 3, so that a row of coefficients is read along x
// and a vertical coupling once.  The iterate sits in LDS with a ring of one node
// (zero outside the grid).  Small tiles: the coarser levels are bound by latency
// and gain from more blocks (4 to 5 us a launch, of which 3.4 is the launch).
constexpr int kRows = 4, kThreads = 128, kTileNodes = kThreads * kRows;
template <int TX_>
struct Tile {
  static constexpr int TX = TX_, TY = kTileNodes / TX, HX = TX + 2, HY = TY + 2, HN = HX * HY;
  static constexpr int SLOTS = (HN + kThreads - 1) / kThreads;
};

// The tile of a level: 32 x 16; on long strips, of which that would hold a few
// columns or rows, 4 x 128 (up to 12 columns) or 128 x 4 (up to 4 rows).  64 fields,
// ms a solve, 32 x 16 -> these (one thread a node, as the sweeps were launched
// before the tiles): TV 2 x 8000 27.8 -> 8.5 (12.8), 8000 x 2 29.8 -> 14.3 (23.8);
// optical 2 x 8000 nodes 9.0 -> 2.9 (3.1), 9 x 8000 16.1 -> 8.2 (10.1).  A strip of up
// to 1024 nodes is bound by latency with either tile, and 13 columns or 5 rows
// fill enough of 32 x 16.
constexpr int kSquareTile = 32, kNarrowTile = 4, kFlatTile = 128, kStrip = 1024;
inline int tile_width(int nx, int ny) {
  if (nx <= 3 * kNarrowTile && ny > kStrip) return kNarrowTile;
  if (ny <= kTileNodes / kFlatTile && nx > kStrip) return kFlatTile;
  return kSquareTile;
}
inline int tiles_x(int nx, int ny) { return (nx + tile_width(nx, ny) - 1) / tile_width(nx, ny); }
inline int tiles(int nx, int ny) {
  const int ty = kTileNodes / tile_width(nx, ny);
  return tiles_x(nx, ny) * ((ny + ty - 1) / ty);
}
// Blocks of a level, a multiple of the eight XCDs: block k runs on XCD k % 8 and
// takes tile first_tile(), so that an XCD's tiles are neighbours and its L2 holds
// the rings they share (a block past the last tile has none).  Level 0 of four
// fields of 513 x 513: update 24.4 -> 19.9 us, dir_q 18.7 -> 16.2, post 17.4 -> 14.4.
inline int blocks(int nx, int ny) { return std::min((tiles(nx, ny) + 7) & ~7, kParts); }
__device__ __forceinline__ int first_tile() { return int((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)); }

struct Slot {   // position s of this thread in the ringed tile
  int pos, k;
  bool in, own;
};
template <class T>
__device__ __forceinline__ Slot slot(int s, int i0, int j0, int nx, int ny) {
  Slot r;
  r.pos = int(threadIdx.x) + kThreads * s;
  const int py = r.pos / T::HX, px = r.pos - T::HX * py, i = i0 - 1 + px, j = j0 - 1 + py;
  r.in = r.pos < T::HN && i >= 0 && i < nx && j >= 0 && j < ny;
  r.own = r.in && px >= 1 && px <= T::TX && py >= 1 && py <= T::TY;
  r.k = r.in ? j * nx + i : 0;
  return r;
}

// Sum of the np partials of field b, in every lane (each wave adds them all).
__device__ __forceinline__ double wave_total(const double* __restrict__ part, int b, int np) {
  const double* p = part + size_t(b) * kParts;
  const int lane = threadIdx.x & 63;
  double v = 0.0;
  for (int k0 = 0; k0 < np; k0 += 512) {
    double t[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int i = k0 + 64 * k + lane;
      t[k] = p[i < np ? i : np - 1];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) v += k0 + 64 * k + lane < np ? t[k] : 0.0;
  }
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
// Block sum of one value per thread, in thread 0.
__device__ __forceinline__ double tile_sum(double v) {
  __shared__ double red[kThreads / 64];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kThreads / 64; ++w) s += red[w];
  return s;
}

// A u at node (column x, row y) of the tile, from the ringed LDS tile
template <class Op, class T>
__device__ __forceinline__ double tile_op(const typename Op::Coef& C, const double* u, int x, int y) {
  constexpr int H = T::HX;
  const double* c = u + (y + 1) * H + x + 1;
  return Op::product(C, c[0], c[1], c[-1], c[H], c[-H], c[H + 1], c[-H - 1]);
}
template <class Op>
__device__ __forceinline__ void tile_coefs(const typename Op::Level& L, size_t base, int i, int j, typename Op::Coef* C) {
  const int ic = i < L.nx ? i : L.nx - 1;
#pragma unroll
  for (int y = 0; y < kRows; ++y) {
    const int jc = j + y < L.ny ? j + y : L.ny - 1;
    C[y] = Op::coef(L, base, ic, jc);
  }
}

// ---------------------------------------------------------------- iteration
// p = z + beta p, q = A p, partials of p.q.  beta = rz_new / rz_old, 0 while
// rz_old is 0: the first iteration, whose p is 0.
// Bound by memory: it reads z, p and the stencil and writes p and q.
template <class Op, class T>
__global__ void __launch_bounds__(kThreads)
dir_q_kernel(Vectors c, typename Op::Level L, int par, int ntx, int nt, int np) {
  __shared__ double u[T::HN];
  const int b = blockIdx.y, nx = L.nx, ny = L.ny;
  const size_t base = size_t(b) * nx * ny;
  const double *z = c.z + base, *po = (par ? c.p[1] : c.p[0]) + base;
  double *pn = (par ? c.p[0] : c.p[1]) + base, *q = c.q + base;
  double zv[T::SLOTS], pv[T::SLOTS];
  auto load = [&](int t) {
    const int ty = t / ntx, i0 = (t - ty * ntx) * T::TX, j0 = ty * T::TY;
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      zv[s] = z[S.k], pv[s] = po[S.k];
    }
  };
  load(min(first_tile(), nt - 1));
  const double rzn = wave_total(c.part_rz, b, np), rz = c.rz[size_t(par) * c.batch + b];
  const double beta = rz > 0.0 ? rzn / rz : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) c.rz[size_t(1 - par) * c.batch + b] = rzn;
  const int x = threadIdx.x & (T::TX - 1), y0 = kRows * (threadIdx.x / T::TX);
  double pq = 0.0;
  for (int t = first_tile(); t < nt; t += gridDim.x) {
    const int ty = t / ntx, i0 = (t - ty * ntx) * T::TX, j0 = ty * T::TY, i = i0 + x;
    typename Op::Coef C[kRows];
    tile_coefs<Op>(L, base, i, j0 + y0, C);
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      const double v = S.in ? zv[s] + beta * pv[s] : 0.0;
      if (S.pos < T::HN) u[S.pos] = v;
      if (S.own) pn[S.k] = v;
    }
    __syncthreads();
#pragma unroll
    for (int y = 0; y < kRows; ++y) {
      const double v = tile_op<Op, T>(C[y], u, x, y0 + y);
      if (i < nx && j0 + y0 + y < ny) {
        q[size_t(j0 + y0 + y) * nx + i] = v;
        pq += u[(y0 + y + 1) * T::HX + x + 1] * v;
      }
    }
    __syncthreads();
    if (t + int(gridDim.x) < nt) load(t + gridDim.x);
  }
  const double s = tile_sum(pq);
  if (threadIdx.x == 0) c.part_pq[size_t(b) * kParts + blockIdx.x] = s;
}

// The coarse right-hand side of a tile: aggregate sums of b - A x of the first
// sweep x = om dinv b.  FINE: level 0, whose b is the CG residual, updated here:
// alpha = r.z / p.q (0 once the field has converged), x += alpha p,
// r -= alpha q, partials of r.r.
// Bound by memory on level 0 (it reads x, p, r, q, dinv and the stencil and
// writes x, r and a quarter of them), by latency on the others.
template <class Op, class T, bool FINE>
__global__ void __launch_bounds__(kThreads)
restrict_kernel(Vectors c, typename Op::Level L, double* __restrict__ bc_all, size_t fsc, int par, double tol2, int ntx,
                int nt, int np) {
  __shared__ double u[T::HN], rb[T::TX * T::TY];
  const int b = blockIdx.y, nx = L.nx, ny = L.ny, nxc = (nx + 1) >> 1, nyc = (ny + 1) >> 1;
  const size_t base = size_t(b) * L.fs;
  double* bc = bc_all + size_t(b) * fsc;
  const double *ro = FINE ? (par ? c.r[1] : c.r[0]) + base : L.b + base, *q = c.q + base;
  const double* pn = (par ? c.p[0] : c.p[1]) + base;
  double *rn = (par ? c.r[0] : c.r[1]) + base, *xv = c.x + base;
  const double* dinv = L.dinv + base;
  double rv[T::SLOTS], qv[T::SLOTS], dv[T::SLOTS], px[T::SLOTS], xx[T::SLOTS];
  auto load = [&](int t) {
    const int ty = t / ntx, i0 = (t - ty * ntx) * T::TX, j0 = ty * T::TY;
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      rv[s] = ro[S.k], dv[s] = dinv[S.k];
      if (FINE) {
        qv[s] = q[S.k];
        if (S.own) px[s] = pn[S.k], xx[s] = xv[S.k];
      }
    }
  };
  load(min(first_tile(), nt - 1));
  double alpha = 0.0, rr = 0.0;
  if (FINE) {
    const double pq = wave_total(c.part_pq, b, np), rz = c.rz[size_t(1 - par) * c.batch + b];
    const bool live = c.rr[b] > tol2 * c.bb[b] && pq > 0.0;
    alpha = live ? rz / pq : 0.0;
  }
  const int x = threadIdx.x & (T::TX - 1), y0 = kRows * (threadIdx.x / T::TX);
  for (int t = first_tile(); t < nt; t += gridDim.x) {
    const int ty = t / ntx, i0 = (t - ty * ntx) * T::TX, j0 = ty * T::TY, i = i0 + x;
    typename Op::Coef C[kRows];
    tile_coefs<Op>(L, base, i, j0 + y0, C);
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      const double r = FINE ? rv[s] - alpha * qv[s] : rv[s];
      if (S.pos < T::HN) u[S.pos] = S.in ? kOmega * dv[s] * r : 0.0;
      const int py = S.pos / T::HX, px_ = S.pos - T::HX * py;
      if (S.own) {
        rb[(py - 1) * T::TX + px_ - 1] = r;
        if (FINE) {
          xv[S.k] = xx[s] + alpha * px[s];
          rn[S.k] = r;
          rr += r * r;
        }
      }
    }
    __syncthreads();
    double e[kRows];
#pragma unroll
    for (int y = 0; y < kRows; ++y) {
      const double v = tile_op<Op, T>(C[y], u, x, y0 + y);
      e[y] = (i < nx && j0 + y0 + y < ny) ? rb[(y0 + y) * T::TX + x] - v : 0.0;
    }
#pragma unroll
    for (int y = 0; y < kRows; y += 2) {
      double a = e[y] + __shfl_xor(e[y], 1, 64);
      a += e[y + 1];
      a += __shfl_xor(e[y + 1], 1, 64);
      const int I = i >> 1, J = (j0 + y0 + y) >> 1;
      if (!(x & 1) && I < nxc && J < nyc) bc[size_t(J) * nxc + I] = a;
    }
    __syncthreads();
    if (t + int(gridDim.x) < nt) load(t + gridDim.x);
  }
  if (FINE) {
    const double s = tile_sum(rr);
    if (threadIdx.x == 0) c.part_rr[size_t(b) * kParts + blockIdx.x] = s;
  }
}

// Coarse correction and post-smoothing of a tile.  FINE: level 0 (b is the CG
// residual, the result z): partials of r.z, and block 0 stores r.r; start: also
// as that of the right-hand side.
template <class Op, class T, bool FINE>
__global__ void __launch_bounds__(kThreads)
post_kernel(Vectors c, typename Op::Level L, const double* __restrict__ xc_all, size_t fsc, const double* __restrict__ b_all,
            double* __restrict__ t_all, int start, int ntx, int nt, int np) {
  __shared__ double u[T::HN];
  const int b = blockIdx.y, nx = L.nx, ny = L.ny, nxc = (nx + 1) >> 1;
  const size_t base = size_t(b) * L.fs;
  const double *bf = b_all + base, *dinv = L.dinv + base, *xc = xc_all + size_t(b) * fsc;
  double* out = t_all + base;
  const int x = threadIdx.x & (T::TX - 1), y0 = kRows * (threadIdx.x / T::TX);
  double rz = 0.0;
  for (int t = first_tile(); t < nt; t += gridDim.x) {
    const int ty = t / ntx, i0 = (t - ty * ntx) * T::TX, j0 = ty * T::TY, i = i0 + x;
    double bv[T::SLOTS], dv[T::SLOTS], cv[T::SLOTS];
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      const int py = S.pos / T::HX, jj = j0 - 1 + py, ii = i0 - 1 + S.pos - T::HX * py;
      bv[s] = bf[S.k], dv[s] = dinv[S.k], cv[s] = xc[S.in ? (jj >> 1) * nxc + (ii >> 1) : 0];
    }
    typename Op::Coef C[kRows];
    tile_coefs<Op>(L, base, i, j0 + y0, C);
    double bo[kRows], dn[kRows];
#pragma unroll
    for (int y = 0; y < kRows; ++y) {
      const int ic = i < nx ? i : nx - 1, jc = j0 + y0 + y < ny ? j0 + y0 + y : ny - 1;
      bo[y] = bf[size_t(jc) * nx + ic], dn[y] = dinv[size_t(jc) * nx + ic];
    }
#pragma unroll
    for (int s = 0; s < T::SLOTS; ++s) {
      const Slot S = slot<T>(s, i0, j0, nx, ny);
      if (S.pos < T::HN) u[S.pos] = S.in ? kOmega * dv[s] * bv[s] + cv[s] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int y = 0; y < kRows; ++y) {
      const double v = tile_op<Op, T>(C[y], u, x, y0 + y);
      const double w = u[(y0 + y + 1) * T::HX + x + 1] + kOmega * dn[y] * (bo[y] - v);
      if (i < nx && j0 + y0 + y < ny) {
        out[size_t(j0 + y0 + y) * nx + i] = w;
        if (FINE) rz += bo[y] * w;
      }
    }
    __syncthreads();
  }
  if (FINE) {
    const double s = tile_sum(rz);
    if (threadIdx.x == 0) c.part_rz[size_t(b) * kParts + blockIdx.x] = s;
    if (blockIdx.x == 0 && threadIdx.x < 64) {
      const double rr = wave_total(c.part_rr, b, np);
      if (threadIdx.x == 0) {
        c.rr[b] = rr;
        if (start) c.bb[b] = rr;
      }
    }
  }
}

// ---------------------------------------------------------------- tail
// The levels from the first that fits one workgroup's LDS with its stencil,
// down and up, one workgroup a field.  A level is bound by latency (an LDS
// round trip, seven dependent adds, a barrier), so everything is laid out to
// read a node's operands at once, without a branch: the levels sit in zero
// rings (Level::pitch = nx + 2 in memory already), the four nodes of an
// aggregate in a quad of lanes.  33 x 33 nodes down to one: 9 to 12 us, against
// 13 launches of 4.  (A first level of 65 x 65 nodes with its
// stencil read from L2 saved two launches of 4.7 us and took 17 us.)
constexpr int kTailThreads = 1024, kTailLevels = 13, kTailLds = 160 * 1024;

template <class Op>
struct Tail {
  typename Op::Level lv[kTailLevels];
  int off[kTailLevels];   // first value of a level (its ring) in the field's arrays
  int n;                  // levels
  int m;                  // values of all levels, with their rings
};
inline size_t padded(size_t nx, size_t ny) { return (nx + 2) * (ny + 2); }
template <class Op>
size_t tail_lds(size_t m) { return (Op::kArrays + 2) * m * sizeof(double); }

// v of the lane whose index differs in bit 0 / bit 1
template <int BIT>
__device__ __forceinline__ double quad_xor(double v) {
  constexpr int perm = BIT == 0 ? 0xB1 : 0x4E;   // quad_perm [1,0,3,2] / [2,3,0,1]
  union {
    double d;
    int i[2];
  } a{v}, r;
  r.i[0] = __builtin_amdgcn_mov_dpp(a.i[0], perm, 0xF, 0xF, true);
  r.i[1] = __builtin_amdgcn_mov_dpp(a.i[1], perm, 0xF, 0xF, true);
  return r.d;
}
// k / n for 0 <= k < 2^20, rn = 1 / n: exact, the half keeps quotients off the integers
__device__ __forceinline__ int quot(int k, float rn) { return int((float(k) + 0.5f) * rn); }

template <class Op>
__global__ void __launch_bounds__(kTailThreads) tail_kernel(Tail<Op> A) {
  extern __shared__ double lds[];
  const int b = blockIdx.x, tid = threadIdx.x, m = A.m, n = A.n;
  const typename Op::Level& L0 = A.lv[0];
  const int nx0 = L0.nx, n0 = nx0 * L0.ny;
  const size_t base = size_t(b) * L0.fs, ring = size_t(nx0 + 3);   // L0's arrays start at its node (0, 0)
  // bl, ul: right-hand side (then the result) and first sweep; arr: stencils
  double *bl = lds, *ul = bl + m, *arr = ul + m;
  const double* dl = arr + (Op::kArrays - 1) * m;   // inverse diagonals: the last array
  for (int i = tid; i < m; i += kTailThreads) {
    double v[Op::kArrays];
#pragma unroll
    for (int a = 0; a < Op::kArrays; ++a) v[a] = (Op::array(L0, a) - ring)[base + i];
#pragma unroll
    for (int a = 0; a < Op::kArrays; ++a) arr[a * m + i] = v[a];
    bl[i] = 0.0, ul[i] = 0.0;
  }
  __syncthreads();
  // b and the first sweep of node k; the last level is solved
  auto store = [&](int k, double v, bool last) {
    bl[k] = last ? dl[k] * v : v;
    ul[k] = kOmega * dl[k] * v;
  };
  const float rnx0 = 1.0f / float(nx0);
  for (int q = tid; q < n0; q += kTailThreads) {
    const int j = quot(q, rnx0), i = q - j * nx0;
    store((j + 1) * (nx0 + 2) + i + 1, L0.b[base + q], n == 1);
  }
  __syncthreads();
  for (int l = 0; l + 1 < n; ++l) {
    const int nx = A.lv[l].nx, w = nx + 2, off = A.off[l], nxc = (nx + 1) >> 1, wc = nxc + 2;
    const int nq = 4 * nxc * ((A.lv[l].ny + 1) >> 1), offc = A.off[l + 1];
    const float rnc = 1.0f / float(nxc);
    for (int q = tid; q < nq; q += kTailThreads) {
      // (a node past an odd edge is in the ring: all 0)
      const int K = q >> 2, J = quot(K, rnc), I = K - J * nxc;
      const int k = off + (2 * J + ((q >> 1) & 1) + 1) * w + 2 * I + (q & 1) + 1;
      const double* u = ul + k;
      double v = bl[k] - Op::product(Op::ringed(arr, m, k, w), u[0], u[1], u[-1], u[w], u[-w], u[w + 1], u[-w - 1]);
      v += quad_xor<0>(v);
      v += quad_xor<1>(v);
      if ((q & 3) == 0) store(offc + (J + 1) * wc + I + 1, v, l + 2 == n);
    }
    __syncthreads();
  }
  for (int l = n - 2; l >= 0; --l) {
    const int nx = A.lv[l].nx, w = nx + 2, off = A.off[l], wc = ((nx + 1) >> 1) + 2, nl = nx * A.lv[l].ny;
    const double* tc = bl + A.off[l + 1] + wc + 1;   // its node (0, 0)
    const float rnx = 1.0f / float(nx);
    for (int q = tid; q < nl; q += kTailThreads) {
      const int j = quot(q, rnx), i = q - j * nx, k = off + (j + 1) * w + i + 1;
      const double* u = ul + k;
      auto x = [&](int di, int dj) { return u[dj * w + di] + tc[((j + dj) >> 1) * wc + ((i + di) >> 1)]; };
      const double uc = x(0, 0);
      const double v = Op::product(Op::ringed(arr, m, k, w), uc, x(1, 0), x(-1, 0), x(0, 1), x(0, -1), x(1, 1), x(-1, -1));
      const double t = uc + kOmega * dl[k] * (bl[k] - v);
      if (l == 0)
        L0.t[base + q] = t;
      else
        bl[k] = t;
    }
    __syncthreads();
  }
  if (n == 1 && tid == 0) L0.t[base] = bl[nx0 + 3];   // a single node
}

// ---------------------------------------------------------------- set-up
constexpr int kSetupThreads = 256, kSetupBlocks = 1024;

// Galerkin operator P^T A P of level c from level f, a thread per coarse node.
template <class Op>
__global__ void __launch_bounds__(kSetupThreads) coarsen_kernel(typename Op::Level f, typename Op::Level c) {
  const int nc = c.nx * c.ny;
  const size_t bf = size_t(blockIdx.y) * f.fs, bc = size_t(blockIdx.y) * c.fs;
  for (int k = blockIdx.x * kSetupThreads + threadIdx.x; k < nc; k += gridDim.x * kSetupThreads) Op::coarsen(f, bf, c, bc, k);
}
// All levels of the tail in their rings, from the level before it, one workgroup
// a field.
template <class Op>
__global__ void __launch_bounds__(kTailThreads) coarsen_tail_kernel(typename Op::Level fine, Tail<Op> A) {
  const size_t base = size_t(blockIdx.x) * A.lv[0].fs;
  for (int l = 0; l < A.n; ++l) {
    const typename Op::Level f = l ? A.lv[l - 1] : fine, c = A.lv[l];
    const size_t bf = size_t(blockIdx.x) * f.fs;
    const int w = c.nx + 2, np = w * (c.ny + 2);
    for (int p = threadIdx.x; p < np; p += kTailThreads) {
      const int j = p / w - 1, i = p - (j + 1) * w - 1;
      if (i >= 0 && i < c.nx && j >= 0 && j < c.ny)
        Op::coarsen(f, bf, c, base, j * c.nx + i);
      else   // the ring
        for (int a = 0; a < Op::kArrays; ++a) (Op::array(c, a) + base)[j * w + i] = 0.0;
    }
    __threadfence_block();
    __syncthreads();
  }
}

// ---------------------------------------------------------------- host
// The levels of a solver and the launches of its iteration.
template <class Op>
struct Levels {
  using Level = typename Op::Level;
  std::vector<Level> lv;
  int tail = 0;      // first level of the tail, at least 1
  int tail_m = 0;    // values of its levels, with their rings

  // Sizes of the levels of an nx x ny node grid (more than one node); false if
  // there are too many.
  bool plan(int nx, int ny) {
    lv.clear();
    for (int w = nx, h = ny;; w = (w + 1) / 2, h = (h + 1) / 2) {
      Level L{};
      L.nx = w, L.ny = h, L.pitch = w, L.fs = size_t(w) * h;
      lv.push_back(L);
      if (size_t(w) * h == 1) break;
    }
    if (int(lv.size()) > kMaxLevels) return false;
    for (tail = 1;; ++tail) {
      size_t m = 0;
      for (size_t l = tail; l < lv.size(); ++l) m += padded(lv[l].nx, lv[l].ny);
      if (int(lv.size()) - tail <= kTailLevels && tail_lds<Op>(m) <= size_t(kTailLds)) {
        tail_m = int(m);
        break;
      }
    }
    for (size_t l = tail; l < lv.size(); ++l) lv[l].fs = size_t(tail_m), lv[l].pitch = lv[l].nx + 2;
    return true;
  }
  // doubles of the levels above 0 (stencil arrays, b, t)
  size_t words(int batch) const {
    size_t w = 0;
    for (int l = 1; l <= tail; ++l) w += lv[l].fs * (Op::kArrays + 2);
    return w * batch;
  }
  // Hands out those from take(count): an array of a field's tail holds its levels
  // one after another, each in its ring.
  template <typename Take>
  void carve(int batch, Take take) {
    for (int l = 1; l <= tail; ++l) {
      Level& L = lv[l];
      for (int a = 0; a < Op::kArrays; ++a) Op::array(L, a) = take(L.fs * batch);
      L.b = take(L.fs * batch);
      L.t = take(L.fs * batch);
    }
    size_t off = padded(lv[tail].nx, lv[tail].ny);
    for (size_t l = tail + 1; l < lv.size(); ++l) {
      for (int a = 0; a < Op::kArrays; ++a) Op::array(lv[l], a) = Op::array(lv[tail], a) + off + lv[l].pitch + 1;
      off += padded(lv[l].nx, lv[l].ny);
    }
    for (int a = 0; a < Op::kArrays; ++a) Op::array(lv[tail], a) += lv[tail].pitch + 1;
  }
  static hipError_t allow_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&tail_kernel<Op>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kTailLds);
  }

  Tail<Op> tail_args() const {
    Tail<Op> T{};
    T.n = int(lv.size()) - tail;
    T.m = tail_m;
    int off = 0;
    for (int l = 0; l < T.n; ++l) {
      T.lv[l] = lv[tail + l];
      T.off[l] = off;
      off += int(padded(T.lv[l].nx, T.lv[l].ny));
    }
    return T;
  }
  // The stencils of levels 1 and up, from that of level 0.
  hipError_t setup(int batch, hipStream_t st) const {
    for (int l = 0; l + 1 < tail; ++l) {
      const int n = lv[l + 1].nx * lv[l + 1].ny, nb = std::min(kSetupBlocks, (n + kSetupThreads - 1) / kSetupThreads);
      hipLaunchKernelGGL((coarsen_kernel<Op>), dim3(nb, batch), dim3(kSetupThreads), 0, st, lv[l], lv[l + 1]);
    }
    hipLaunchKernelGGL((coarsen_tail_kernel<Op>), dim3(batch), dim3(kTailThreads), 0, st, lv[tail - 1], tail_args());
    return hipGetLastError();
  }

  // f with the tile of a level
  template <typename F>
  static void with_tile(const Level& L, F f) {
    switch (tile_width(L.nx, L.ny)) {
      case kNarrowTile: return f(Tile<kNarrowTile>());
      case kFlatTile: return f(Tile<kFlatTile>());
      default: return f(Tile<kSquareTile>());
    }
  }
  // z = V-cycle of the residual, after the CG update (not at the start); partials of r.z
  void vcycle(const Vectors& c, int par, double tol2, bool start, hipStream_t st) const {
    const int np = blocks(lv[0].nx, lv[0].ny);
    auto grid = [&](const Level& L) { return dim3(unsigned(blocks(L.nx, L.ny)), unsigned(c.batch)); };
    for (int l = 0; l < tail; ++l) {
      const Level &L = lv[l], &C = lv[l + 1];
      const int ntx = tiles_x(L.nx, L.ny), nt = tiles(L.nx, L.ny);
      with_tile(L, [&](auto t) {
        using T = decltype(t);
        if (l == 0 && !start)
          hipLaunchKernelGGL((restrict_kernel<Op, T, true>), grid(L), dim3(kThreads), 0, st, c, L, C.b, C.fs, par, tol2,
                             ntx, nt, np);
        else
          hipLaunchKernelGGL((restrict_kernel<Op, T, false>), grid(L), dim3(kThreads), 0, st, c, L, C.b, C.fs, par, tol2,
                             ntx, nt, np);
      });
    }
    const Tail<Op> T = tail_args();
    const size_t lds = tail_lds<Op>(tail_m);
    hipLaunchKernelGGL((tail_kernel<Op>), dim3(c.batch), dim3(kTailThreads), lds, st, T);
    for (int l = tail - 1; l >= 0; --l) {
      const Level &L = lv[l], &C = lv[l + 1];
      const int ntx = tiles_x(L.nx, L.ny), nt = tiles(L.nx, L.ny);
      with_tile(L, [&](auto t) {
        using T = decltype(t);
        if (l == 0)
          hipLaunchKernelGGL((post_kernel<Op, T, true>), grid(L), dim3(kThreads), 0, st, c, L, C.t, C.fs,
                             c.r[par ? 0 : 1], c.z, start ? 1 : 0, ntx, nt, np);
        else
          hipLaunchKernelGGL((post_kernel<Op, T, false>), grid(L), dim3(kThreads), 0, st, c, L, C.t, C.fs, L.b, L.t, 0,
                             ntx, nt, np);
      });
    }
  }
  // After x = p[0] = 0, r[0] = the right-hand side, rz[0] = 0 and the partials
  // of r.r: z and its partials.  (par = 1: the V-cycle reads r[0].)
  hipError_t start(const Vectors& c, hipStream_t st) const {
    vcycle(c, 1, 0.0, true, st);
    return hipGetLastError();
  }
  hipError_t iteration(const Vectors& c, int par, double tol2, hipStream_t st) const {
    const Level& L = lv[0];
    const int np = blocks(L.nx, L.ny);
    with_tile(L, [&](auto t) {
      hipLaunchKernelGGL((dir_q_kernel<Op, decltype(t)>), dim3(np, c.batch), dim3(kThreads), 0, st, c, L, par,
                         tiles_x(L.nx, L.ny), tiles(L.nx, L.ny), np);
    });
    vcycle(c, par, tol2, false, st);
    return hipGetLastError();
  }
};

// x = p[0] = 0 and r[0] = the right-hand side, rz[0] = 0, partials of r.r
// (np blocks a field, kThreads threads)
template <typename T>
__global__ void __launch_bounds__(kThreads) start_kernel(Vectors c, const T* __restrict__ rhs, size_t n) {
  const int b = blockIdx.y;
  const size_t base = size_t(b) * n;
  double rr = 0.0;
  for (size_t k = size_t(blockIdx.x) * kThreads + threadIdx.x; k < n; k += size_t(gridDim.x) * kThreads) {
    const double r = double(rhs[base + k]);
    c.x[base + k] = 0.0;
    c.p[0][base + k] = 0.0;
    c.r[0][base + k] = r;
    rr += r * r;
  }
  const double s = tile_sum(rr);
  if (threadIdx.x == 0) {
    c.part_rr[size_t(b) * kParts + blockIdx.x] = s;
    if (blockIdx.x == 0) c.rz[b] = 0.0;
  }
}

}  // namespace cgmg
}  // namespace qpat

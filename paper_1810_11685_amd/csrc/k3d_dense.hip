// 3-D passes whose axis transforms are matrix products (lengths 18 to 63).
//
// The paper's 3-D axes (33, 37, 49, 53 points) are short and mostly odd or
// prime, and any length must do, so a Stockham FFT either runs few butterflies
// per stage through many barriers (49 = 7 7: eight LDS stages a plane, 343
// butterflies each) or, at a prime, is a direct sum anyway.  Here an axis is
// transformed by the symmetric DFT of dense3() on the FP32 matrix
// instructions (v_mfma_f32_16x16x4_f32): 16 outputs q times 16 lines per
// instruction, real cosine and sine matrices (FP64, rounded once), the real
// and imaginary parts as separate accumulators, so output q and its mirror
// n - q come out of one lane without an exchange.
//   row pass   - 16 x-lines a tile: inverse transforms straight from the
//                spectra in global memory, the pointwise update from LDS with
//                its operands prefetched, forward transforms to global memory;
//                two barriers.
//   plane pass - y forward straight from global memory, z forward, the
//                multiplier and z inverse in one wave's registers (the
//                accumulators of a product are the next one's second operand,
//                with the matrix columns in that order), y inverse straight to
//                global memory; two barriers.
// The kernels are instanced per length class (steps and row tiles), so no step
// is guarded and LDS offsets are immediates, and every edge is in the matrices:
// rows q past n/2 hold the true factors and give the mirrored output again (the
// same bits), columns past n/2 are zero, columns read twice (r = 0 of the
// chained form, r = n/2) are halved.
// Bound: latency of the dependent phases at few vectors (a plane's matrix
// instructions take 3 us of its 9), the matrix unit and L2 at many.  Microseconds
// an iterate, one / three / sixteen vectors, FFT stages -> these passes:
//   53 x 53 x 53  107 / 142 / 477 -> 50 / 65 / 200
//   60 x 48 x 40   72 /  93 / 215 -> 46 / 63 / 162
//   48 x 48 x 48   90 / 102 / 259 -> 44 / 52 / 148
//   32 x 32 x 32   55 /  58 /  99 -> 36 / 38 /  78
//   24 x 24 x 24   52 /  53 /  68 -> 28 / 28 /  36
// (shorter than 18 an axis has too few steps for the matrix unit; from 64 the
// products grow past what the FFT stages take).
#include "k3d_device.hpp"

namespace qpat3 {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 splat(float v) {
  f4 r = {v, v, v, v};
  return r;
}

// A copy of v that the compiler knows nothing about: what is computed from it
// inside a loop body stays there (hoisted, the addresses of all phases of a
// block would be live at once and spill).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Two complex values in one access (lines start at any 8-byte boundary).
typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));
__device__ __forceinline__ void ld2(const float2* p, float2& a, float2& b) {
  const f4u v = *reinterpret_cast<const f4u*>(p);
  a = make_float2(v.x, v.y);
  b = make_float2(v.z, v.w);
}
__device__ __forceinline__ void st2(float2* p, float2 a, float2 b) {
  const f4u v = {a.x, a.y, b.x, b.y};
  *reinterpret_cast<f4u*>(p) = v;
}

constexpr int kDenseThreads = 512;   // most threads of a block of these kernels

// Length classes: S steps of four inputs, MT row tiles, MAXN the longest axis.
// r = 1 .. 4 S and q = 0 .. 16 MT - 1 stay below the shortest length of a class.
template <int C>
struct Cls {
  static constexpr int S = dense3_steps(C);
  static constexpr int MT = C == 0 ? 1 : 2;
  static constexpr int MINN = C == 0 ? 18 : C == 1 ? 32 : C == 2 ? 34 : 50;
  static constexpr int MAXN = C == 0 ? 31 : C == 1 ? 33 : C == 2 ? 49 : 63;
  static_assert(4 * S < MINN && 16 * MT - 1 < MINN && MAXN / 2 <= 4 * S && MAXN / 2 < 16 * MT, "class");
};

// One row tile of a matrix at this lane (kDenseTable layout): K steps.
template <int K>
struct Mat {
  f4 v[K / 2];
  __device__ __forceinline__ float c(int s) const { return v[s >> 1][2 * (s & 1)]; }
  __device__ __forceinline__ float s(int k) const { return v[k >> 1][2 * (k & 1) + 1]; }
};
template <int K>
__device__ __forceinline__ void mat_load(Mat<K>& R, const float* __restrict__ t, int tile, int lane) {
  const f4* p = reinterpret_cast<const f4*>(t) + tile * (kDenseSteps / 2) * 64;
#pragma unroll
  for (int k = 0; k < K / 2; ++k) R.v[k] = p[k * 64 + lane];
}

// Lanes 32 to 63 of a against lanes 0 to 31 of b (both halves of the wave active).
__device__ __forceinline__ void half_swap(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void half_swap(float2& a, float2& b) {
  half_swap(a.x, b.x);
  half_swap(a.y, b.y);
}

// The order of a sum.  A smooth field in the middle of the grid is small at r = 0
// and large towards r = n/2, and its transform at high q is a difference of large
// terms; a spectrum is large at q = 0.  What a sum loses is its roundings while it
// is large, so forward transforms add r upwards, inverse ones downwards with the
// term of r = 0 last, each as two chains, one per half of the steps (two
// accumulators: half as many roundings in a row, and two independent chains for the
// matrix unit).  Relative L2 error of d/dx of five blobs, 1e-7: FFT stages / even
// and odd steps of inputs a quarter of the range apart / so ordered: 31^3 4.6 / 5.9 /
// 3.9, 53^3 4.4 / 6.8 / 4.0, 60^3 7.3 / 8.2 / 4.0; of white noise, 53^3, 2.5 / 2.1 / 2.1.
// A J^T J v of 31 steps: 53^3 3.07 -> 3.11 ms, x 16 12.51 -> 12.38.
// Step i of chain h (0: the half of the small r) of S steps:
template <int S, bool DOWN>
__host__ __device__ constexpr int chain_step(int h, int i) { return h * (S / 2) + (DOWN ? S / 2 - 1 - i : i); }

// LDS row stride (floats) of an x-line, with a slot past its end: 4 times an
// odd number, so that the sixteen lines of a tile start in different banks.
template <int C>
__host__ __device__ constexpr int line_stride() { return 4 * (((Cls<C>::MAXN + 4) / 4) | 1); }
// LDS row stride (complex) of a y-line of a plane, with a slot past its end:
// twice an odd number.
template <int C>
__host__ __device__ constexpr int plane_stride() { return 2 * (((Cls<C>::MAXN + 2) / 2) | 1); }

// ---------------------------------------------------------------- row pass
// Pointwise operands of one element, loaded before the first barrier:
// o[0..2] the fields read (v, rho or the q of A2 in o[3]), o[3..5] medium,
// a[0..2] the PML diagonals of the three axes, c2, and x: p0 or the
// accumulated gradient of the iterates that use them.
struct RowOps {
  float o[6], a[3], c2, x;
};

template <int MODE>
__device__ __forceinline__ void ops_load(RowOps& R, const Medium3& M, const float* __restrict__ fv, const IO3& X,
                                         unsigned N, unsigned idx, int x, int y, int z, int n) {
  if constexpr (MODE == R3_F1 || MODE == R3_A3) {
    R.a[0] = M.avx[x], R.a[1] = M.avy[y], R.a[2] = M.avz[z];
#pragma unroll
    for (int i = 0; i < 3; ++i) R.o[i] = fv[i * N + idx];
    R.o[3] = M.bx[idx], R.o[4] = M.by[idx], R.o[5] = M.bz[idx];
  } else if constexpr (MODE == R3_F2 || MODE == R3_F2L || MODE == R3_A1L || MODE == R3_A2) {
    R.a[0] = M.arx[x], R.a[1] = M.ary[y], R.a[2] = M.arz[z];
#pragma unroll
    for (int i = 0; i < 3; ++i) R.o[i] = fv[(3 + i) * N + idx];
    if constexpr (MODE == R3_A2) R.o[3] = fv[6 * N + idx];
    R.o[4] = M.rho0[idx];
    if (MODE == R3_F2L || MODE == R3_A1L || n <= 0) R.c2 = M.c2[idx];
    if constexpr (MODE == R3_F2 || MODE == R3_F2L) {
      if (n <= 0) R.x = X.in[idx];
    } else {
      if (n == -1 && M.nt >= 2) R.x = X.out[idx];   // accumulated at n = 0
    }
  } else if constexpr (MODE == R3_F3) {
#pragma unroll
    for (int i = 0; i < 3; ++i) R.o[i] = fv[(3 + i) * N + idx];
    R.c2 = M.c2[idx], R.o[3] = M.c2eta[idx], R.o[4] = M.c2tau[idx];
  } else if constexpr (MODE == R3_A1) {
    R.c2 = M.c2[idx], R.o[3] = M.c2eta[idx], R.o[4] = M.c2tau[idx];
  } else if constexpr (MODE == R3_FWD1) {
    R.x = X.in[idx];
  }
}

// The update of one element: in[] the incoming transforms there, out[] the
// outgoing fields (the scheme of k3d.hip's row pass, term by term).
template <int MODE>
__device__ __forceinline__ void ops_update(const RowOps& R, const Medium3& M, float* __restrict__ fv, const IO3& X,
                                           unsigned N, unsigned idx, int n, const float* in, float* out) {
  const float dt = M.dt;
  const bool first = (n == M.nt - 2);
  if constexpr (MODE == R3_F1) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float vo = (n == 0) ? 0.f : R.o[i];
      const float v = R.a[i] * (R.a[i] * vo - R.o[3 + i] * in[i]);
      fv[i * N + idx] = v;
      out[i] = v;
    }
  } else if constexpr (MODE == R3_F2 || MODE == R3_F2L) {
    const bool skip = (n == -1);
    const float r0 = R.o[4];
    const float src = (n <= 0) ? R.x * (1.0f / 6.0f) / R.c2 : 0.f;   // p0 / (2 d c^2), d = 3
    float S = 0.f, u = 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float e = skip ? 0.f : in[i];
      const float ro = skip ? 0.f : R.o[i];
      const float rho = R.a[i] * (R.a[i] * ro - dt * r0 * e) + src;
      fv[(3 + i) * N + idx] = rho;
      S += rho;
      u += R.a[i] * e;
    }
    if constexpr (MODE == R3_F2) {
      out[0] = S;
      out[1] = r0 * u;
    } else {
      out[0] = R.c2 * S;
    }
  } else if constexpr (MODE == R3_F3) {
    const float S = R.o[0] + R.o[1] + R.o[2];
    out[0] = R.c2 * S - R.o[3] * in[0] + R.o[4] * in[1];
  } else if constexpr (MODE == R3_A1) {
    const float pb = -in[0];   // -(sum_i d_i^- g_i) + M^T r: the scatter is already in
    fv[6 * N + idx] = R.c2 * pb;
    out[0] = R.o[3] * pb;
    out[1] = R.o[4] * pb;
  } else if constexpr (MODE == R3_A1L || MODE == R3_A2) {
    const float r0 = R.o[4];
    float sb, ub;
    if constexpr (MODE == R3_A1L) {
      sb = R.c2 * -in[0];
      ub = 0.f;
    } else {
      sb = R.o[3] - in[0];
      ub = in[1];
    }
    float rb[3], sum = 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      rb[i] = (first ? 0.f : R.o[i]) + sb;
      sum += rb[i];
    }
    if (n == 0) X.out[idx] = sum;
    if (n == -1) {
      const float acc = M.nt >= 2 ? R.x : 0.f;
      X.out[idx] = (sum + acc) * (1.0f / 6.0f) / R.c2;
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        out[i] = r0 * R.a[i] * (ub - dt * rb[i]);
        fv[(3 + i) * N + idx] = R.a[i] * R.a[i] * rb[i];
      }
    }
  } else if constexpr (MODE == R3_A3) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float vb = (first ? 0.f : R.o[i]) - in[i];
      out[i] = -R.a[i] * R.o[3 + i] * vb;
      fv[i * N + idx] = R.a[i] * R.a[i] * vb;
    }
  } else if constexpr (MODE == R3_FWD1) {
    out[0] = R.x;
  } else {  // R3_INV1
    X.out[idx] = in[0];
  }
}

// fields a row pass reads or writes through LDS, whichever is more
template <int MODE>
__host__ __device__ constexpr int row_fields() {
  return (MODE == R3_F3 || MODE == R3_A1) ? 2 : (MODE == R3_FWD1 || MODE == R3_INV1) ? 1 : 3;
}
template <int MODE>
__host__ __device__ constexpr int row_in() {
  return MODE == R3_F3 || MODE == R3_A2 ? 2 : (MODE == R3_A1 || MODE == R3_A1L || MODE == R3_INV1) ? 1
                                          : MODE == R3_FWD1 ? 0 : 3;
}

constexpr int kOps = 4;   // elements a thread prefetches (a 16 x 63 tile at 256 threads)

template <int MODE, int C>
__global__ void __launch_bounds__(kDenseThreads) row3_dense_kernel(const Launch3 L, int ntile, int chunk, int n) {
  constexpr int S = Cls<C>::S, MT = Cls<C>::MT, LX = line_stride<C>();
  args3_batch(L, ntile, chunk, n);
  asm volatile("" ::"s"(L.m.dfx), "s"(L.m.dfxi), "s"(L.m.dt), "s"(L.m.ns));
  int item, tile;
  if (!locate(L.nitems, ntile, chunk, item, tile)) return;
  const Medium3& M = L.m;
  const Work3 W = shift(L.w0, item * L.wstride);
  const IO3 X = L.io[item];
  const int nx = M.nx, ny = M.ny, rt = M.rt, nl = M.nlines, ct = M.ct, nxh = nx / 2;
  const int l0 = tile * rt, G = (rt + 15) >> 4, FS = G * 16 * LX;
  const unsigned N = unsigned(nl) * unsigned(nx);
  const int B = blockDim.x, tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = B >> 6;
  extern __shared__ float ldsf[];
  int nin, nout;
  row_counts<MODE>(M, n, nin, nout);
  const unsigned specN = unsigned(M.ctiles) * unsigned(ct) * unsigned(nl);
  const float rct = rcp(ct);
  // offset of spectrum column c (ct columns a tile)
  auto col_off = [&](int c) -> unsigned {
    if (ct == 1) return __umul24(unsigned(c), unsigned(nl));
    const int t = udiv(c, rct);
    return unsigned(t) * unsigned(nl * ct) + unsigned(c - t * ct);
  };

  // ---- the adjoint divergence arrives as its three terms, one per spectrum
  constexpr int NSUM = (MODE == R3_A1 || MODE == R3_A1L) ? 3 : 1;
  float2 x0[NSUM], b[NSUM][S];
  Mat<S> A;
  auto unit_load = [&](int u, int lane) {
    const int g = lane >> 4, m = lane & 15, mt = u % MT, fg = u / MT, f = fg / G, grp = fg - f * G;
    const float2* src = W.s + size_t(f) * specN;
    const unsigned lo = unsigned(min(l0 + 16 * grp + m, nl - 1)) * unsigned(ct);
    mat_load(A, M.dfxi, mt, lane);
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
      const float2* sk = src + size_t(k) * specN;
      x0[k] = sk[lo];
#pragma unroll
      for (int s = 0; s < S; ++s) b[k][s] = sk[lo + col_off(min(dense3_input(s, g) + 1, nxh))];
    }
  };
  const int uin = nin * G * MT;
  if (w < uin) unit_load(w, tid & 63);
  // ---- operands of the first kOps elements of this thread
  const int tot = rt * nx;
  const float rnx = rcp(nx), rny = rcp(ny);
  RowOps ops[kOps];
  auto load = [&](RowOps& R, int t) {
    const int j2 = udiv(t, rnx), x = t - j2 * nx, l = min(l0 + j2, nl - 1);
    const int z = udiv(l, rny), y = l - z * ny;
    ops_load<MODE>(R, M, W.f, X, N, unsigned(l) * unsigned(nx) + unsigned(x), x, y, z, n);
  };
#pragma unroll
  for (int k = 0; k < kOps; ++k)
    if (w * 64 + k * B < tot) load(ops[k], min(tid + k * B, tot - 1));
  // ---- sensors: the adjoint's contribution to this thread's first node, the
  // forward's first tap
  int na = 0, nb = 0;
  ScatterNode nd{};
  Tap3 tp{};
  auto node_sum = [&](const ScatterNode& q) {
    // one thread per receiving node, its entries summed in a fixed order
    const float* r = X.in + size_t(n + 1) * M.ns;
    float acc = 0.f;
    for (int e = q.e0; e < q.e1; ++e) {
      const ScatterEntry en = M.entries[e];
      acc += en.w * r[en.s];
    }
    return acc;
  };
  float nacc = 0.f;
  if constexpr (MODE == R3_A1 || MODE == R3_A1L) {
    na = M.node_off[l0], nb = M.node_off[min(l0 + rt, nl)];
    if (na + tid < nb) {
      nd = M.nodes[na + tid];
      nacc = node_sum(nd);
    }
  }
  if constexpr (MODE == R3_F2L || MODE == R3_F3) {
    na = M.tap_off[l0], nb = M.tap_off[min(l0 + rt, nl)];
    if (na + tid < nb) tp = M.taps[na + tid];
  }

  // ---- inverse transforms: x_j = P_j - Q_j and x_{n-j} = P_j + Q_j with
  // P = sum_q w_q Re X_q cos, Q = sum_q w_q Im X_q sin (w_q = 2, 1 at q = 0, n/2;
  // in the matrix)
  if (nin > 0) {
    for (int u = w; u < uin; u += nw) {
      const int lane = opaque(tid & 63), g = lane >> 4, m = lane & 15;
      if (u != w) unit_load(u, lane);
      const int mt = u % MT, fg = u / MT, f = fg / G, grp = fg - f * G;
      float p0 = x0[0].x;
      if constexpr (NSUM == 3) p0 = (x0[0].x + x0[1].x) + x0[2].x;
      f4 P[2] = {splat(0.f), splat(0.f)}, Q[2] = {splat(0.f), splat(0.f)};
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const int s = chain_step<S, true>(k & 1, k >> 1);
        float2 v = b[0][s];
        if constexpr (NSUM == 3) v = cadd(cadd(b[0][s], b[1][s]), b[2][s]);
        P[k & 1] = mma(A.c(s), v.x, P[k & 1]);
        Q[k & 1] = mma(A.s(s), v.y, Q[k & 1]);
      }
      float* row = ldsf + f * FS + (16 * grp + m) * LX;
      const int j = 16 * mt + 4 * g;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float c = (P[1][i] + P[0][i]) + p0, d = Q[1][i] + Q[0][i];
        row[j + i] = c - d;
        row[nx - j - i] = c + d;   // j = 0: the slot past the line
      }
    }
  } else if (MODE == R3_A1 || MODE == R3_A1L) {
    for (int t = tid; t < FS; t += B) ldsf[t] = 0.f;
  }
  // the forward matrices of this wave's first unit, read over the barrier
  const int uout = nout * G * MT;
  if (w < uout) mat_load(A, M.dfx, w % MT, tid & 63);
  __syncthreads();
  if constexpr (MODE == R3_A1 || MODE == R3_A1L) {
    // the update takes p* = -(what is in LDS)
    for (int k = na + tid; k < nb; k += B) {
      const bool pre = k == na + tid;
      const ScatterNode q = pre ? nd : M.nodes[k];
      ldsf[(q.line - l0) * LX + q.ix] -= pre ? nacc : node_sum(q);
    }
    __syncthreads();
  }

  // ---- pointwise update, in place in LDS
  constexpr int NI = row_in<MODE>(), NF = row_fields<MODE>();
  for (int base = 0; base < tot; base += kOps * B) {
#pragma unroll
    for (int k = 0; k < kOps; ++k) {
      const int t = base + tid + k * B;
      if (t < tot) {
        const int j2 = udiv(t, rnx), x = t - j2 * nx, l = l0 + j2;
        float* e = ldsf + j2 * LX + x;
        if (base > 0) load(ops[k], t);
        float in[3] = {0.f, 0.f, 0.f}, out[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < NI; ++f)
          if (nin > 0 || MODE == R3_A1 || MODE == R3_A1L) in[f] = e[f * FS];
        if (l < nl) ops_update<MODE>(ops[k], M, W.f, X, N, unsigned(l) * unsigned(nx) + unsigned(x), n, in, out);
#pragma unroll
        for (int f = 0; f < NF; ++f) e[f * FS] = out[f];
      }
    }
  }
  if (nout == 0) return;
  __syncthreads();
  if constexpr (MODE == R3_F2L || MODE == R3_F3) {
    // sensor partials of this tile's lines: part[n+1][s][slot]
    for (int e = na + tid; e < nb; e += B) {
      if (e != na + tid) tp = M.taps[e];
      const float* row = ldsf + (tp.line - l0) * LX;
      W.part[(size_t(n + 1) * M.ns + tp.s) * 4 + tp.slot] = tp.wl * row[tp.ixl] + tp.wr * row[tp.ixr];
    }
  }

  // ---- forward transforms: Re X_q = x_0 + sum_r cos e_r, Im X_q = -sum_r sin o_r
  for (int u = w; u < uout; u += nw) {
    const int lane = opaque(tid & 63), g = lane >> 4, m = lane & 15;
    const int mt = u % MT, og = u / MT, o = og / G, grp = og - o * G;
    if (MT > 1 && mt != w % MT) mat_load(A, M.dfx, mt, lane);
    const float* row = ldsf + o * FS + (16 * grp + m) * LX;
    const float *up = row + g + 1, *dn = row + (nx - g - 1);
    f4 P[2] = {splat(row[0]), splat(0.f)}, Q[2] = {splat(0.f), splat(0.f)};
#pragma unroll
    for (int k = 0; k < S; ++k) {
      const int s = chain_step<S, false>(k & 1, k >> 1);
      const float xa = up[dense3_input(s, 0)], xm = dn[-dense3_input(s, 0)];
      P[k & 1] = mma(A.c(s), xa + xm, P[k & 1]);
      Q[k & 1] = mma(A.s(s), xa - xm, Q[k & 1]);
    }
    if (MT > 1 && mt != w % MT) mat_load(A, M.dfx, w % MT, lane);
    const int l = l0 + 16 * grp + m;
    // the pressure goes to spectrum 3, which the gradient pass reads while it
    // writes spectra 0..2
    const int of = (MODE == R3_F2L || MODE == R3_F3) ? 3 : o;
    float2* dst = W.s + size_t(of) * specN + unsigned(l) * unsigned(ct);
    if (16 * grp + m < rt && l < nl) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int q = 16 * mt + 4 * g + i;
        if (q <= nxh) dst[col_off(q)] = make_float2(P[0][i] + P[1][i], -(Q[0][i] + Q[1][i]));
      }
    }
  }
}

// ---------------------------------------------------------------- plane pass
// One row tile of a complex transform: cos and sin products of the real and
// imaginary parts, in two chains (above), eight independent ones in all, which
// keeps the matrix unit busy.  One tile at a time, so that this costs no registers.
struct Acc {
  f4 cr, ci, sr, si;
};
// e, o: x_r +- x_{n-r} of the steps
template <bool DOWN, int S>
__device__ __forceinline__ Acc tile_products(float2 x0, const float2* e, const float2* o, const Mat<S>& A) {
  const f4 zero = splat(0.f);
  Acc a[2] = {{DOWN ? zero : splat(x0.x), DOWN ? zero : splat(x0.y), zero, zero}, {zero, zero, zero, zero}};
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const int h = k & 1, s = chain_step<S, DOWN>(h, k >> 1);
    a[h].cr = mma(A.c(s), e[s].x, a[h].cr);
    a[h].ci = mma(A.c(s), e[s].y, a[h].ci);
    a[h].sr = mma(A.s(s), o[s].x, a[h].sr);
    a[h].si = mma(A.s(s), o[s].y, a[h].si);
  }
  Acc r = {a[1].cr + a[0].cr, a[1].ci + a[0].ci, a[1].sr + a[0].sr, a[1].si + a[0].si};
  if (DOWN) r.cr += splat(x0.x), r.ci += splat(x0.y);
  return r;
}
// outputs q and n - q of register i: C -+ i S (forward), the other way inverse
template <bool INV>
__device__ __forceinline__ void acc_out(const Acc& a, int i, float2& q, float2& mq) {
  const float2 lo = make_float2(a.cr[i] + a.si[i], a.ci[i] - a.sr[i]);
  const float2 hi = make_float2(a.cr[i] - a.si[i], a.ci[i] + a.sr[i]);
  q = INV ? hi : lo;
  mq = INV ? lo : hi;
}

// Which spectrum a plane block reads and which operator it applies, from its
// sub-block (the launcher fills it from the pass kind).
struct PlaneOps {
  int nsplit;       // blocks per column tile, one per output
  int in;           // spectrum read by every block, or -1: its own
  int code[3];      // operator of each output
};

// A wave holds the matrices in registers, read from L2 before they are used
// (160 to 248 registers, so two blocks of 256 threads a CU; with the matrices in
// LDS, read per product, three share it, for no gain: 60 x 48 x 40, 16 vectors,
// 161.8 against 162.3 us an iterate, 53^3 216.4 against 202.8).
template <int CY, int CZ>
__global__ void __launch_bounds__(256, 2)
plane3_dense_kernel(const Launch3 L, int ntile, int chunk, PlaneOps P, int n) {
  constexpr int SY = Cls<CY>::S, MY = Cls<CY>::MT, SZ = Cls<CZ>::S, MZ = Cls<CZ>::MT, LY = plane_stride<CY>();
  args3_batch(L, ntile, chunk, n);
  asm volatile("" ::"s"(L.m.dfy), "s"(L.m.dfz), "s"(L.m.dfzc), "s"(P.nsplit), "s"(P.in), "s"(P.code[0]),
               "s"(P.code[1]), "s"(P.code[2]), "s"(L.m.kap), "s"(L.m.ldis), "s"(L.m.labs));
  int item, tile;
  if (!locate(L.nitems, ntile, chunk, item, tile)) return;
  const Medium3& M = L.m;
  int sub = 0;   // the field (diagonal passes) or output (gradient) of this block
  if (P.nsplit > 1) {
    const int t = tile / P.nsplit;
    sub = tile - t * P.nsplit;
    tile = t;
  }
  const int cd = sub == 0 ? P.code[0] : sub == 1 ? P.code[1] : P.code[2];
  const Work3 W = shift(L.w0, item * L.wstride);
  const int ct = M.ct, ny = M.ny, nz = M.nz, nl = M.nlines, nyh = ny / 2;
  const int c0 = tile * ct, ncols = min(ct, M.nxh1 - c0);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nw = int(blockDim.x) >> 6;
  const int NTy = (ny + 15) >> 4, NTz = (nz + 15) >> 4;
  const size_t specN = size_t(M.ctiles) * ct * nl;
  const float2* const in = W.s + size_t(P.in >= 0 ? P.in : sub) * specN + size_t(tile) * nl * ct;
  float2* const out = W.s + size_t(sub) * specN + size_t(tile) * nl * ct;
  extern __shared__ float2 lds2[];   // the plane, the z symbol
  const bool hasz = cd == OP_DZP || cd == OP_DZM;
  float2* const lz = lds2 + nz * LY;   // the z symbol, where the operator has one

  // y forward inputs of z-lines m of tile zt: x_0, x_r, x_{n-r}
  float2 x0, xa[SY], xm[SY];
  auto y_load = [&](int zt, int c, int lane) {
    const int g = lane >> 4, m = lane & 15;
    const unsigned base = unsigned(min(16 * zt + m, nz - 1) * ny) * unsigned(ct) + unsigned(c);
    x0 = in[base];
    if (ct == 1) {
      // (pairs, traded between the lanes before use)
      const float2 *up = in + base + (2 * g + 1), *dn = in + base + (ny - 2 * g - 2);
#pragma unroll
      for (int s = 0; s < SY; s += 2) {
        ld2(up + dense3_input(s, 0), xa[s], xa[s + 1]);
        ld2(dn - dense3_input(s, 0), xm[s + 1], xm[s]);
      }
    } else {
      const unsigned r0 = unsigned(dense3_input_y(0, g) + 1);
      const unsigned lo = base + r0 * unsigned(ct), hi = base + (unsigned(ny) - r0) * unsigned(ct);
#pragma unroll
      for (int s = 0; s < SY; ++s) {
        xa[s] = in[lo + unsigned(dense3_input(s, 0) * ct)];
        xm[s] = in[hi - unsigned(dense3_input(s, 0) * ct)];
      }
    }
  };
  // k-space factors of rows q = dense3_input(4 mt + i, g) and n - q of register i, row tile mt, column ky
  float kf[MZ][4][2];
  float2 one;
  auto sym_load = [&](int kt, int col, int lane) {
    const int g = lane >> 4, m = lane & 15, ky = min(16 * kt + m, ny - 1);
    const float* tab = (cd == OP_LDIS ? M.ldis : cd == OP_LABS ? M.labs : M.kap) + size_t(col) * nl;
    one = cd == OP_DXP ? M.dxp[col] : cd == OP_DXM ? M.dxm[col] : cd == OP_DYP ? M.dyp[ky]
          : cd == OP_DYM ? M.dym[ky] : make_float2(1.f, 0.f);
    const unsigned lo = unsigned(g * ny + ky), hi = unsigned((nz - g) * ny + ky);
#pragma unroll
    for (int mt = 0; mt < MZ; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const unsigned d = unsigned(dense3_input(4 * mt + i, 0) * ny);
        kf[mt][i][0] = tab[lo + d];
        kf[mt][i][1] = tab[(mt == 0 && i == 0 && g == 0) ? lo : hi - d];   // the mirror of row 0 is row 0
      }
  };
  // (no branch on the operator: the factors of all rows are read together)
  auto sym_mul = [&](float k, int q, float2 v) {
    const float2 zs = lz[q], s = make_float2(hasz ? zs.x : one.x, hasz ? zs.y : one.y);
    return cmul(v, cscale(s, k));
  };

  // ---- load phase: the first column's y-lines, the matrices, the multipliers
  if (w < NTz) y_load(w, 0, tid & 63);
  Mat<SY> Ay[MY];
  Mat<SZ> Az[MZ];
  Mat<4 * MZ> Ac[MZ];
#pragma unroll
  for (int mt = 0; mt < MY; ++mt) mat_load(Ay[mt], M.dfy, mt, tid & 63);
  if (w < NTy) sym_load(w, c0, tid & 63);
#pragma unroll
  for (int mt = 0; mt < MZ; ++mt) mat_load(Az[mt], M.dfz, mt, tid & 63);
  if (hasz)
    for (int i = tid; i < nz; i += blockDim.x) lz[i] = (cd == OP_DZP ? M.dzp : M.dzm)[i];

  for (int c = 0; c < ncols; ++c) {
    if (c > 0) __syncthreads();   // the plane of the column before is still being read
    // ---- y forward
    for (int zt = w; zt < NTz; zt += nw) {
      const int lane = opaque(tid & 63), g = lane >> 4, m = lane & 15;
      if (c > 0 || zt != w) y_load(zt, c, lane);
      if (ct == 1) {
#pragma unroll
        for (int s = 0; s < SY; s += 2) half_swap(xa[s], xa[s + 1]), half_swap(xm[s], xm[s + 1]);
      }
      float2 e[SY], o[SY];
#pragma unroll
      for (int s = 0; s < SY; ++s) e[s] = cadd(xa[s], xm[s]), o[s] = csub(xa[s], xm[s]);
      const int z = 16 * zt + m;
      float2 *lo = lds2 + z * LY + 4 * g, *hi = lds2 + z * LY + ny - 4 * g;
#pragma unroll
      for (int mt = 0; mt < MY; ++mt) {
        const Acc acc = tile_products<false>(x0, e, o, Ay[mt]);
        if (z < nz)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float2 a, b;
            acc_out<false>(acc, i, a, b);
            lo[16 * mt + i] = a;
            hi[-(16 * mt + i)] = b;   // q = 0: the slot past the line
          }
      }
    }
    __syncthreads();
    // ---- z forward, multiplier, z inverse (columns ky of tile kt, this wave's own)
    for (int kt = w; kt < NTy; kt += nw) {
      const int lane = opaque(tid & 63), g = lane >> 4, m = lane & 15;
      if (c > 0 || kt != w) sym_load(kt, c0 + c, lane);
      const int ky = 16 * kt + m;
      const float2* src = lds2 + min(ky, ny - 1);
      const float2 *up = src + (g + 1) * LY, *dn = src + (nz - g - 1) * LY;
      const float2 z0 = src[0];
#pragma unroll
      for (int mt = 0; mt < MZ; ++mt) mat_load(Ac[mt], M.dfzc, mt, lane);   // arrives over the z forward products
      float2 e[SZ], o[SZ];
#pragma unroll
      for (int s = 0; s < SZ; ++s) {
        const float2 a = up[dense3_input(s, 0) * LY], b = dn[-dense3_input(s, 0) * LY];
        e[s] = cadd(a, b), o[s] = csub(a, b);
      }
      // multiplied rows q and n - q, folded again: the inputs of the inverse
      float2 ei[4 * MZ], oi[4 * MZ];
#pragma unroll
      for (int mt = 0; mt < MZ; ++mt) {
        const Acc acc = tile_products<false>(z0, e, o, Az[mt]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int q = dense3_input(4 * mt + i, g);
          float2 a, b;
          acc_out<false>(acc, i, a, b);
          a = sym_mul(kf[mt][i][0], q, a);
          b = sym_mul(kf[mt][i][1], (mt == 0 && i == 0 && g == 0) ? 0 : nz - q, b);
          ei[4 * mt + i] = cadd(a, b), oi[4 * mt + i] = csub(a, b);
        }
      }
#pragma unroll
      for (int mt = 0; mt < MY; ++mt) mat_load(Ay[mt], M.dfy, mt, lane);   // again: held over the z products they spill
      // rows past n/2 and the mirror of row 0 fall on rows written already, with the same bits
      float2 *lo = lds2 + 4 * g * LY + ky, *hi = lds2 + (nz - 4 * g) * LY + ky;
#pragma unroll
      for (int mt = 0; mt < MZ; ++mt) {
        const Acc acc = tile_products<true>(make_float2(0.f, 0.f), ei, oi, Ac[mt]);
        if (ky < ny)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float2 a, b;
            acc_out<true>(acc, i, a, b);
            lo[(16 * mt + i) * LY] = a;
            float2* h = hi - (16 * mt + i) * LY;
            if (mt == 0 && i == 0) h = g == 0 ? lo : h;
            *h = b;
          }
      }
    }
    __syncthreads();
    // ---- y inverse, to global memory
    for (int zt = w; zt < NTz; zt += nw) {
      const int lane = opaque(tid & 63), g = lane >> 4, m = lane & 15;
      const int z = 16 * zt + m;
      const float2* src = lds2 + min(z, nz - 1) * LY;
      const float2 *up = src + 2 * g + 1, *dn = src + (ny - 2 * g - 1);
      const float2 y0 = src[0];
      float2 e[SY], o[SY];
#pragma unroll
      for (int s = 0; s < SY; s += 2) {
        const int d = dense3_input(s, 0);
        const float2 a = up[d], b = dn[-d], a1 = up[d + 1], b1 = dn[-d - 1];
        e[s] = cadd(a, b), o[s] = csub(a, b);
        e[s + 1] = cadd(a1, b1), o[s + 1] = csub(a1, b1);
        half_swap(e[s], e[s + 1]), half_swap(o[s], o[s + 1]);
      }
      float2* dst = out + unsigned(z * ny) * unsigned(ct) + c;
#pragma unroll
      for (int mt = 0; mt < MY; ++mt) {
        const Acc acc = tile_products<true>(y0, e, o, Ay[mt]);
        if (z < nz) {
          const int j = 16 * mt + 4 * g;   // rows j .. j + 3 and their mirrors
          float2 a[4], b[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) acc_out<true>(acc, i, a[i], b[i]);
          if (ct == 1) {
            // (a group that straddles n/2 stores some rows twice, the same bits)
            if (j <= nyh) {
              st2(dst + j, a[0], a[1]);
              st2(dst + j + 2, a[2], a[3]);
            }
            if (2 * j < ny) {
              float2* h = dst + ny - j;
              st2(h - 3, b[3], b[2]);
              if (mt > 0 || g > 0) st2(h - 1, b[1], b[0]);
              else h[-1] = b[1];   // row 0 is its own mirror
            }
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (j + i <= nyh) dst[unsigned((j + i) * ct)] = a[i];
              if (j + i >= 1 && 2 * (j + i) < ny) dst[unsigned((ny - j - i) * ct)] = b[i];
            }
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------- launchers
template <int MODE, int C>
static hipError_t row_c(const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  const int G = (L.m.rt + 15) / 16, thr = L.m.rthr < kDenseThreads ? L.m.rthr : kDenseThreads;
  const size_t lds = size_t(row_fields<MODE>()) * G * 16 * line_stride<C>() * sizeof(float);
  hipLaunchKernelGGL((row3_dense_kernel<MODE, C>), dim3(chunk * kXcds), dim3(thr), lds, st, L, ntile, chunk, n);
  return hipGetLastError();
}
template <int MODE>
static hipError_t row_t(const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  switch (dense3_class(L.m.nx)) {
    case 0: return row_c<MODE, 0>(L, ntile, chunk, n, st);
    case 1: return row_c<MODE, 1>(L, ntile, chunk, n, st);
    case 2: return row_c<MODE, 2>(L, ntile, chunk, n, st);
    default: return row_c<MODE, 3>(L, ntile, chunk, n, st);
  }
}

hipError_t launch_row3_dense(int mode, const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  switch (mode) {
    case R3_F1: return row_t<R3_F1>(L, ntile, chunk, n, st);
    case R3_F2: return row_t<R3_F2>(L, ntile, chunk, n, st);
    case R3_F2L: return row_t<R3_F2L>(L, ntile, chunk, n, st);
    case R3_F3: return row_t<R3_F3>(L, ntile, chunk, n, st);
    case R3_A1: return row_t<R3_A1>(L, ntile, chunk, n, st);
    case R3_A1L: return row_t<R3_A1L>(L, ntile, chunk, n, st);
    case R3_A2: return row_t<R3_A2>(L, ntile, chunk, n, st);
    case R3_A3: return row_t<R3_A3>(L, ntile, chunk, n, st);
    case R3_FWD1: return row_t<R3_FWD1>(L, ntile, chunk, n, st);
    case R3_INV1: return row_t<R3_INV1>(L, ntile, chunk, n, st);
    default: return hipErrorInvalidValue;
  }
}

template <int CY, int CZ>
static hipError_t plane_c(const Launch3& L, int ntile, int chunk, const PlaneOps& P, int n, hipStream_t st) {
  // (four waves cover the at most four tiles of either axis)
  const int thr = L.m.pthr < 256 ? L.m.pthr : 256;
  const size_t lds = size_t(L.m.nz) * (plane_stride<CY>() + 1) * sizeof(float2);
  hipLaunchKernelGGL((plane3_dense_kernel<CY, CZ>), dim3(chunk * kXcds), dim3(thr), lds, st, L, ntile, chunk, P, n);
  return hipGetLastError();
}
template <int CY>
static hipError_t plane_y(const Launch3& L, int ntile, int chunk, const PlaneOps& P, int n, hipStream_t st) {
  switch (dense3_class(L.m.nz)) {
    case 0: return plane_c<CY, 0>(L, ntile, chunk, P, n, st);
    case 1: return plane_c<CY, 1>(L, ntile, chunk, P, n, st);
    case 2: return plane_c<CY, 2>(L, ntile, chunk, P, n, st);
    default: return plane_c<CY, 3>(L, ntile, chunk, P, n, st);
  }
}

hipError_t launch_plane3_dense(int mode, int code, const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  PlaneOps P{plane3_split(mode), mode == P3_GRADP1 ? 3 : -1, {code, code, code}};
  for (int f = 0; f < 3; ++f) {
    switch (mode) {
      case P3_GRADP1: P.code[f] = plane_code<P3_GRADP1>(f, code); break;
      case P3_GRADM2: P.code[f] = plane_code<P3_GRADM2>(f, code); break;
      case P3_FRAC: P.code[f] = plane_code<P3_FRAC>(f, code); break;
      case P3_GRADP2: P.code[f] = plane_code<P3_GRADP2>(f, code); break;
      case P3_APPLY: break;
      default: return hipErrorInvalidValue;
    }
  }
  switch (dense3_class(L.m.ny)) {
    case 0: return plane_y<0>(L, ntile, chunk, P, n, st);
    case 1: return plane_y<1>(L, ntile, chunk, P, n, st);
    case 2: return plane_y<2>(L, ntile, chunk, P, n, st);
    default: return plane_y<3>(L, ntile, chunk, P, n, st);
  }
}

}  // namespace qpat3

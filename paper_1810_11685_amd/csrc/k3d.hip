// 3-D k-space PSTD passes for gfx950 (Section 3.2.3 with d = 3).
//
// One iterate is three (row pass, plane pass) pairs, as in 2-D:
//   row pass   - rt consecutive x-lines: inverse x-FFT of the incoming half
//                spectra (two real lines per complex FFT), the pointwise
//                update of the scheme, forward x-FFT of the outgoing fields;
//   plane pass - ct spectrum columns of every y-z plane: forward y- and
//                z-FFTs, the k-space multiplier, inverse z- and y-FFTs.
// The FFTs are mixed-radix Stockham transforms in LDS with a runtime plan per
// axis: radices 2, 3, 4, 5, 7, 8 as butterflies, any other prime factor as a
// direct DFT stage, so any length runs without padding.  Axes of 18 to 63 points
// are transformed as matrix products instead (k3d_dense.hip; dense3 and
// dense3_plane say which); lengths of two equal stages have kernels of their own
// (staged3).
#include "k3d_device.hpp"

namespace qpat3 {

// ---------------------------------------------------------------- small DFTs
// cos and sin of 2 pi m / R for the odd radices (folded at compile time).
__host__ __device__ constexpr float ucos(int R, int m) {
  return R == 3 ? (m == 0 ? 1.0f : -0.5f)
       : R == 5 ? (m == 0 ? 1.0f : (m == 1 || m == 4) ? 0.309016994f : -0.809016994f)
       : (m == 0 ? 1.0f : (m == 1 || m == 6) ? 0.623489802f : (m == 2 || m == 5) ? -0.222520934f : -0.900968868f);
}
__host__ __device__ constexpr float usin(int R, int m) {
  return R == 3 ? (m == 0 ? 0.0f : m == 1 ? 0.866025404f : -0.866025404f)
       : R == 5 ? (m == 0 ? 0.0f : m == 1 ? 0.951056516f : m == 2 ? 0.587785252f : m == 3 ? -0.587785252f
                                                                                    : -0.951056516f)
       : (m == 0 ? 0.0f : m == 1 ? 0.781831482f : m == 2 ? 0.974927912f : m == 3 ? 0.433883739f
          : m == 4 ? -0.433883739f : m == 5 ? -0.974927912f : -0.781831482f);
}

// x * (-i) (forward) or x * (+i) (inverse)
template <bool INV>
__device__ __forceinline__ float2 rot90(float2 x) {
  return INV ? make_float2(-x.y, x.x) : make_float2(x.y, -x.x);
}

template <int R, bool INV>
__device__ __forceinline__ void dft(float2* v) {
  if constexpr (R == 2) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const float2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const float2 s13 = cadd(v[1], v[3]), d13 = rot90<INV>(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, d13);
    v[3] = csub(d02, d13);
  } else if constexpr (R == 8) {
    float2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft<4, INV>(e);
    dft<4, INV>(o);
    constexpr float h = 0.707106781f;
    const float2 w1 = INV ? make_float2(h, h) : make_float2(h, -h);
    const float2 w3 = INV ? make_float2(-h, h) : make_float2(-h, -h);
    o[1] = cmul(o[1], w1);
    o[2] = rot90<INV>(o[2]);
    o[3] = cmul(o[3], w3);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = cadd(e[q], o[q]);
      v[q + 4] = csub(e[q], o[q]);
    }
  } else {
    // odd R: pair inputs r and R - r.  With a_r = x_r + x_{R-r} and
    // b_r = x_r - x_{R-r}, output q is x_0 + sum_r cos(2 pi r q / R) a_r
    // -+ i sum_r sin(2 pi r q / R) b_r, and output R - q takes the other sign.
    constexpr int H = (R - 1) / 2;
    float2 a[H], b[H];
#pragma unroll
    for (int r = 1; r <= H; ++r) {
      a[r - 1] = cadd(v[r], v[R - r]);
      b[r - 1] = csub(v[r], v[R - r]);
    }
    float2 y0 = v[0];
#pragma unroll
    for (int r = 0; r < H; ++r) y0 = cadd(y0, a[r]);
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      float2 A = v[0], S = make_float2(0.f, 0.f);
#pragma unroll
      for (int r = 1; r <= H; ++r) {
        const int m = (r * q) % R;
        const float c = ucos(R, m), sn = usin(R, m);
        A.x += c * a[r - 1].x;
        A.y += c * a[r - 1].y;
        S.x += sn * b[r - 1].x;
        S.y += sn * b[r - 1].y;
      }
      // forward: y_q = A - i S, y_{R-q} = A + i S (inverse: the signs swap)
      const float2 iS = make_float2(-S.y, S.x);
      v[q] = INV ? cadd(A, iS) : csub(A, iS);
      v[R - q] = INV ? csub(A, iS) : cadd(A, iS);
    }
    v[0] = y0;
  }
}

// ---------------------------------------------------------------- LDS line FFTs
// Element e of line L sits at line_off(L) + e * es, line_off(L) = (L / lpg) *
// gs + (L % lpg) * ls: x-lines of a row block, y- and z-lines of a plane block.
struct LineMap {
  int nlines, lpg, gs, ls, es;
};
__device__ __forceinline__ unsigned line_off(const LineMap m, unsigned L, float rlpg) {
  const unsigned g = unsigned(udiv(int(L), rlpg));
  return __umul24(g, unsigned(m.gs)) + __umul24(L - __umul24(g, unsigned(m.lpg)), unsigned(m.ls));
}

// One Stockham stage of radix R over every line: butterfly j (of n/R) reads
// src[j + r n/R], twiddles input r by w^(r k n/(Ns R)) with k = j mod Ns, and
// writes dst[(j - k) R + k + r Ns].  Every index is below 2^24, so products
// take the 24-bit multiplier, and the strides between a butterfly's inputs
// and outputs are block-uniform.
template <int R, bool INV>
__device__ void stage_small(const float2* __restrict__ src, float2* __restrict__ dst, const LineMap m, int n,
                            int Ns, const float2* __restrict__ tw) {
  const unsigned nb = unsigned(n / R), ns = unsigned(Ns), tstep = unsigned(n / (Ns * R));
  const unsigned total = unsigned(m.nlines) * nb, es = unsigned(m.es);
  const unsigned istep = nb * es, ostep = ns * es;
  const float rnb = rcp(nb), rns = rcp(Ns), rlpg = rcp(m.lpg);
  for (unsigned t = threadIdx.x; t < total; t += blockDim.x) {
    const unsigned L = unsigned(udiv(int(t), rnb)), j = t - __umul24(L, nb);
    const unsigned off = line_off(m, L, rlpg);
    const unsigned k = j - __umul24(unsigned(udiv(int(j), rns)), ns);
    const float2* s = src + (off + __umul24(j, es));
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[r * istep];
    if (Ns > 1) {  // the first stage's twiddles are all 1 (block-uniform test)
      const unsigned kt = __umul24(k, tstep);
      unsigned e = 0;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        e += kt;   // r k tstep
        float2 w = tw[e];
        if (INV) w.y = -w.y;
        v[r] = cmul(v[r], w);
      }
    }
    dft<R, INV>(v);
    float2* d = dst + (off + __umul24(__umul24(j - k, unsigned(R)) + k, es));
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * ostep] = v[r];
  }
}

// A stage of an odd prime radix R without a butterfly of its own, in the
// symmetric form of the odd butterflies: with the twiddled inputs x_r of
// butterfly j, a_r = x_r + x_{R-r} and b_r = x_r - x_{R-r} (r = 1 .. H,
// H = (R - 1) / 2), output q is x_0 + sum_r cos(2 pi r q / R) a_r
// -+ i sum_r sin(2 pi r q / R) b_r and output R - q takes the other sign.  A
// work item is one butterfly and one q in [0, H] (q = 0: the sum of all
// inputs), so each pair of outputs shares its loads and its H products.
template <bool INV>
__device__ void stage_generic(const float2* __restrict__ src, float2* __restrict__ dst, const LineMap m, int n,
                              int Ns, int R, const float2* __restrict__ tw) {
  const int nb = n / R, tstep = n / (Ns * R), H = (R - 1) / 2, per = nb * (H + 1);
  const int total = m.nlines * per;
  const unsigned es = unsigned(m.es), istep = unsigned(nb) * es;
  const float rper = rcp(per), rnb = rcp(nb), rns = rcp(Ns), rlpg = rcp(m.lpg);
  for (int t = threadIdx.x; t < total; t += blockDim.x) {
    const int L = udiv(t, rper), it = t - L * per;
    const int q = udiv(it, rnb), j = it - q * nb;   // butterflies fastest
    const unsigned off = line_off(m, unsigned(L), rlpg);
    const int k = j - udiv(j, rns) * Ns, kt = k * tstep;  // input twiddle step (r kt < n)
    const float2* s = src + (off + __umul24(unsigned(j), es));
    // twiddled input r (conjugated twiddle for the inverse)
    auto input = [&](int r) {
      const float2 x = s[unsigned(r) * istep];
      if (kt == 0) return x;
      float2 w = tw[r * kt];
      if (INV) w.y = -w.y;
      return cmul(x, w);
    };
    const float2 x0 = input(0);
    float2 A = x0, S = make_float2(0.f, 0.f);
    int p = 0;   // (r q) mod R
    for (int r = 1; r <= H; ++r) {
      const float2 xr = input(r), xm = input(R - r);
      const float2 a = cadd(xr, xm), b = csub(xr, xm);
      if (q == 0) {
        A = cadd(A, a);
      } else {
        p += q;
        if (p >= R) p -= R;
        const float2 w = tw[p * nb];   // cos(2 pi p / R) - i sin(2 pi p / R)
        const float c = w.x, sn = -w.y;
        A.x += c * a.x;
        A.y += c * a.y;
        S.x += sn * b.x;
        S.y += sn * b.y;
      }
    }
    const int base = (j - k) * R + k;
    if (q == 0) {
      dst[off + __umul24(unsigned(base), es)] = A;
    } else {
      // forward: y_q = A - i S, y_{R-q} = A + i S (the inverse swaps them)
      const float2 iS = make_float2(-S.y, S.x);
      dst[off + __umul24(unsigned(base + q * Ns), es)] = INV ? cadd(A, iS) : csub(A, iS);
      dst[off + __umul24(unsigned(base + (R - q) * Ns), es)] = INV ? csub(A, iS) : cadd(A, iS);
    }
  }
}

// The stage of stage_small for a compile-time length N and stage (radix R,
// NS = product of the earlier radices): the butterfly count, twiddle step and
// k = j mod NS fold to constants, leaving the line offset as the only index
// arithmetic done at run time.  Same operations in the same order.
template <int R, bool INV, int N, int NS>
__device__ __forceinline__ void stage_ct(const float2* __restrict__ src, float2* __restrict__ dst, const LineMap m,
                                         const float2* __restrict__ tw) {
  constexpr unsigned NB = N / R, TSTEP = N / (NS * R);
  constexpr float RNB = 1.0f / float(NB);
  const unsigned total = unsigned(m.nlines) * NB, es = unsigned(m.es);
  const unsigned istep = NB * es, ostep = NS * es;
  const float rlpg = rcp(m.lpg);
  for (unsigned t = threadIdx.x; t < total; t += blockDim.x) {
    const unsigned L = unsigned(udiv(int(t), RNB)), j = t - L * NB;
    const unsigned off = line_off(m, L, rlpg);
    // j < NB, so k = j mod NS is 0 in a first stage and j once NS >= NB
    const unsigned k = NS == 1 ? 0u : (NS >= int(NB) ? j : j % NS);
    const float2* s = src + (off + __umul24(j, es));
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[r * istep];
    if constexpr (NS > 1) {
      const unsigned kt = k * TSTEP;
      unsigned e = 0;
#pragma unroll
      for (int r = 1; r < R; ++r) {
        e += kt;   // r k tstep
        float2 w = tw[e];
        if (INV) w.y = -w.y;
        v[r] = cmul(v[r], w);
      }
    }
    dft<R, INV>(v);
    float2* d = dst + (off + __umul24((j - k) * R + k, es));
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * ostep] = v[r];
  }
}

// The runtime plan of an axis: every stage through stage_small or
// stage_generic (barrier after each); returns the buffer holding the result.
template <bool INV>
__device__ __forceinline__ float2* fft_axis_rt(float2* a, float2* b, const LineMap m, const AxisPlan P,
                                               const float2* tw) {
  // radices packed 8 bits a stage: a dynamic index into P would put P in scratch
  unsigned long long rad = 0;
#pragma unroll
  for (int st = 0; st < kMaxStages; ++st) rad |= (unsigned long long)(P.r[st] & 255) << (8 * st);
  float2* s = a;
  float2* d = b;
  int Ns = 1;
  for (int st = 0; st < P.nst; ++st) {
    const int R = int((rad >> (8 * st)) & 255);
    switch (R) {
      case 2: stage_small<2, INV>(s, d, m, P.n, Ns, tw); break;
      case 3: stage_small<3, INV>(s, d, m, P.n, Ns, tw); break;
      case 4: stage_small<4, INV>(s, d, m, P.n, Ns, tw); break;
      case 5: stage_small<5, INV>(s, d, m, P.n, Ns, tw); break;
      case 7: stage_small<7, INV>(s, d, m, P.n, Ns, tw); break;
      case 8: stage_small<8, INV>(s, d, m, P.n, Ns, tw); break;
      default: stage_generic<INV>(s, d, m, P.n, Ns, R, tw); break;
    }
    __syncthreads();
    float2* t = s;
    s = d;
    d = t;
    Ns *= R;
  }
  return s;
}

// All stages of one axis (barrier after each); returns the buffer holding the
// result (a or b).  AX is the axis length of a kernel instance whose every
// transformed axis has that length (49 = 7 x 7 and 64 = 8 x 8: compile-time
// stages only, no runtime plan in the instance); AX = 0 runs the runtime plan.
// The launchers pick AX from the plan's axis lengths.
template <bool INV, int AX>
__device__ __forceinline__ float2* fft_axis(float2* a, float2* b, const LineMap m, const AxisPlan P,
                                            const float2* tw) {
  if constexpr (AX == 0) {
    return fft_axis_rt<INV>(a, b, m, P, tw);
  } else {
    constexpr int R = staged3(AX);
    static_assert(R * R == AX, "two equal stages");
    stage_ct<R, INV, AX, 1>(a, b, m, tw);
    __syncthreads();
    stage_ct<R, INV, AX, R>(b, a, m, tw);
    __syncthreads();
    return a;
  }
}

// ---------------------------------------------------------------- row pass
// value of line j2 (of the tile) of field f in a buffer of paired lines
__device__ __forceinline__ float& pc(float2* buf, int hp, int nx, int f, int j2, int x) {
  float2& z = buf[(f * hp + (j2 >> 1)) * nx + x];
  return (j2 & 1) ? z.y : z.x;
}

template <int MODE, int AX>
__global__ void __launch_bounds__(kRowMax) row3_kernel(const Launch3 L, int ntile, int chunk, int n) {
  args3_batch(L, ntile, chunk, n);
  asm volatile("" ::"s"(L.m.twx), "s"(L.m.dt), "s"(L.m.ns));
  int item, tile;
  if (!locate(L.nitems, ntile, chunk, item, tile)) return;
  const Medium3& M = L.m;
  const Work3 W = shift(L.w0, item * L.wstride);
  const IO3 X = L.io[item];
  const int nx = M.nx, ny = M.ny, rt = M.rt, hp = rt / 2, nl = M.nlines;
  const int l0 = tile * rt;
  const unsigned N = unsigned(nl) * unsigned(nx);
  const int B = blockDim.x, tid = threadIdx.x;
  extern __shared__ float2 lds[];
  float2* bufA = lds;
  float2* bufB = lds + 3 * hp * nx;
  float2* tw = lds + 6 * hp * nx;
  int nin, nout;
  row_counts<MODE>(M, n, nin, nout);
  const bool first = (n == M.nt - 2);
  const float dt = M.dt;

  for (int i = tid; i < nx; i += B) tw[i] = M.twx[i];
  // incoming half spectra -> full spectra of the paired lines (a + i b)
  const int ncol = M.nxh1;
  const float rhp = rcp(hp), rncol = rcp(ncol), rnx = rcp(nx), rny = rcp(ny);
  // the adjoint divergence arrives as its three terms d_i^- g_i, one per
  // spectrum, summed here in a fixed order
  constexpr int NSUM = (MODE == R3_A1 || MODE == R3_A1L) ? 3 : 1;
  for (int t = tid; t < nin * ncol * hp; t += B) {
    const int fc = udiv(t, rhp), j = t - fc * hp, f = udiv(fc, rncol), c = fc - f * ncol;
    const int la = l0 + 2 * j, lb = la + 1;
    float2 a = make_float2(0.f, 0.f), b = make_float2(0.f, 0.f);
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
      if (la < nl) a = cadd(a, W.s[spec_index(M, f + k, c, la)]);
      if (lb < nl) b = cadd(b, W.s[spec_index(M, f + k, c, lb)]);
    }
    float2* Z = bufA + (f * hp + j) * nx;
    Z[c] = make_float2(a.x - b.y, a.y + b.x);
    if (c != 0 && 2 * c != nx) Z[nx - c] = make_float2(a.x + b.y, b.x - a.y);
  }
  if (nin == 0) {
    for (int t = tid; t < 3 * hp * nx; t += B) bufA[t] = make_float2(0.f, 0.f);
  }
  __syncthreads();
  float2* R = bufA;
  if (nin > 0) {
    const LineMap lm{nin * hp, nin * hp, 0, nx, 1};
    R = fft_axis<true, AX>(bufA, bufB, lm, M.px, tw);
  }
  float2* O = (R == bufA) ? bufB : bufA;

  if constexpr (MODE == R3_A1 || MODE == R3_A1L) {
    // p* = -(sum_i d_i^- g_i) + M^T r_{n+1}
    for (int t = tid; t < hp * nx; t += B) {
      const float2 z = R[t];
      R[t] = make_float2(-z.x, -z.y);
    }
    __syncthreads();
    {
      // one thread per receiving node, its entries summed in a fixed order
      const float* r = X.in + size_t(n + 1) * M.ns;
      const int a = M.node_off[l0], b = M.node_off[min(l0 + rt, nl)];
      for (int k = a + tid; k < b; k += B) {
        const ScatterNode nd = M.nodes[k];
        float acc = 0.f;
        for (int e = nd.e0; e < nd.e1; ++e) {
          const ScatterEntry en = M.entries[e];
          acc += en.w * r[en.s];
        }
        pc(R, hp, nx, 0, nd.line - l0, nd.ix) += acc;
      }
    }
    __syncthreads();
  }

  for (int t = tid; t < rt * nx; t += B) {
    const int j2 = udiv(t, rnx), x = t - j2 * nx, l = l0 + j2;
    if (l >= nl) {
      for (int o = 0; o < nout; ++o) pc(O, hp, nx, o, j2, x) = 0.f;
      continue;
    }
    const int z = udiv(l, rny), y = l - z * ny;
    const unsigned idx = unsigned(l) * unsigned(nx) + unsigned(x);
    float* const fv = W.f;   // v_x v_y v_z rho_x rho_y rho_z q
    if constexpr (MODE == R3_F1) {
      const float av[3] = {M.avx[x], M.avy[y], M.avz[z]};
      const float bb[3] = {M.bx[idx], M.by[idx], M.bz[idx]};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const float g = pc(R, hp, nx, i, j2, x);
        const float vo = (n == 0) ? 0.f : fv[i * N + idx];
        const float v = av[i] * (av[i] * vo - bb[i] * g);
        fv[i * N + idx] = v;
        pc(O, hp, nx, i, j2, x) = v;
      }
    } else if constexpr (MODE == R3_F2 || MODE == R3_F2L) {
      const bool skip = (n == -1);
      const float ar[3] = {M.arx[x], M.ary[y], M.arz[z]};
      const float r0 = M.rho0[idx], c2 = M.c2[idx];
      const float src = (n <= 0) ? X.in[idx] * (1.0f / 6.0f) / c2 : 0.f;   // p0 / (2 d c^2), d = 3
      float S = 0.f, u = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const float e = skip ? 0.f : pc(R, hp, nx, i, j2, x);
        const float ro = skip ? 0.f : fv[(3 + i) * N + idx];
        const float rho = ar[i] * (ar[i] * ro - dt * r0 * e) + src;
        fv[(3 + i) * N + idx] = rho;
        S += rho;
        u += ar[i] * e;
      }
      if constexpr (MODE == R3_F2) {
        pc(O, hp, nx, 0, j2, x) = S;
        pc(O, hp, nx, 1, j2, x) = r0 * u;
      } else {
        pc(O, hp, nx, 0, j2, x) = c2 * S;
      }
    } else if constexpr (MODE == R3_F3) {
      const float S = fv[3 * N + idx] + fv[4 * N + idx] + fv[5 * N + idx];
      const float ys = pc(R, hp, nx, 0, j2, x), yu = pc(R, hp, nx, 1, j2, x);
      pc(O, hp, nx, 0, j2, x) = M.c2[idx] * S - M.c2eta[idx] * ys + M.c2tau[idx] * yu;
    } else if constexpr (MODE == R3_A1) {
      const float pb = pc(R, hp, nx, 0, j2, x);
      fv[6 * N + idx] = M.c2[idx] * pb;
      pc(O, hp, nx, 0, j2, x) = M.c2eta[idx] * pb;
      pc(O, hp, nx, 1, j2, x) = M.c2tau[idx] * pb;
    } else if constexpr (MODE == R3_A1L || MODE == R3_A2) {
      const float ar[3] = {M.arx[x], M.ary[y], M.arz[z]};
      const float r0 = M.rho0[idx], c2 = M.c2[idx];
      float sb, ub;
      if constexpr (MODE == R3_A1L) {
        sb = c2 * pc(R, hp, nx, 0, j2, x);
        ub = 0.f;
      } else {
        sb = fv[6 * N + idx] - pc(R, hp, nx, 0, j2, x);
        ub = pc(R, hp, nx, 1, j2, x);
      }
      float rb[3], sum = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        rb[i] = (first ? 0.f : fv[(3 + i) * N + idx]) + sb;
        sum += rb[i];
      }
      if (n == 0) X.out[idx] = sum;
      if (n == -1) {
        const float acc = M.nt >= 2 ? X.out[idx] : 0.f;
        X.out[idx] = (sum + acc) * (1.0f / 6.0f) / c2;
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          pc(O, hp, nx, i, j2, x) = r0 * ar[i] * (ub - dt * rb[i]);
          fv[(3 + i) * N + idx] = ar[i] * ar[i] * rb[i];
        }
      }
    } else if constexpr (MODE == R3_A3) {
      const float av[3] = {M.avx[x], M.avy[y], M.avz[z]};
      const float bb[3] = {M.bx[idx], M.by[idx], M.bz[idx]};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const float vb = (first ? 0.f : fv[i * N + idx]) - pc(R, hp, nx, i, j2, x);
        pc(O, hp, nx, i, j2, x) = -av[i] * bb[i] * vb;
        fv[i * N + idx] = av[i] * av[i] * vb;
      }
    } else if constexpr (MODE == R3_FWD1) {
      pc(O, hp, nx, 0, j2, x) = X.in[idx];
    } else {  // R3_INV1
      X.out[idx] = pc(R, hp, nx, 0, j2, x);
    }
  }
  __syncthreads();

  if constexpr (MODE == R3_F2L || MODE == R3_F3) {
    // sensor partials of this tile's lines: part[n+1][s][slot]
    const int e0 = M.tap_off[l0], e1 = M.tap_off[min(l0 + rt, nl)];
    for (int e = e0 + tid; e < e1; e += B) {
      const Tap3 tp = M.taps[e];
      const int j2 = tp.line - l0;
      W.part[(size_t(n + 1) * M.ns + tp.s) * 4 + tp.slot] =
          tp.wl * pc(O, hp, nx, 0, j2, tp.ixl) + tp.wr * pc(O, hp, nx, 0, j2, tp.ixr);
    }
  }
  if (nout == 0) return;

  // outgoing fields -> half spectra of each line
  const LineMap lm{nout * hp, nout * hp, 0, nx, 1};
  float2* Z = fft_axis<false, AX>(O, R, lm, M.px, tw);
  for (int t = tid; t < nout * ncol * hp; t += B) {
    const int oc = udiv(t, rhp), j = t - oc * hp, o = udiv(oc, rncol), c = oc - o * ncol;
    const float2* Zl = Z + (o * hp + j) * nx;
    const float2 zk = Zl[c], zm = Zl[c == 0 ? 0 : nx - c];
    const int la = l0 + 2 * j, lb = la + 1;
    // the pressure goes to spectrum 3, which the gradient pass reads while it
    // writes spectra 0..2
    const int of = (MODE == R3_F2L || MODE == R3_F3) ? 3 : o;
    if (la < nl) W.s[spec_index(M, of, c, la)] = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    if (lb < nl) W.s[spec_index(M, of, c, lb)] = make_float2(0.5f * (zk.y + zm.y), 0.5f * (zm.x - zk.x));
  }
}

// ---------------------------------------------------------------- plane pass
__device__ __forceinline__ float2 symbol(const Medium3& M, int code, int col, int y, int z) {
  const size_t k = size_t(col) * M.nlines + size_t(z) * M.ny + y;
  switch (code) {
    case OP_DXP: return cscale(M.dxp[col], M.kap[k]);
    case OP_DXM: return cscale(M.dxm[col], M.kap[k]);
    case OP_DYP: return cscale(M.dyp[y], M.kap[k]);
    case OP_DYM: return cscale(M.dym[y], M.kap[k]);
    case OP_DZP: return cscale(M.dzp[z], M.kap[k]);
    case OP_DZM: return cscale(M.dzm[z], M.kap[k]);
    case OP_LDIS: return make_float2(M.ldis[k], 0.f);
    default: return make_float2(M.labs[k], 0.f);
  }
}

template <int MODE, int AX>
__global__ void __launch_bounds__(kPlaneMax) plane3_kernel(const Launch3 L, int ntile, int chunk, int code, int n) {
  args3_batch(L, ntile, chunk, n);
  asm volatile("" ::"s"(L.m.twy), "s"(L.m.twz), "s"(code));
  int item, tile;
  if (!locate(L.nitems, ntile, chunk, item, tile)) return;
  const Medium3& M = L.m;
  constexpr int NSPLIT = plane3_split(MODE);
  int sub = 0;   // the field (diagonal passes) or output (gradient) of this block
  if constexpr (NSPLIT > 1) {
    sub = tile % NSPLIT;
    tile /= NSPLIT;
  }
  const Work3 W = shift(L.w0, item * L.wstride);
  const int ct = M.ct, ny = M.ny, nz = M.nz, nl = M.nlines;
  const int c0 = tile * ct, ncols = min(ct, M.nxh1 - c0);
  const int cnt = nl * ct;
  const int B = blockDim.x, tid = threadIdx.x;
  extern __shared__ float2 lds[];
  float2* twy = lds;
  float2* twz = twy + ny;
  float2* buf = twz + nz;
  float2* b0 = buf;
  float2* b1 = buf + cnt;
  for (int i = tid; i < ny; i += B) twy[i] = M.twy[i];
  for (int i = tid; i < nz; i += B) twz[i] = M.twz[i];
  const size_t specN = size_t(M.ctiles) * ct * nl;
  auto chunk_of = [&](int f) { return W.s + size_t(f) * specN + size_t(tile) * cnt; };
  // y-lines: (z, c) -> z * ny * ct + c, stride ct; z-lines: (y, c) -> y * ct + c, stride ny * ct
  const LineMap my{nz * ct, ct, ny * ct, 1, ct};
  const LineMap mz{ny * ct, ny * ct, 0, 1, ny * ct};
  auto fwd = [&](float2* a, float2* b) {
    float2* r = fft_axis<false, AX>(a, b, my, M.py, twy);
    return fft_axis<false, AX>(r, r == a ? b : a, mz, M.pz, twz);
  };
  auto inv = [&](float2* a, float2* b) {
    float2* r = fft_axis<true, AX>(a, b, mz, M.pz, twz);
    return fft_axis<true, AX>(r, r == a ? b : a, my, M.py, twy);
  };
  auto load = [&](int f, float2* dst) {
    const float2* src = chunk_of(f);
    for (int i = tid; i < cnt; i += B) dst[i] = src[i];
  };
  auto store = [&](int f, const float2* src) {
    float2* dst = chunk_of(f);
    for (int i = tid; i < cnt; i += B) dst[i] = src[i];
  };
  // multiplier at chunk element i for operator `cd` (0 in the padding columns)
  const float rct = rcp(ct), rny = rcp(ny);
  auto mult = [&](int cd, int i) {
    const int l = udiv(i, rct), c = i - l * ct, z = udiv(l, rny), y = l - z * ny;
    return c < ncols ? symbol(M, cd, c0 + c, y, z) : make_float2(0.f, 0.f);
  };

  // one field of a diagonal pass (reads and writes only its own spectrum),
  // one output of the gradient (reads spectrum 3), or a single operator
  load(MODE == P3_GRADP1 ? 3 : sub, b0);
  __syncthreads();
  float2* F = fwd(b0, b1);
  const int cd = plane_code<MODE>(sub, code);
  for (int i = tid; i < cnt; i += B) F[i] = cmul(F[i], mult(cd, i));
  __syncthreads();
  store(sub, inv(F, F == b0 ? b1 : b0));
}

// ---------------------------------------------------------------- sensor data
__global__ void combine3_kernel(const Launch3 L) {
  const Medium3& M = L.m;
  const Work3 W = shift(L.w0, blockIdx.y * L.wstride);
  float* out = L.io[blockIdx.y].out;
  const int total = M.nt * M.ns;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const float* p = W.part + size_t(i) * 4;
    out[i] = (p[0] + p[1]) + (p[2] + p[3]);
  }
}

// ---------------------------------------------------------------- launchers
template <int MODE>
static hipError_t row_t(const Launch3& L, int ntile, int chunk, int n, size_t lds, hipStream_t st) {
  const dim3 g(chunk * kXcds), t(L.m.rthr);
  // (49-point lines take the dense row pass)
  if (L.m.px.n == 64)
    hipLaunchKernelGGL((row3_kernel<MODE, 64>), g, t, lds, st, L, ntile, chunk, n);
  else
    hipLaunchKernelGGL((row3_kernel<MODE, 0>), g, t, lds, st, L, ntile, chunk, n);
  return hipGetLastError();
}

hipError_t launch_row3(int mode, const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  if (dense3(L.m.nx)) return launch_row3_dense(mode, L, ntile, chunk, n, st);
  const size_t lds = row3_lds(L.m.nx, L.m.rt);
  switch (mode) {
    case R3_F1: return row_t<R3_F1>(L, ntile, chunk, n, lds, st);
    case R3_F2: return row_t<R3_F2>(L, ntile, chunk, n, lds, st);
    case R3_F2L: return row_t<R3_F2L>(L, ntile, chunk, n, lds, st);
    case R3_F3: return row_t<R3_F3>(L, ntile, chunk, n, lds, st);
    case R3_A1: return row_t<R3_A1>(L, ntile, chunk, n, lds, st);
    case R3_A1L: return row_t<R3_A1L>(L, ntile, chunk, n, lds, st);
    case R3_A2: return row_t<R3_A2>(L, ntile, chunk, n, lds, st);
    case R3_A3: return row_t<R3_A3>(L, ntile, chunk, n, lds, st);
    case R3_FWD1: return row_t<R3_FWD1>(L, ntile, chunk, n, lds, st);
    case R3_INV1: return row_t<R3_INV1>(L, ntile, chunk, n, lds, st);
    default: return hipErrorInvalidValue;
  }
}

template <int MODE>
static hipError_t plane_t(const Launch3& L, int ntile, int chunk, int code, int n, size_t lds, hipStream_t st) {
  const dim3 g(chunk * kXcds), t(L.m.pthr);
  // an instance with compile-time stages only when both transformed axes have its length
  const int R = L.m.py.n == L.m.pz.n ? staged3(L.m.py.n) : 0;
  if (R == 7)
    hipLaunchKernelGGL((plane3_kernel<MODE, 49>), g, t, lds, st, L, ntile, chunk, code, n);
  else if (R == 8)
    hipLaunchKernelGGL((plane3_kernel<MODE, 64>), g, t, lds, st, L, ntile, chunk, code, n);
  else
    hipLaunchKernelGGL((plane3_kernel<MODE, 0>), g, t, lds, st, L, ntile, chunk, code, n);
  return hipGetLastError();
}

hipError_t launch_plane3(int mode, int code, const Launch3& L, int ntile, int chunk, int n, hipStream_t st) {
  if (dense3_plane(L.m.ny, L.m.nz)) return launch_plane3_dense(mode, code, L, ntile, chunk, n, st);
  const size_t lds = plane3_lds(L.m.ny, L.m.nz, L.m.ct);
  switch (mode) {
    case P3_GRADP1: return plane_t<P3_GRADP1>(L, ntile, chunk, code, n, lds, st);
    case P3_GRADM2: return plane_t<P3_GRADM2>(L, ntile, chunk, code, n, lds, st);
    case P3_FRAC: return plane_t<P3_FRAC>(L, ntile, chunk, code, n, lds, st);
    case P3_GRADP2: return plane_t<P3_GRADP2>(L, ntile, chunk, code, n, lds, st);
    case P3_APPLY: return plane_t<P3_APPLY>(L, ntile, chunk, code, n, lds, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_combine3(const Launch3& L, hipStream_t st) {
  int bx = (L.m.nt * L.m.ns + kBlock - 1) / kBlock;
  if (bx > 1024) bx = 1024;
  if (bx < 1) bx = 1;
  hipLaunchKernelGGL(combine3_kernel, dim3(bx, L.nitems), dim3(kBlock), 0, st, L);
  return hipGetLastError();
}

template <typename K>
static hipError_t allow(K* k, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(bytes));
}

template <int MODE>
static hipError_t allow_row(size_t bytes) {
  const hipError_t e = allow(&row3_kernel<MODE, 0>, bytes);
  return e != hipSuccess ? e : allow(&row3_kernel<MODE, 64>, bytes);
}
template <int MODE>
static hipError_t allow_plane(size_t bytes) {
  hipError_t e = allow(&plane3_kernel<MODE, 0>, bytes);
  if (e == hipSuccess) e = allow(&plane3_kernel<MODE, 49>, bytes);
  if (e == hipSuccess) e = allow(&plane3_kernel<MODE, 64>, bytes);
  return e;
}

hipError_t k3d_allow_lds(size_t bytes) {
  const hipError_t es[] = {allow_row<R3_F1>(bytes),       allow_row<R3_F2>(bytes),        allow_row<R3_F2L>(bytes),
                           allow_row<R3_F3>(bytes),       allow_row<R3_A1>(bytes),        allow_row<R3_A1L>(bytes),
                           allow_row<R3_A2>(bytes),       allow_row<R3_A3>(bytes),        allow_row<R3_FWD1>(bytes),
                           allow_row<R3_INV1>(bytes),     allow_plane<P3_GRADP1>(bytes),  allow_plane<P3_GRADM2>(bytes),
                           allow_plane<P3_FRAC>(bytes),   allow_plane<P3_GRADP2>(bytes),  allow_plane<P3_APPLY>(bytes)};
  for (hipError_t e : es)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace qpat3

// Row and column passes of the k-space acoustic operator for gfx950 (MI355X).
//
// Every spectral operator F^-1 diag(m) F of Section 3.2.2 (staggered
// gradients of eq grr, fractional Laplacians Y_dis and Y_abs) is split into
//   row pass  : inverse row FFTs of the previous spectra, the pointwise update
//               of eqs num-vel / num-rho / num-p (or their transposes), and the
//               forward row FFTs of the next fields, all on rows held in LDS;
//   column pass: forward column FFT, multiplier(s), inverse column FFT, on a
//               tile of spectrum columns held in LDS.
// Two real fields share one complex row FFT (z = a + i b); spectra are stored
// as half spectra [ny][nx/2] with the (real) DC and Nyquist columns packed as
// the real and imaginary parts of column 0.  FFTs are radix-2/3/4/6/8/12 Stockham
// passes between two LDS buffers; inverse transforms use conj(FFT(conj(.))).
// The 1/(nx ny) normalisation is folded into the multiplier tables.
//
// A launch covers any number of problems ("items", possibly of different
// sizes): block b reads (item, tile) from a block map built on the host, which
// places consecutive tiles of one item on the same XCD.
#pragma once

#include <type_traits>

#include "qpat_internal.hpp"

// Row and column lengths with compile-time kernel instances.
#define QPAT_FOR_LENGTHS(X) \
  X(32) X(48) X(64) X(96) X(128) X(192) X(256) X(384) X(512) X(768) X(1024)

namespace qpat {

// ---------------------------------------------------------------- complex
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// Complex product with its two fused multiply-adds written out: left to the
// compiler, which product of each part it fuses depends on the surrounding
// code, so two inlined copies of one FFT stage could round differently.
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(__builtin_fmaf(a.x, b.x, -(a.y * b.y)), __builtin_fmaf(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }  // -i * a

// ---------------------------------------------------------------- butterflies (forward DFT)
template <int R> __device__ __forceinline__ void bfly(float2* v);

template <> __device__ __forceinline__ void bfly<2>(float2* v) {
  const float2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <> __device__ __forceinline__ void bfly<3>(float2* v) {
  const float s = 0.86602540378443864676f;  // sin(pi/3)
  const float2 t1 = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  const float2 t2 = make_float2(__builtin_fmaf(-0.5f, t1.x, v[0].x), __builtin_fmaf(-0.5f, t1.y, v[0].y));
  v[0] = cadd(v[0], t1);
  v[1] = make_float2(__builtin_fmaf(s, d.y, t2.x), __builtin_fmaf(-s, d.x, t2.y));
  v[2] = make_float2(__builtin_fmaf(-s, d.y, t2.x), __builtin_fmaf(s, d.x, t2.y));
}

template <> __device__ __forceinline__ void bfly<4>(float2* v) {
  const float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
  const float2 t2 = cadd(v[1], v[3]), t3 = mul_mi(csub(v[1], v[3]));
  v[0] = cadd(t0, t2);
  v[2] = csub(t0, t2);
  v[1] = cadd(t1, t3);
  v[3] = csub(t1, t3);
}

template <> __device__ __forceinline__ void bfly<8>(float2* v) {
  const float c = 0.70710678118654752440f;
  float2 e[4] = {v[0], v[2], v[4], v[6]};
  float2 o[4] = {v[1], v[3], v[5], v[7]};
  bfly<4>(e);
  bfly<4>(o);
  // W8^1 o1 = c (s1 + i d1) and W8^3 o3 = c (d3 - i s3), each scaling fused
  // into the adds and subtracts that use it (written out, as in cmul)
  const float s1 = o[1].x + o[1].y, d1 = o[1].y - o[1].x;
  const float s3 = o[3].x + o[3].y, d3 = o[3].y - o[3].x;
  const float2 o2 = mul_mi(o[2]);  // W8^2
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = make_float2(__builtin_fmaf(c, s1, e[1].x), __builtin_fmaf(c, d1, e[1].y));
  v[5] = make_float2(__builtin_fmaf(-c, s1, e[1].x), __builtin_fmaf(-c, d1, e[1].y));
  v[2] = cadd(e[2], o2);
  v[6] = csub(e[2], o2);
  v[3] = make_float2(__builtin_fmaf(c, d3, e[3].x), __builtin_fmaf(-c, s3, e[3].y));
  v[7] = make_float2(__builtin_fmaf(-c, d3, e[3].x), __builtin_fmaf(c, s3, e[3].y));
}

// Radices 6 = 2 x 3 and 12 = 4 x 3 as prime-factor transforms (no inner
// twiddles): input n = 3 n1 + R1 n2 (mod R) gives the R1 x 3 transform whose
// entry (k mod R1, k mod 3) is output k.
template <> __device__ __forceinline__ void bfly<6>(float2* v) {
  float2 a[3] = {v[0], v[2], v[4]}, b[3] = {v[3], v[5], v[1]};
  bfly<3>(a);
  bfly<3>(b);
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = (k & 1) ? csub(a[k % 3], b[k % 3]) : cadd(a[k % 3], b[k % 3]);
}

template <> __device__ __forceinline__ void bfly<12>(float2* v) {
  float2 t[4][3] = {{v[0], v[4], v[8]}, {v[3], v[7], v[11]}, {v[6], v[10], v[2]}, {v[9], v[1], v[5]}};
#pragma unroll
  for (int n = 0; n < 4; ++n) bfly<3>(t[n]);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    float2 w[4] = {t[0][q], t[1][q], t[2][q], t[3][q]};
    bfly<4>(w);
#pragma unroll
    for (int k = q; k < 12; k += 3) v[k] = w[k & 3];
  }
}

// 24-bit unsigned product (full-rate multiply); every grid and spectrum
// index of a pass is below 2^24.
__device__ __forceinline__ unsigned mul24(unsigned a, unsigned b) { return __umul24(a, b); }

// Quotient a / d for 0 <= a < 2^22 without an integer divide: a float
// reciprocal estimate and one exact correction step.
__device__ __forceinline__ int fdiv(int a, int d, float rcp) {
  int q = static_cast<int>(static_cast<float>(a) * rcp);
  const int r = a - q * d;
  q += (r >= d) - (r < 0);
  return q;
}

// column index of element ix of spectrum tile column tx
__device__ __forceinline__ int k_of(int tx, int ix, int lct) { return (tx << lct) + ix; }

// One Stockham stage for butterfly j: reads src[j + r nb], twiddles by
// W_{Ns R}^{k r} (k = j mod Ns, Ns a power of two except in a last stage, where
// nb = Ns and k = j), writes dst[(j - k) R + k + r Ns].
// Twiddles are stored per stage as [r - 1][k] (the stage's block starts at
// Ns - R0, R0 the first radix), so the lanes of a wave read consecutive
// entries.
template <int R>
__device__ __forceinline__ void stockham(const float2* src, float2* dst, int j, int nb, int Ns,
                                         int off, const float2* tw) {
  float2 v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = src[px(j + r * nb)];
  const int k = Ns == nb ? j : j & (Ns - 1);
  if (Ns > 1) {
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[off + (r - 1) * Ns + k]);
  }
  bfly<R>(v);
  const int base = (j - k) * R + k;
#pragma unroll
  for (int r = 0; r < R; ++r) dst[px(base + r * Ns)] = v[r];
}

// Forward FFT of `nlines` lines (line stride ls) held in LDS buffer a, of a
// length n without kernels of its own: 8 to 24, radices 2, 3, 4 and 8.  b is
// the ping-pong partner and tw the twiddle table (LDS).  The radix plans keep
// Ns a power of two in every stage but the last.  All threads of the block take
// part; returns the buffer that holds the result.  The caller must have
// synchronised after writing the input; the routine ends synchronised.
// (With the radix 6 and 12 stages of the longer lengths in here, every kernel
// that calls it took 20 to 80 registers more: 3 waves a SIMD instead of 4 to 8,
// and a J^T J v of 60 steps 4.19 ms instead of 3.31 at 8 x 8, 5.24 instead of 4.27
// at 24 x 24.)
__device__ float2* fft_lines(float2* a, float2* b, int nlines, int n, int ls, uint32_t rad, int nst,
                             const float2* tw) {
  int Ns = 1;
  const int R0 = rad & 15;
  for (int s = 0; s < nst; ++s) {
    const int R = (rad >> (4 * s)) & 15;
    const int nb = n / R;
    const float rnb = 1.0f / static_cast<float>(nb);
    const int off = Ns - R0;
    const int total = nlines * nb;
    for (int it = threadIdx.x; it < total; it += blockDim.x) {
      const int line = fdiv(it, nb, rnb);
      const int j = it - line * nb;
      const float2* src = a + line * ls;
      float2* dst = b + line * ls;
      if (R == 8)
        stockham<8>(src, dst, j, nb, Ns, off, tw);
      else if (R == 4)
        stockham<4>(src, dst, j, nb, Ns, off, tw);
      else if (R == 2)
        stockham<2>(src, dst, j, nb, Ns, off, tw);
      else
        stockham<3>(src, dst, j, nb, Ns, off, tw);
    }
    __syncthreads();
    float2* t = a;
    a = b;
    b = t;
    Ns *= R;
  }
  return a;
}

// Compile-time versions of the same radix plans (see plan_radix) for the
// common line lengths: every stage's radix, stride and twiddle step is a
// constant, so index arithmetic folds into shifts and LDS immediate offsets.
__host__ __device__ constexpr int ilog2c(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}
__host__ __device__ constexpr int plan_nst(int n) {
  const bool three = n % 3 == 0;
  const int a = ilog2c(three ? n / 3 : n);
  if (three && a >= 4) return 3;
  return (a % 3 ? 1 : 0) + a / 3 + (three ? 1 : 0);
}
// Power-of-two part 2^a: radix 8 stages, with the remainder as two radix-4
// stages at both ends (a = 3q + 1: 4 8..8 4) or one radix-4 second stage
// (a = 3q + 2: 8 4 8..8), so that a plan of two or more stages starts and
// ends with the same radix where it can (the row passes fuse the boundary
// stage of two FFTs; of the lengths with kernels only 32 = 8 4 cannot).  3 2^a with a >= 4: the factor 3 in the middle stage of
// three (48: 4 3 4, 96: 4 6 4, 192: 8 3 8, 384: 8 6 8, 768: 8 12 8), so those
// plans read the same both ways and fuse like the powers of two (with the
// radix-3 stage last the column passes went through LDS between all phases:
// 384 x 192, 4 vectors, one iterate 58.4 us, now 37.9; 768^2 99.6, now 55.5;
// 64 x 64, whose plan was a run-time one, 54.9, now 33.1); shorter ones (12,
// 24) end with a radix-3 stage.
__host__ __device__ constexpr int plan_radix(int n, int s) {
  const bool three = n % 3 == 0;
  const int a = ilog2c(three ? n / 3 : n);
  if (three && a >= 4) {
    const int e = a >= 6 ? 3 : 2;
    return s == 1 ? 3 << (a - 2 * e) : 1 << e;
  }
  const int rem = a % 3, q = a / 3;
  const int np2 = (rem ? 1 : 0) + q;  // power-of-two stages
  if (s >= np2) return 3;
  if (rem == 0) return 8;
  if (rem == 1) return q == 0 ? 2 : ((s == 0 || s == np2 - 1) ? 4 : 8);
  return q == 0 ? 4 : (s == 1 ? 4 : 8);
}

// Padded offset of a displacement d from a base position b when b + d stays
// in b's run of 8 or d is a multiple of 8: px(b + d) = px(b) + pxd(d).
__host__ __device__ constexpr int pxd(int d) { return d + (d >> 3); }

// Whether a stage's butterfly accesses have that form: reads j + r NB with NB
// a multiple of 8; writes base + r NS with NS a multiple of 8, or base =
// (j - k) R + k whose residue mod 8 (k, or a multiple of R when NS = 1) leaves
// room for r NS mod 8.  A stage without it (lengths 32 and 48) pads each
// position by itself.
__host__ __device__ constexpr bool reads_fold(int NB) { return NB % 8 == 0; }
__host__ __device__ constexpr bool writes_fold(int R, int NS) {
  return NS % 8 == 0 || (R != 3 && 8 % NS == 0 && (NS == 1 ? 8 % R == 0 : (NS * R) % 8 == 0));
}
// k = j mod NS of butterfly j < NB: NS is a power of two except in a last
// stage, where NB = NS
template <int NS, int NB>
__device__ __forceinline__ unsigned stage_k(unsigned j) {
  if constexpr (NS == NB) return j;
  else return j & (NS - 1);
}

// The three parts of a compile-time stage for butterfly j: gather its inputs
// from an LDS line, twiddle and transform in registers, scatter its outputs.
template <int R, int NB>
__device__ __forceinline__ void stage_load(float2* v, const float2* src, unsigned j) {
  if constexpr (reads_fold(NB)) {
    const float2* s = src + px(int(j));
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[pxd(r * NB)];
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[px(int(j) + r * NB)];
  }
}
template <int R, int NS, int OFF, int NB>
__device__ __forceinline__ void stage_regs(float2* v, unsigned j, const float2* tw) {
  if constexpr (NS > 1) {
    const float2* t = tw + OFF + stage_k<NS, NB>(j);
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], t[(r - 1) * NS]);
  }
  bfly<R>(v);
}
template <int R, int NS, int NB>
__device__ __forceinline__ void stage_store(const float2* v, float2* dst, unsigned j) {
  const unsigned k = stage_k<NS, NB>(j);
  const int base = int((j - k) * R + k);
  if constexpr (writes_fold(R, NS)) {
    float2* d = dst + px(base);
#pragma unroll
    for (int r = 0; r < R; ++r) d[pxd(r * NS)] = v[r];
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) dst[px(base + r * NS)] = v[r];
  }
}

template <int R, int NS, int NB, int OFF>
__device__ __forceinline__ void stockham_c(const float2* src, float2* dst, unsigned j, const float2* tw) {
  float2 v[R];
  stage_load<R, NB>(v, src, j);
  stage_regs<R, NS, OFF, NB>(v, j, tw);
  stage_store<R, NS, NB>(v, dst, j);
}

// LS: line stride (a compile-time constant, so line offsets fold too).
template <int N, int LS, int S, int NS>
__device__ __forceinline__ float2* fft_c(float2* a, float2* b, int nlines, const float2* tw) {
  if constexpr (S == plan_nst(N)) {
    return a;
  } else {
    constexpr int R = plan_radix(N, S), NB = N / R, OFF = NS - plan_radix(N, 0);
    const unsigned total = unsigned(nlines) * NB;
    for (unsigned it = threadIdx.x; it < total; it += blockDim.x) {
      const unsigned line = it / NB, j = it % NB;
      stockham_c<R, NS, NB, OFF>(a + line * LS, b + line * LS, j, tw);
    }
    __syncthreads();
    return fft_c<N, LS, S + 1, NS * R>(b, a, nlines, tw);
  }
}

// In-place version: every thread gathers and transforms all its butterflies
// of a stage, the block synchronises, then every thread scatters its outputs
// into the same buffer.  A thread holds at most kMaxPer values per stage
// (the host bounds a tile to kMaxPer elements per thread).
template <int N, int LS, int S, int NS>
__device__ __forceinline__ float2* fft_c_ip(float2* a, int nlines, const float2* tw) {
  if constexpr (S == plan_nst(N)) {
    return a;
  } else {
    constexpr int R = plan_radix(N, S), NB = N / R, OFF = NS - plan_radix(N, 0);
    constexpr int MB = (kMaxPer + R - 1) / R;
    const unsigned total = unsigned(nlines) * NB;
    float2 v[MB][R];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const unsigned it = threadIdx.x + i * blockDim.x;
      if (it < total) {
        const unsigned line = it / NB, j = it % NB;
        stage_load<R, NB>(v[i], a + line * LS, j);
        stage_regs<R, NS, OFF, NB>(v[i], j, tw);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const unsigned it = threadIdx.x + i * blockDim.x;
      if (it < total) {
        const unsigned line = it / NB, j = it % NB;
        stage_store<R, NS, NB>(v[i], a + line * LS, j);
      }
    }
    __syncthreads();
    return fft_c_ip<N, LS, S + 1, NS * R>(a, nlines, tw);
  }
}

// Radix of stage s of the compile-time plan of length N, or of that plan in
// reverse order (REV).  Every compile-time plan reversed still has a
// power-of-two Ns in every stage but the last; its per-stage twiddles form
// their own table.
template <int N, bool REV>
__host__ __device__ constexpr int radix_of(int s) {
  return REV ? plan_radix(N, plan_nst(N) - 1 - s) : plan_radix(N, s);
}

// Stages S .. S1-1 of the plan (direction REV) on `nlines` LDS lines of
// stride LS, ping-ponging from a; NS = product of the radices before S.
// Returns the buffer holding the result; ends synchronised.
template <int N, bool REV, int LS, int S, int S1, int NS>
__device__ __forceinline__ float2* fft_stages(float2* a, float2* b, int nlines, const float2* tw) {
  if constexpr (S == S1) {
    return a;
  } else {
    constexpr int R = radix_of<N, REV>(S), NB = N / R, OFF = NS - radix_of<N, REV>(0);
    const unsigned total = unsigned(nlines) * NB;
    for (unsigned it = threadIdx.x; it < total; it += blockDim.x) {
      const unsigned line = it / NB, j = it % NB;
      stockham_c<R, NS, NB, OFF>(a + line * LS, b + line * LS, j, tw);
    }
    __syncthreads();
    return fft_stages<N, REV, LS, S + 1, S1, NS * R>(b, a, nlines, tw);
  }
}

// Stages S .. S1-1 of the plan of length N (REV: the plan in reverse order)
// in place (see fft_c_ip).
template <int N, int LS, int S, int S1, int NS, bool REV = false>
__device__ __forceinline__ float2* fft_range_ip(float2* a, int nlines, const float2* tw) {
  if constexpr (S == S1) {
    return a;
  } else {
    constexpr int R = radix_of<N, REV>(S), NB = N / R, OFF = NS - radix_of<N, REV>(0);
    constexpr int MB = (kMaxPer + R - 1) / R;
    const unsigned total = unsigned(nlines) * NB;
    float2 v[MB][R];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const unsigned it = threadIdx.x + i * blockDim.x;
      if (it < total) {
        const unsigned line = it / NB, j = it % NB;
        stage_load<R, NB>(v[i], a + line * LS, j);
        stage_regs<R, NS, OFF, NB>(v[i], j, tw);
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const unsigned it = threadIdx.x + i * blockDim.x;
      if (it < total) {
        const unsigned line = it / NB, j = it % NB;
        stage_store<R, NS, NB>(v[i], a + line * LS, j);
      }
    }
    __syncthreads();
    return fft_range_ip<N, LS, S + 1, S1, NS * R, REV>(a, nlines, tw);
  }
}

// Row lines whose plan starts and ends with the same radix (512 = 8 8 8):
// the two FFTs of a row pass around a pointwise update share their boundary
// stage in registers.  The last stage of the first FFT leaves butterfly jj of
// a line with the values at jj + r N/R, exactly the inputs of butterfly jj in
// the first stage of the second FFT, so one thread per (line, jj) runs that
// last stage, the update `pw(line, jj, v)` on its R values, and that first
// stage, skipping an LDS round trip and a barrier on each side of the
// update.  The arithmetic is the unfused sequence's.  Ends synchronised with
// the second FFT's result in the returned buffer.
template <int N>
__host__ __device__ constexpr bool row_fusable() {
  return N >= 32 && plan_radix(N, 0) == plan_radix(N, plan_nst(N) - 1) && plan_nst(N) >= 2;
}
template <int N>
__host__ __device__ constexpr int fused_slots() { return (kMaxPer + plan_radix(N, 0) - 1) / plan_radix(N, 0); }
// pw(i, line, jj, v): the update of butterfly slot i (0 <= i < fused_slots)
// of this thread, (line, jj), on its R values v.  A thread has at most
// fused_slots butterflies (the host bounds a tile to kMaxPer elements per
// thread), slot i being butterfly threadIdx.x + i blockDim.x.
template <int N, bool IP, class PW>
__device__ __forceinline__ float2* fft_fused(float2* a, float2* b, int nlines, const float2* tw, PW pw) {
  constexpr int LS = lstride(N), NST = plan_nst(N), R = plan_radix(N, 0), NB = N / R, MB = fused_slots<N>();
  constexpr int OFFL = NB - R;  // twiddles of the last stage (Ns = N / R)
  float2* r;
  if constexpr (IP) r = fft_range_ip<N, LS, 0, NST - 1, 1>(a, nlines, tw);
  else r = fft_stages<N, false, LS, 0, NST - 1, 1>(a, b, nlines, tw);
  float2* o = IP ? r : (r == a ? b : a);
  const unsigned total = unsigned(nlines) * NB;
  float2 v[MB][R];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const unsigned line = it / NB, jj = it % NB;
      stage_load<R, NB>(v[i], r + line * LS, jj);
      stage_regs<R, NB, OFFL, NB>(v[i], jj, tw);
    }
  }
  if constexpr (IP) __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const unsigned line = it / NB, jj = it % NB;
      // The values pass an LDS store and load in the unfused sequence; the
      // empty asm statements keep them opaque here too, so no multiply of
      // one side is contracted with an add of the other (same rounding).
#pragma unroll
      for (int q = 0; q < R; ++q) asm volatile("" : "+v"(v[i][q].x), "+v"(v[i][q].y));
      pw(i, int(line), int(jj), v[i]);
#pragma unroll
      for (int q = 0; q < R; ++q) asm volatile("" : "+v"(v[i][q].x), "+v"(v[i][q].y));
      stage_regs<R, 1, 0, NB>(v[i], jj, tw);
      stage_store<R, 1, NB>(v[i], o + line * LS, jj);
    }
  }
  __syncthreads();
  if constexpr (IP) return fft_range_ip<N, LS, 1, NST, R>(o, nlines, tw);
  else return fft_stages<N, false, LS, 1, NST, R>(o, r, nlines, tw);
}

// The same fusion for updates that read two lines and write two lines per
// position (rows 2l and 2l+1 packed as one complex line on one side of the
// update, each row its own line on the other): work item (l, jj) runs the
// last stage on lines inl(l, 0) and inl(l, 1), `pw(i, l, jj, va, vb)` on their
// values, and the first stage on lines outl(l, 0) and outl(l, 1).
template <int N>
__host__ __device__ constexpr int fused2_slots() { return (kMaxPer / 2 + plan_radix(N, 0) - 1) / plan_radix(N, 0); }
template <int N, bool IP, class IL, class OL, class PW>
__device__ __forceinline__ float2* fft_fused2(float2* a, float2* b, int nlines, const float2* tw, IL inl, OL outl,
                                              PW pw) {
  constexpr int LS = lstride(N), NST = plan_nst(N), R = plan_radix(N, 0), NB = N / R, MB = fused2_slots<N>();
  constexpr int OFFL = NB - R;
  float2* r;
  if constexpr (IP) r = fft_range_ip<N, LS, 0, NST - 1, 1>(a, nlines, tw);
  else r = fft_stages<N, false, LS, 0, NST - 1, 1>(a, b, nlines, tw);
  float2* o = IP ? r : (r == a ? b : a);
  const unsigned total = unsigned(nlines / 2) * NB;
  float2 va[MB][R], vb[MB][R];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const int l = int(it / NB);
      const unsigned jj = it % NB;
      stage_load<R, NB>(va[i], r + inl(l, 0) * LS, jj);
      stage_regs<R, NB, OFFL, NB>(va[i], jj, tw);
      stage_load<R, NB>(vb[i], r + inl(l, 1) * LS, jj);
      stage_regs<R, NB, OFFL, NB>(vb[i], jj, tw);
    }
  }
  if constexpr (IP) __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const int l = int(it / NB);
      const unsigned jj = it % NB;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        asm volatile("" : "+v"(va[i][q].x), "+v"(va[i][q].y));
        asm volatile("" : "+v"(vb[i][q].x), "+v"(vb[i][q].y));
      }
      pw(i, l, int(jj), va[i], vb[i]);
#pragma unroll
      for (int q = 0; q < R; ++q) {
        asm volatile("" : "+v"(va[i][q].x), "+v"(va[i][q].y));
        asm volatile("" : "+v"(vb[i][q].x), "+v"(vb[i][q].y));
      }
      stage_regs<R, 1, 0, NB>(va[i], jj, tw);
      stage_store<R, 1, NB>(va[i], o + outl(l, 0) * LS, jj);
      stage_regs<R, 1, 0, NB>(vb[i], jj, tw);
      stage_store<R, 1, NB>(vb[i], o + outl(l, 1) * LS, jj);
    }
  }
  __syncthreads();
  if constexpr (IP) return fft_range_ip<N, LS, 1, NST, R>(o, nlines, tw);
  else return fft_stages<N, false, LS, 1, NST, R>(o, r, nlines, tw);
}

// First thread index of this thread's wavefront as a scalar, so that tests on
// it compile to scalar branches: a wave whose lanes have no work item skips a
// fused section (and its operand loads) as a whole, while the lanes of a wave
// with work stay together for the lane exchanges.
__device__ __forceinline__ unsigned wave_base() { return __builtin_amdgcn_readfirstlane(threadIdx.x) & ~63u; }

// The value x of the adjacent lane (lane ^ 1): a DPP quad permutation
// [1, 0, 3, 2], a VALU move (no LDS round trip).  Both lanes of a pair must
// be active.
__device__ __forceinline__ float lane_pair_swap(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));
}

// The same fusion for updates that pair rows 2l and 2l+1 as one complex line
// on one side of the update and keep each row its own line on the other.
// Work item (l, sd, jj) runs the last stage on line inl(l, sd), the update
// `pw(i, l, sd, jj, v, active)` of row 2l + sd, and the first stage on line
// outl(l, sd).  Consecutive work items hold the two rows of a pair, so the
// two lanes of a pair trade the half of a packed line each needs with one
// lane shuffle per value inside pw; pw therefore runs on every lane (lanes
// without a work item hold zeros and `active` false).
template <int N, bool IP, class IL, class OL, class PW>
__device__ __forceinline__ float2* fft_fused_pairs(float2* a, float2* b, int nlines, const float2* tw, IL inl,
                                                   OL outl, PW pw) {
  constexpr int LS = lstride(N), NST = plan_nst(N), R = plan_radix(N, 0), NB = N / R, MB = fused_slots<N>();
  constexpr int OFFL = NB - R;
  float2* r;
  if constexpr (IP) r = fft_range_ip<N, LS, 0, NST - 1, 1>(a, nlines, tw);
  else r = fft_stages<N, false, LS, 0, NST - 1, 1>(a, b, nlines, tw);
  float2* o = IP ? r : (r == a ? b : a);
  const unsigned total = unsigned(nlines) * NB;  // even: pairs are both in range or both out
  float2 v[MB][R];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    const unsigned p = it >> 1, sd = it & 1u, l = p / NB, jj = p % NB;
    if (it < total) {
      stage_load<R, NB>(v[i], r + inl(int(l), int(sd)) * LS, jj);
      stage_regs<R, NB, OFFL, NB>(v[i], jj, tw);
    } else {
#pragma unroll
      for (int q = 0; q < R; ++q) v[i][q] = make_float2(0.f, 0.f);
    }
  }
  if constexpr (IP) __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (wave_base() + i * blockDim.x < total) {  // wave-uniform: the exchanges see whole waves
      const unsigned it = threadIdx.x + i * blockDim.x;
      const unsigned p = it >> 1, sd = it & 1u, l = p / NB, jj = p % NB;
      const bool active = it < total;
#pragma unroll
      for (int q = 0; q < R; ++q) asm volatile("" : "+v"(v[i][q].x), "+v"(v[i][q].y));
      pw(i, int(l), int(sd), int(jj), v[i], active);
#pragma unroll
      for (int q = 0; q < R; ++q) asm volatile("" : "+v"(v[i][q].x), "+v"(v[i][q].y));
      if (active) {
        stage_regs<R, 1, 0, NB>(v[i], jj, tw);
        stage_store<R, 1, NB>(v[i], o + outl(int(l), int(sd)) * LS, jj);
      }
    }
  }
  __syncthreads();
  if constexpr (IP) return fft_range_ip<N, LS, 1, NST, R>(o, nlines, tw);
  else return fft_stages<N, false, LS, 1, NST, R>(o, r, nlines, tw);
}

// FFT of `nlines` row lines, same contract as fft_lines.  NF != 0: an instance
// for lines of length NF (n == NF), which carries that compile-time plan only; IP:
// its stages run in place in a (b unused).  NF == 0: an instance for several
// lengths, with MIX all of them (a table launch), else 8 to 24 only.  Each length
// keeps its compile-time plan in such a launch: one launch set over grids of
// 96^2, 128^2 and 192^2, J^T J v of 40 to 50 steps, 5.64 ms with run-time plans
// for the rows, now 4.59; 768^2, 512^2 and 96^2 8.59, now 7.15.
template <int NF, bool IP, bool MIX>
__device__ __forceinline__ float2* fft_any(float2* a, float2* b, int nlines, int n, int ls, uint32_t rad,
                                           int nst, const float2* tw) {
  if constexpr (NF != 0) {
    if constexpr (IP) return fft_c_ip<NF, lstride(NF), 0, 1>(a, nlines, tw);
    else return fft_c<NF, lstride(NF), 0, 1>(a, b, nlines, tw);
  } else {
    if constexpr (MIX) {
#define QPAT_FFT_CASE(N) \
  case N: return fft_c<N, lstride(N), 0, 1>(a, b, nlines, tw);
      switch (n) {
        QPAT_FOR_LENGTHS(QPAT_FFT_CASE)
        default: break;
      }
#undef QPAT_FFT_CASE
    }
    return fft_lines(a, b, nlines, n, ls, rad, nst, tw);
  }
}

// ---------------------------------------------------------------- packing
// Conjugated inverse-FFT input of the pair (A, B) of packed half-spectrum
// rows: Z = A + iB with Hermitian completion; writes Z[k] and Z[n-k].
__device__ __forceinline__ void build_inv(float2* L, float2 A, float2 B, int k, int nx, int nxh) {
  if (k == 0) {
    L[0] = make_float2(A.x, -B.x);
    L[px(nxh)] = make_float2(A.y, -B.y);
  } else {
    L[px(k)] = make_float2(A.x - B.y, -(A.y + B.x));
    L[px(nx - k)] = make_float2(A.x + B.y, -(B.x - A.y));
  }
}

// Split the FFT Z of a + i b into the packed half spectra A (of a), B (of b).
__device__ __forceinline__ void unpack(const float2* L, int k, int nx, int nxh, float2& A, float2& B) {
  if (k == 0) {
    const float2 z0 = L[0], zn = L[px(nxh)];
    A = make_float2(z0.x, zn.x);
    B = make_float2(z0.y, zn.y);
  } else {
    const float2 zk = L[px(k)], zm = L[px(nx - k)];
    A = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
    B = make_float2(0.5f * (zk.y + zm.y), 0.5f * (zm.x - zk.x));
  }
}

__device__ __forceinline__ float2* other(float2* r, float2* a, float2* b) { return r == a ? b : a; }

// Half spectra are stored in tiles of rt rows x ct columns (the row- and
// column-pass tile sizes): element (ky, kx) sits at
//   ((ky / rt) (nxh / ct) + kx / ct) rt ct + (ky mod rt) ct + kx mod ct,
// so the rt rows of one row tile form one contiguous run and a column tile is
// a sequence of runs of rt*ct elements.  All loops below walk memory order.

// The load phase of a block issues every global load before its first LDS
// write: fetch_* gathers into registers, put_* scatters into LDS, so the phase
// costs one memory round trip rather than one per loop iteration.  Bounds
// (enforced on the host): a row tile holds rt*nx <= kMaxPer*B reals, hence at
// most kPairIt complex pairs per thread; a line length is at most kMaxPer*B.
constexpr int kPairIt = kMaxPer / 2;
constexpr int kRowPairIt = kMaxPer / 4;

struct PairRegs {
  float2 a[kPairIt], b[kPairIt];
};
struct RowPairRegs {
  float2 a[kRowPairIt], b[kRowPairIt];
};
template <int K>
struct TwRegsK {
  float2 t[K];
};
using TwRegs = TwRegsK<kMaxPer>;

// Row length of a row-pass instance: the compile-time length NF when the
// instance carries one (it is launched only for rows of that length), else
// the plan's.  nxh = nx / 2 (half-spectrum columns).
template <int NF>
__device__ __forceinline__ int row_len(const Medium& M) { return NF > 0 ? NF : M.nx; }
template <int NF>
__device__ __forceinline__ int row_half(const Medium& M) { return NF > 0 ? NF / 2 : M.nxh; }

// Spectra are stored in tiles of srt rows x ct columns (row tiles of srt
// rows one after another, the column tiles of one row tile one after another,
// each tile row-major).  A row block's rt rows (srt a multiple of rt) are rows
// r0 .. r0 + rt - 1 of one storage row tile.  The block enumerates its
// elements p in the order of an rt x ct tiling (column tile major); element p
// sits at spec_row_base + spec_row_off(p).  With srt = rt that is base + p.
template <int NF>
__device__ __forceinline__ unsigned spec_row_base(const Medium& M, int tile) {
  const unsigned y0 = unsigned(tile) << M.lrt;
  return mul24(y0 >> M.lsrt, unsigned(M.srt * row_half<NF>(M))) + ((y0 & unsigned(M.srt - 1)) << M.lct);
}
__device__ __forceinline__ unsigned spec_row_off(const Medium& M, unsigned p) {
  const int s = M.lrt + M.lct;
  return ((p >> s) << (M.lsrt + M.lct)) + (p & ((1u << s) - 1u));
}

// line j <- rows j of the row tile (s0, s1)
template <int NF>
__device__ __forceinline__ void fetch_pair(PairRegs& R, const Medium& M, const float2* __restrict__ s0,
                                           const float2* __restrict__ s1, int tile) {
  const int tot = M.rt * row_half<NF>(M);
  const unsigned base = spec_row_base<NF>(M, tile);
#pragma unroll
  for (int k = 0; k < kPairIt; ++k) {
    const int p = threadIdx.x + k * blockDim.x;
    if (p < tot) {
      const unsigned o = base + spec_row_off(M, p);
      R.a[k] = s0[o];
      R.b[k] = s1[o];
    }
  }
}
template <int NF>
__device__ __forceinline__ void put_pair(const PairRegs& R, float2* buf, const Medium& M) {
  const int nx = row_len<NF>(M), nxh = row_half<NF>(M), LS = lstride(nx), rc = M.rt * M.ct, tot = M.rt * nxh;
#pragma unroll
  for (int k = 0; k < kPairIt; ++k) {
    const int p = threadIdx.x + k * blockDim.x;
    if (p < tot) {
      const int w = p & (rc - 1);
      const int j = w >> M.lct, kx = ((p >> (M.lrt + M.lct)) << M.lct) + (w & (M.ct - 1));
      build_inv(buf + j * LS, R.a[k], R.b[k], kx, nx, nxh);
    }
  }
}

// line l <- rows (2l, 2l+1) of the row tile of s0
template <int NF>
__device__ __forceinline__ void fetch_rowpair(RowPairRegs& R, const Medium& M, const float2* __restrict__ s0,
                                              int tile) {
  const int nxh = row_half<NF>(M), hc = (M.rt >> 1) * M.ct, tot = (M.rt >> 1) * nxh;
  const unsigned base = spec_row_base<NF>(M, tile);
#pragma unroll
  for (int k = 0; k < kRowPairIt; ++k) {
    const int q = threadIdx.x + k * blockDim.x;
    if (q < tot) {
      const int tx = q >> (M.lrt - 1 + M.lct), w2 = q & (hc - 1);
      const int l = w2 >> M.lct, ix = w2 & (M.ct - 1);
      const unsigned off = base + (unsigned(tx) << (M.lsrt + M.lct)) + (2 * l) * M.ct + ix;
      R.a[k] = s0[off];
      R.b[k] = s0[off + M.ct];
    }
  }
}
template <int NF>
__device__ __forceinline__ void put_rowpair(const RowPairRegs& R, float2* buf, const Medium& M) {
  const int nx = row_len<NF>(M), nxh = row_half<NF>(M), LS = lstride(nx), hc = (M.rt >> 1) * M.ct,
            tot = (M.rt >> 1) * nxh;
#pragma unroll
  for (int k = 0; k < kRowPairIt; ++k) {
    const int q = threadIdx.x + k * blockDim.x;
    if (q < tot) {
      const int tx = q >> (M.lrt - 1 + M.lct), w2 = q & (hc - 1);
      const int l = w2 >> M.lct, ix = w2 & (M.ct - 1);
      build_inv(buf + l * LS, R.a[k], R.b[k], k_of(tx, ix, M.lct), nx, nxh);
    }
  }
}

template <int K>
__device__ __forceinline__ void fetch_tw(TwRegsK<K>& R, const float2* __restrict__ tw, int n) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = threadIdx.x + k * blockDim.x;
    if (i < n) R.t[k] = tw[i];
  }
}
template <int K>
__device__ __forceinline__ void put_tw(const TwRegsK<K>& R, float2* dst, int n) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = threadIdx.x + k * blockDim.x;
    if (i < n) dst[i] = R.t[k];
  }
}

// Spectrum store; NT (launches of about one block per CU): non-temporal, so
// the kernel's end has fewer dirty L2 lines to write back before the next
// pass, on other XCDs, reads them.  With many blocks per CU the plain store is
// the faster one (measured: one 512^2 vector 154.0 -> 152.0 ms non-temporal,
// 1024^2 x 8 pass sum 554 -> 661 us).
typedef float f2v_t __attribute__((ext_vector_type(2)));
template <bool NT>
__device__ __forceinline__ void st_spec(float2* p, float2 v) {
  if constexpr (NT) {
    f2v_t x;
    x.x = v.x;
    x.y = v.y;
    __builtin_nontemporal_store(x, reinterpret_cast<f2v_t*>(p));
  } else {
    *p = v;
  }
}

// (the store loops are unrolled so that the LDS reads of several iterations
// are in flight together: the global stores in between cannot alias LDS)
template <int NF, bool NT = false>
__device__ __forceinline__ void store_pair_spectra(const float2* buf, const Medium& M, float2* __restrict__ s0,
                                                   float2* __restrict__ s1, int tile) {
  const int nx = row_len<NF>(M), nxh = row_half<NF>(M), LS = lstride(nx), rc = M.rt * M.ct;
  const unsigned base = spec_row_base<NF>(M, tile);
#pragma unroll 4
  for (int p = threadIdx.x; p < M.rt * nxh; p += blockDim.x) {
    const int w = p & (rc - 1);
    const int j = w >> M.lct, k = ((p >> (M.lrt + M.lct)) << M.lct) + (w & (M.ct - 1));
    float2 A, B;
    unpack(buf + j * LS, k, nx, nxh, A, B);
    const unsigned o = base + spec_row_off(M, p);
    st_spec<NT>(s0 + o, A);
    st_spec<NT>(s1 + o, B);
  }
}

template <int NF, bool NT = false>
__device__ __forceinline__ void store_rowpair_spectra(const float2* buf, const Medium& M, float2* __restrict__ s0,
                                                      int tile) {
  const int nx = row_len<NF>(M), nxh = row_half<NF>(M), LS = lstride(nx), hc = (M.rt >> 1) * M.ct;
  const unsigned base = spec_row_base<NF>(M, tile);
#pragma unroll 4
  for (int q = threadIdx.x; q < (M.rt >> 1) * nxh; q += blockDim.x) {
    const int tx = q >> (M.lrt - 1 + M.lct), w2 = q & (hc - 1);
    const int l = w2 >> M.lct, ix = w2 & (M.ct - 1);
    const unsigned off = base + (unsigned(tx) << (M.lsrt + M.lct)) + (2 * l) * M.ct + ix;
    float2 A, B;
    unpack(buf + l * LS, k_of(tx, ix, M.lct), nx, nxh, A, B);
    st_spec<NT>(s0 + off, A);
    st_spec<NT>(s0 + off + M.ct, B);
  }
}

// Row-pair LDS layout: row y0+j lives in component (j & 1) of line j >> 1.
__device__ __forceinline__ float& pcomp(float2* buf, int j, int x, int nx) {
  float2* e = buf + (j >> 1) * lstride(nx) + px(x);
  return (j & 1) ? e->y : e->x;
}

// Value of row y0+j after an inverse FFT of row-pair lines (conj trick undone).
__device__ __forceinline__ float rowpair_val(const float2* buf, int j, int x, int nx) {
  const float2 e = buf[(j >> 1) * lstride(nx) + px(x)];
  return (j & 1) ? -e.y : e.x;
}

// Sensor taps of the tile's rows (and, in the adjoint, the residual samples
// they need, in tap order) are staged in LDS; entries beyond the LDS capacity
// are read from global memory.  The tap range is read with the first loads of
// a block; the taps themselves are fetched after the first barrier (thread i
// holds tap e0 + i, blockDim.x >= kTapCap) and written to LDS only where the
// sensors are used, so their latency hides behind the first FFT.

struct TapStage {
  Tap* tl;     // [kTapCap]
  float* rv;   // [kTapCap]
  int e0, e1;  // CSR range of the tile
  int w[8];    // this thread's tap, word by word
  float r;     // and its residual sample
  int n0, n1;  // adjoint: CSR range of the tile's scatter nodes
  int4 nd;     // this thread's node (y, x, c0, c1)
  int con[kConRegs];  // and its first contributions
};

__device__ __forceinline__ void taps_range(TapStage& T, const Medium& M, void* base, int y0, int rt,
                                           bool nodes = false) {
  T.tl = reinterpret_cast<Tap*>(base);
  T.rv = reinterpret_cast<float*>(T.tl + kTapCap);
  T.e0 = M.tap_off[y0];
  T.e1 = M.tap_off[y0 + rt];
  if (nodes) {
    T.n0 = M.node_off[y0];
    T.n1 = M.node_off[y0 + rt];
  }
}

// Adjoint: this thread's scatter node and its first contributions, one record
// (issued early, consumed after the inverse FFT).
__device__ __forceinline__ void nodes_fetch(TapStage& T, const Medium& M) {
  const int i = threadIdx.x;
  if (i < T.n1 - T.n0) {
    const int4* rec = M.nodes + 2 * (T.n0 + i);
    T.nd = rec[0];
    const int4 c = rec[1];
    T.con[0] = c.x;
    T.con[1] = c.y;
    T.con[2] = c.z;
    T.con[3] = c.w;
  }
}

// rtap: residual samples in tap order for sample m ([nt][ntap]), or null
__device__ __forceinline__ void taps_fetch(TapStage& T, const Medium& M, const float* __restrict__ rtap, int m) {
  const int i = threadIdx.x;
  if (i < min(T.e1 - T.e0, kTapCap)) {
    const int4* src = reinterpret_cast<const int4*>(M.taps + T.e0 + i);
    const int4 lo = src[0], hi = src[1];
    T.w[0] = lo.x, T.w[1] = lo.y, T.w[2] = lo.z, T.w[3] = lo.w;
    T.w[4] = hi.x, T.w[5] = hi.y, T.w[6] = hi.z, T.w[7] = hi.w;
    if (rtap) T.r = rtap[unsigned(m) * unsigned(2 * M.ns) + T.e0 + i];
  }
}

__device__ __forceinline__ void taps_put(const TapStage& T, bool with_res) {
  const int i = threadIdx.x;
  if (i < min(T.e1 - T.e0, kTapCap)) {
    int4* dst = reinterpret_cast<int4*>(T.tl + i);
    dst[0] = make_int4(T.w[0], T.w[1], T.w[2], T.w[3]);
    dst[1] = make_int4(T.w[4], T.w[5], T.w[6], T.w[7]);
    if (with_res) T.rv[i] = T.r;
  }
}

__device__ __forceinline__ Tap tap_at(const Medium& M, const TapStage& T, int e) {
  const Tap* src = (e - T.e0 < kTapCap) ? T.tl + (e - T.e0) : M.taps + e;
  Tap t;
  t.s = src->s;
  t.slot = src->slot;
  t.y = src->y;
  t.ixl = src->ixl;
  t.ixr = src->ixr;
  t.wl = src->wl;
  t.wr = src->wr;
  t.pad = 0;
  return t;
}

// Forward sensor partials for rows y0 .. y0+rt-1 (bilinear taps, eq num-m).
__device__ __forceinline__ void sensor_partials(const Medium& M, const TapStage& T, float2* buf, int y0,
                                                float* __restrict__ part, int m) {
  for (int e = T.e0 + threadIdx.x; e < T.e1; e += blockDim.x) {
    const Tap t = tap_at(M, T, e);
    const int j = t.y - y0;
    const float v = t.wl * pcomp(buf, j, t.ixl, M.nx) + t.wr * pcomp(buf, j, t.ixr, M.nx);
    part[(unsigned(m) * unsigned(M.ns) + t.s) * 2 + t.slot] = v;
  }
}

// Adjoint sensor scatter M^T r for rows y0 .. y0+rt-1 as a gather: one thread
// per grid node a tap touches adds that node's contributions in increasing
// tap index, the order of a serial scatter over the row's taps, so the result
// does not depend on the thread count.
__device__ __forceinline__ float scatter_term(const Medium& M, const TapStage& T, const float* __restrict__ rtap,
                                              int m, float acc, int code) {
  const int e = code >> 1;
  const bool staged = e - T.e0 < kTapCap;
  const Tap* src = staged ? T.tl + (e - T.e0) : M.taps + e;
  const float w = (code & 1) ? src->wr : src->wl;
  const float rv = staged ? T.rv[e - T.e0] : rtap[unsigned(m) * unsigned(2 * M.ns) + e];
  return acc + w * rv;
}

__device__ __forceinline__ void sensor_scatter(const Medium& M, const TapStage& T, float2* buf, int y0,
                                               const float* __restrict__ rtap, int m) {
  const int nn = T.n1 - T.n0;
  for (int i = threadIdx.x; i < nn; i += blockDim.x) {
    const bool pre = i == int(threadIdx.x);  // the first round's node was fetched early
    const int4 nd = pre ? T.nd : M.nodes[2 * (T.n0 + i)];
    float& v = pcomp(buf, nd.x - y0, nd.y, M.nx);
    float acc = v;
#pragma unroll
    for (int k = 0; k < kConRegs; ++k)
      if (nd.z + k < nd.w) acc = scatter_term(M, T, rtap, m, acc, pre ? T.con[k] : M.scon[nd.z + k]);
    for (int c = nd.z + kConRegs; c < nd.w; ++c) acc = scatter_term(M, T, rtap, m, acc, M.scon[c]);
    v = acc;
  }
}

// ---------------------------------------------------------------- block -> (item, tile)
// Uniform launches (all items are vectors of one plan) carry the medium in
// the kernel arguments and find their work buffers by a fixed stride, so the
// first global loads of a block are its data; other launches read the item
// descriptors from device memory, and (item, tile) from a block map unless all
// items have the same number of tiles (ntile > 0).
// Either way consecutive tiles of one item are placed on one XCD.
template <bool U>
__device__ __forceinline__ bool locate(const Launch& L, int ntile, int chunk, int& item, int& tile) {
  if (U || ntile > 0) {
    const int b = blockIdx.x;
    const int i = (b & (kXcds - 1)) * chunk + (b / kXcds);
    if (i >= L.nitems * ntile) return false;
    item = i / ntile;
    tile = i - item * ntile;
    return true;
  }
  const __attribute__((address_space(4))) int2* bm = (const __attribute__((address_space(4))) int2*)L.map + blockIdx.x;
  item = bm->x;
  tile = bm->y;
  return item >= 0;
}

// The descriptors of a table launch are constant while a kernel runs: read
// through the constant address space they come by scalar loads whatever the
// kernel does in between, and their pointers, marked as global ones, give
// global loads (the plain structure in memory gave flat loads, which wait for
// the LDS counter too).  Fields that a pass does not use are not loaded.  Seven
// problems of 256^2 to 512^2, a launch sequence per size: 29.7 -> 27.8 ms (column
// passes of three 256^2 6.7 -> 6.2 us, row passes 8.8 -> 8.4).
typedef const __attribute__((address_space(4))) Item ConstItem;
typedef const __attribute__((address_space(4))) IO ConstIO;
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)p;
}
template <bool U>
using MediumOf = std::conditional_t<U, const Medium&, Medium>;
template <bool U>
using IOOf = std::conditional_t<U, const IO&, IO>;
template <bool U>
__device__ __forceinline__ MediumOf<U> medium_of(const Launch& L, int item) {
  if constexpr (U) {
    return L.m;
  } else {
    ConstItem* t = (ConstItem*)L.items + item;
    Medium m;
#define QPAT_V(f) m.f = t->m.f
#define QPAT_P(f) m.f = as_global(t->m.f)
    QPAT_V(nx), QPAT_V(ny), QPAT_V(nxh), QPAT_V(nt), QPAT_V(ns), QPAT_V(lossy), QPAT_V(dt), QPAT_V(ypow);
    QPAT_V(rt), QPAT_V(ct), QPAT_V(lrt), QPAT_V(lct), QPAT_V(srt), QPAT_V(lsrt), QPAT_V(rthr), QPAT_V(cthr);
    QPAT_V(radx), QPAT_V(rady), QPAT_V(nstx), QPAT_V(nsty);
    QPAT_P(c2), QPAT_P(c2eta), QPAT_P(c2tau), QPAT_P(rho0), QPAT_P(bx), QPAT_P(by);
    QPAT_P(avx), QPAT_P(arx), QPAT_P(avy), QPAT_P(ary);
    QPAT_P(dxp), QPAT_P(dxm), QPAT_P(dyp), QPAT_P(dym);
    QPAT_P(kap), QPAT_P(ldis), QPAT_P(labs), QPAT_P(twx), QPAT_P(twy), QPAT_P(twyr);
    QPAT_P(tap_off), QPAT_P(taps), QPAT_P(node_off), QPAT_P(nodes), QPAT_P(scon);
#undef QPAT_V
#undef QPAT_P
    return m;
  }
}
__device__ __forceinline__ Work table_work(const Launch& L, int item) {
  ConstItem* t = (ConstItem*)L.items + item;
  return Work{as_global(t->w.f0), as_global(t->w.f1), as_global(t->w.f2), as_global(t->w.f3),
              as_global(t->w.q),  as_global(t->w.s0), as_global(t->w.s1), as_global(t->w.part)};
}
template <bool U>
__device__ __forceinline__ IOOf<U> io_of(const Launch& L, int item) {
  if constexpr (U) {
    return L.io[item];
  } else {
    ConstIO* t = (ConstIO*)L.io + item;
    return IO{as_global(t->in), as_global(t->out), as_global(t->sens), as_global(t->gc)};
  }
}

__device__ __forceinline__ Work shift_work(const Work& w, long long off) {
  Work r;
  r.f0 = reinterpret_cast<float*>(reinterpret_cast<char*>(w.f0) + off);
  r.f1 = reinterpret_cast<float*>(reinterpret_cast<char*>(w.f1) + off);
  r.f2 = reinterpret_cast<float*>(reinterpret_cast<char*>(w.f2) + off);
  r.f3 = reinterpret_cast<float*>(reinterpret_cast<char*>(w.f3) + off);
  r.q = reinterpret_cast<float*>(reinterpret_cast<char*>(w.q) + off);
  r.s0 = reinterpret_cast<float2*>(reinterpret_cast<char*>(w.s0) + off);
  r.s1 = reinterpret_cast<float2*>(reinterpret_cast<char*>(w.s1) + off);
  r.part = reinterpret_cast<float*>(reinterpret_cast<char*>(w.part) + off);
  return r;
}

// ---------------------------------------------------------------- kernel arguments
// The scalar cache is cold when a kernel starts, so every kernel-argument
// load is a memory round trip.  The compiler issues loads where their values
// are first needed: behind the early-exit branches of the prologue that makes
// two or three dependent round trips before a block's first data load.  These
// empty asm statements take the fields the prologue and the load phase of a
// uniform launch need (and the block size, an implicit argument) as SGPR
// operands, so their loads issue as one batch at the top of the kernel.  Table
// launches read the same fields from the item table, as one batch once the item
// is located.
__device__ __forceinline__ void launch_args_batch(const Launch& L, int ntile, int chunk, int n, int flags) {
  asm volatile("" ::"s"(ntile), "s"(chunk), "s"(n), "s"(flags), "s"(L.nitems), "s"(L.wstride), "s"(L.map),
               "s"(L.items), "s"(L.io), "s"(blockDim.x));
}
// (one statement: the loads of a later one would wait for the earlier)
#define QPAT_ROW_FIELDS(m)                                                                                   \
  "s"(m.nx), "s"(m.nxh), "s"(m.nt), "s"(m.rt), "s"(m.ct), "s"(m.lrt), "s"(m.lct), "s"(m.twx), "s"(m.srt), \
      "s"(m.lsrt)
template <int BM>
__device__ __forceinline__ void row_fields_batch(const Medium& m, const Work& w) {
  if constexpr (BM == RM_F1 || BM == RM_A3) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.s1), "s"(w.f0), "s"(w.f1), "s"(m.bx), "s"(m.by), "s"(m.avx), "s"(m.avy));
  } else if constexpr (BM == RM_F2 || BM == RM_F2L) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.s1), "s"(w.f2), "s"(w.f3), "s"(m.rho0), "s"(m.arx), "s"(m.ary), "s"(m.c2),
                 "s"(m.tap_off));
  } else if constexpr (BM == RM_F3) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.s1), "s"(w.f2), "s"(w.f3), "s"(m.c2), "s"(m.c2eta), "s"(m.c2tau),
                 "s"(m.tap_off));
  } else if constexpr (BM == RM_A1) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.part), "s"(m.c2), "s"(m.c2eta), "s"(m.c2tau), "s"(m.tap_off),
                 "s"(m.taps), "s"(m.ny), "s"(m.ns), "s"(m.node_off), "s"(m.nodes), "s"(m.scon));
  } else if constexpr (BM == RM_A1L) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.f2), "s"(w.f3), "s"(m.c2), "s"(m.rho0), "s"(m.arx), "s"(m.ary),
                 "s"(m.tap_off), "s"(m.node_off), "s"(m.nodes));
  } else if constexpr (BM == RM_A2) {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0), "s"(w.s1), "s"(w.q), "s"(w.f2), "s"(w.f3), "s"(m.rho0), "s"(m.arx), "s"(m.ary));
  } else {
    asm volatile("" ::QPAT_ROW_FIELDS(m), "s"(w.s0));
  }
}

#undef QPAT_ROW_FIELDS
template <int BM>
__device__ __forceinline__ void row_args_batch(const Launch& L, int ntile, int chunk, int n, int flags) {
  asm volatile("" ::"s"(ntile), "s"(chunk), "s"(n), "s"(flags), "s"(L.nitems), "s"(L.wstride), "s"(L.m.nx),
               "s"(L.m.nxh), "s"(L.m.nt), "s"(L.m.rt), "s"(L.m.ct), "s"(L.m.lrt), "s"(L.m.lct), "s"(L.m.twx),
               "s"(blockDim.x));
  row_fields_batch<BM>(L.m, L.w0);
}

#define QPAT_COL_FIELDS(m)                                                                                  \
  "s"(m.ny), "s"(m.nxh), "s"(m.nt), "s"(m.srt), "s"(m.ct), "s"(m.lsrt), "s"(m.lct), "s"(w.s0), "s"(w.s1), \
      "s"(m.twy), "s"(m.twyr)
template <int CM>
__device__ __forceinline__ void col_fields_batch(const Medium& m, const Work& w) {
  if constexpr (CM == CM_FRAC) {
    asm volatile("" ::QPAT_COL_FIELDS(m), "s"(m.ldis), "s"(m.labs));
  } else if constexpr (CM == CM_GRADP1 || CM == CM_GRADP2) {
    asm volatile("" ::QPAT_COL_FIELDS(m), "s"(m.kap), "s"(m.dxp), "s"(m.dyp));
  } else if constexpr (CM == CM_GRADM2 || CM == CM_DIVM) {
    asm volatile("" ::QPAT_COL_FIELDS(m), "s"(m.kap), "s"(m.dxm), "s"(m.dym));
  } else {
    asm volatile("" ::QPAT_COL_FIELDS(m));
  }
}
#undef QPAT_COL_FIELDS
template <int CM>
__device__ __forceinline__ void col_args_batch(const Launch& L, int ntile, int chunk, int n) {
  const Medium& m = L.m;
  asm volatile("" ::"s"(ntile), "s"(chunk), "s"(n), "s"(L.nitems), "s"(L.wstride), "s"(m.ny), "s"(m.nxh),
               "s"(m.nt), "s"(m.srt), "s"(m.ct), "s"(m.lsrt), "s"(m.lct), "s"(L.w0.s0), "s"(L.w0.s1), "s"(m.twy),
               "s"(m.twyr), "s"(blockDim.x));
  col_fields_batch<CM>(m, L.w0);
}

// ---------------------------------------------------------------- row pass
// Every global load of a pass is issued in one phase at the start: spectra and
// twiddles into LDS, pointwise operands into registers (at most kMaxPer
// elements per thread); the FFT stages then run out of LDS only.
#define FOR_K _Pragma("unroll") for (int k = 0; k < kMaxPer; ++k)
// Load loops skip whole iterations on a block-uniform test and clamp the
// ragged last one (its extra lanes re-read the last element): no per-lane
// branch, so the loads of all iterations issue back to back.
#define FOR_K_LD _Pragma("unroll") for (int k = 0; k < kMaxPer; ++k) if (k * B < tot)

// TG: the FFT stages read their twiddles from the plan's table in global
// memory (L1/L2 resident) instead of a copy staged in LDS.  That takes the
// table load and its LDS writes off a block's critical path, which pays when
// a launch has about one block per CU; with several blocks per CU the LDS
// copy (and the occupancy it costs) is the better trade.
template <int MODE, bool U, int NF, bool TG = false>
__global__ void __launch_bounds__(kMaxThreads)
row_kernel(const Launch L, int ntile, int chunk, int n, int flags) {
  constexpr int BM = MODE & ~(RM_X | RM_FZ);
  constexpr bool FZ = (MODE & RM_FZ) != 0;
  constexpr bool XS = (MODE & RM_X) != 0;
  extern __shared__ float2 lds[];
  if constexpr (U) row_args_batch<BM>(L, ntile, chunk, n, flags);
  else launch_args_batch(L, ntile, chunk, n, flags);
  int item, tile;
  if (!locate<U>(L, ntile, chunk, item, tile)) return;
  const MediumOf<U> M = medium_of<U>(L, item);
  const Work W = U ? shift_work(L.w0, item * L.wstride) : table_work(L, item);
  if constexpr (!U) row_fields_batch<BM>(M, W);
  const IOOf<U> X = io_of<U>(L, item);
  if (n > M.nt - 2) return;  // this problem has finished (uneven batches)
  const int nx = row_len<NF>(M), nxh = row_half<NF>(M), rt = M.rt;
  const int y0 = tile * rt;
  const int B = blockDim.x;
  const int LS = lstride(nx);
  // IP: instances with a compile-time length run their FFT stages in place in
  // one LDS buffer unless they read global twiddles (TG, launches of about
  // one block per CU, where the extra barriers would cost): the freed LDS lets
  // more blocks share a CU.
  constexpr bool IP = NF > 0 && !TG;
  constexpr int NBUF = IP ? 1 : 2;
  float2* bufA = lds;
  float2* bufB = IP ? lds : lds + rt * LS;
  float2* const twl = lds + NBUF * rt * LS;
  const float2* const tw = TG ? static_cast<const float2*>(M.twx) : twl;
  void* tap_base = lds + NBUF * rt * LS + (TG ? 0 : nx);
  const int tot = rt * nx;
  const float dt = M.dt;
  const float rnx = 1.0f / static_cast<float>(nx);
  // row j of element it of the tile, and the offset of grid row y (integer
  // shifts / a constant divide when the instance has a compile-time length)
  auto rowdiv = [&](int it) -> int {
    if constexpr (NF > 0) return int(unsigned(it) / unsigned(NF));
    else return fdiv(it, nx, rnx);
  };
  auto rowoff = [&](int y) -> unsigned {
    if constexpr (NF > 0) return unsigned(y) * unsigned(NF);
    else return mul24(y, nx);
  };
  // RM_X variants: this iterate's slot of the sound-speed sensitivities
  float* const sens = XS ? X.sens + size_t(unsigned(flags) >> kSlotShift) * unsigned(nx * M.ny) : nullptr;

  if constexpr ((BM == RM_F1 || BM == RM_A3) && row_fusable<NF>()) {
    // eq num-vel (RM_F1: v_i = A_i (A_i v_i - dt/rho_i d/dr_i^+ p)) and its
    // transpose (RM_A3) with the update between the two FFTs in registers:
    // butterfly (row j, jj) of the boundary stage holds the row's values at
    // x = jj + q N/R
    constexpr int R = plan_radix(NF, 0), NB = NF / R, MB = fused_slots<NF>();
    const bool first = BM == RM_F1 ? (n == 0) : (n == M.nt - 2);  // the state starts at zero
    float v0x[MB][R], v0y[MB][R], bx[MB][R], by[MB][R], ax[MB][R], ay[MB];
    PairRegs S;
    TwRegs TW;
    fetch_pair<NF>(S, M, W.s0, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      if (wave_base() + i * B < rt * NB) {
        const unsigned it = min(unsigned(threadIdx.x + i * B), unsigned(rt * NB) - 1u);
        const int j = int(it / NB), jj = int(it % NB), y = y0 + j;
        const unsigned base = rowoff(y) + jj;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          v0x[i][q] = W.f0[base + q * NB];
          v0y[i][q] = W.f1[base + q * NB];
          bx[i][q] = M.bx[base + q * NB];
          by[i][q] = M.by[base + q * NB];
          ax[i][q] = M.avx[jj + q * NB];
        }
        ay[i] = M.avy[y];
      }
    }
    put_pair<NF>(S, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    auto pw = [&](int i, int j, int jj, float2* v) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
      const unsigned base = rowoff(y0 + j) + jj;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const float2 z = v[q];
        if constexpr (BM == RM_F1) {
          const float vx = ax[i][q] * (ax[i][q] * (first ? 0.f : v0x[i][q]) - bx[i][q] * z.x);
          const float vy = ay[i] * (ay[i] * (first ? 0.f : v0y[i][q]) + by[i][q] * z.y);
          W.f0[base + q * NB] = vx;
          W.f1[base + q * NB] = vy;
          v[q] = make_float2(vx, vy);
        } else {
          const float vbx = (first ? 0.f : v0x[i][q]) - z.x;
          const float vby = (first ? 0.f : v0y[i][q]) + z.y;
          W.f0[base + q * NB] = ax[i][q] * ax[i][q] * vbx;
          W.f1[base + q * NB] = ay[i] * ay[i] * vby;
          v[q] = make_float2(-ax[i][q] * bx[i][q] * vbx, -ay[i] * by[i][q] * vby);
        }
      }
    };
    float2* r = fft_fused<NF, IP>(bufA, bufB, rt, tw, pw);
    store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
  } else if constexpr (BM == RM_F1) {
    // eq num-vel: v_i = A_i (A_i v_i - dt/rho_i d/dr_i^+ p)
    const bool first = (n == 0);  // v^{-1/2} = 0
    float vxo[kMaxPer], vyo[kMaxPer], bx[kMaxPer], by[kMaxPer], ax[kMaxPer], ay[kMaxPer];
    PairRegs S;
    TwRegs TW;
    fetch_pair<NF>(S, M, W.s0, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx, y = y0 + j;
        const unsigned idx = rowoff(y) + x;
        vxo[k] = W.f0[idx];
        vyo[k] = W.f1[idx];
        bx[k] = M.bx[idx];
        by[k] = M.by[idx];
        ax[k] = M.avx[x];
        ay[k] = M.avy[y];
      }
    }
    put_pair<NF>(S, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt, nx, LS, M.radx, M.nstx, tw);
    float2* o = other(r, bufA, bufB);
    // all LDS reads of the loop first: its LDS writes go to the other buffer,
    // which the compiler cannot tell, so an interleaved loop waits per element
    float2 zr[kMaxPer];
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        zr[k] = r[j * LS + px(x)];
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        const float2 z = zr[k];
        const float vx = ax[k] * (ax[k] * (first ? 0.f : vxo[k]) - bx[k] * z.x);
        const float vy = ay[k] * (ay[k] * (first ? 0.f : vyo[k]) + by[k] * z.y);
        W.f0[idx] = vx;
        W.f1[idx] = vy;
        o[j * LS + px(x)] = make_float2(vx, vy);
      }
    }
    __syncthreads();
    r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
    store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
  } else if constexpr (FZ) {
    // RM_FZ instances of the lossy density passes (forward eq num-rho and its
    // transpose) at iterates n >= 1, past the source and the zero initial
    // state: only the fused path is compiled, so the first iterates' code does
    // not set these kernels' register count.  The host launches them only for
    // compile-time lengths whose plan fuses (kernels_row_fused).  Plans whose
    // boundary stage has radix 8 (64, 192 to 768) hold one row per work item, the
    // rows 2l and 2l+1 of a pair in adjacent lanes (fft_fused_pairs); radix-4
    // ones (48, 96, 128, 1024) two rows per work item (fft_fused2), which is
    // faster at 128 and 1024, and only where the twiddles sit in LDS.
    constexpr bool PAIRS = plan_radix(NF > 0 ? NF : 8, 0) > 4;
    if constexpr (BM == RM_F2 && row_fusable<NF>() && PAIRS) {
      // each row's inverse line in, S and u lines (rows 2l, 2l+1 packed) out
      constexpr int R = plan_radix(NF, 0), NB = NF / R, MB = fused_slots<NF>();
      const int half = rt / 2;
      float rxo[MB][R], ryo[MB][R], r0[MB][R], ax[MB][R], ay[MB];
      PairRegs S;
      TwRegs TW;
      fetch_pair<NF>(S, M, W.s0, W.s1, tile);
      if constexpr (!TG) fetch_tw(TW, M.twx, nx);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (wave_base() + i * B < rt * NB) {
          const unsigned it = min(unsigned(threadIdx.x + i * B), unsigned(rt * NB) - 1u);
          const unsigned p = it >> 1, l = p / NB, jj = p % NB;
          const int y = y0 + 2 * int(l) + int(it & 1u);
          const unsigned base = rowoff(y) + jj;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            rxo[i][q] = W.f2[base + q * NB];
            ryo[i][q] = W.f3[base + q * NB];
            r0[i][q] = M.rho0[base + q * NB];
            ax[i][q] = M.arx[jj + q * NB];
          }
          ay[i] = M.ary[y];
        }
      }
      put_pair<NF>(S, bufA, M);
      if constexpr (!TG) put_tw(TW, twl, nx);
      __syncthreads();
      auto inl = [&](int l, int sd) { return 2 * l + sd; };
      auto outl = [&](int l, int sd) { return sd * half + l; };
      auto pw = [&](int i, int l, int sd, int jj, float2* v, bool active) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const unsigned base = rowoff(y0 + 2 * l + sd) + jj;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const float ex = v[q].x, ey = -v[q].y;
          const float s = 0.f;
          const float rx = ax[i][q] * (ax[i][q] * rxo[i][q] - dt * r0[i][q] * ex) + s;
          const float ry = ay[i] * (ay[i] * ryo[i][q] - dt * r0[i][q] * ey) + s;
          if (active) {
            W.f2[base + q * NB] = rx;
            W.f3[base + q * NB] = ry;
          }
          const float sum = rx + ry, u = r0[i][q] * (ax[i][q] * ex + ay[i] * ey);
          // row 2l keeps S and sends u; row 2l+1 keeps u and sends S
          const float got = lane_pair_swap(sd ? sum : u);
          v[q] = sd ? make_float2(got, u) : make_float2(sum, got);
        }
      };
      float2* r = fft_fused_pairs<NF, IP>(bufA, bufB, rt, tw, inl, outl, pw);
      store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
      store_rowpair_spectra<NF, TG>(r + half * LS, M, W.s1, tile);
    } else if constexpr (BM == RM_F2 && row_fusable<NF>() && !TG) {
      // iterates past the source: the update between the two FFTs in
      // registers, rows 2l and 2l+1 of each position together (their S and
      // u values share one complex line each on the output side)
      constexpr int R = plan_radix(NF, 0), NB = NF / R, MB = fused2_slots<NF>();
      const int half = rt / 2;
      float rxa[MB][R], rya[MB][R], r0a[MB][R], rxb[MB][R], ryb[MB][R], r0b[MB][R], ax[MB][R];
      float aya[MB], ayb[MB];
      PairRegs S;
      TwRegs TW;
      fetch_pair<NF>(S, M, W.s0, W.s1, tile);
      if constexpr (!TG) fetch_tw(TW, M.twx, nx);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (wave_base() + i * B < half * NB) {
          const unsigned it = min(unsigned(threadIdx.x + i * B), unsigned(half * NB) - 1u);
          const int l = int(it / NB), jj = int(it % NB), ya = y0 + 2 * l;
          const unsigned ba = rowoff(ya) + jj, bb = ba + nx;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            rxa[i][q] = W.f2[ba + q * NB];
            rya[i][q] = W.f3[ba + q * NB];
            r0a[i][q] = M.rho0[ba + q * NB];
            rxb[i][q] = W.f2[bb + q * NB];
            ryb[i][q] = W.f3[bb + q * NB];
            r0b[i][q] = M.rho0[bb + q * NB];
            ax[i][q] = M.arx[jj + q * NB];
          }
          aya[i] = M.ary[ya];
          ayb[i] = M.ary[ya + 1];
        }
      }
      put_pair<NF>(S, bufA, M);
      if constexpr (!TG) put_tw(TW, twl, nx);
      __syncthreads();
      auto inl = [&](int l, int sd) { return 2 * l + sd; };
      auto outl = [&](int l, int sd) { return sd * half + l; };
      auto pw = [&](int i, int l, int jj, float2* va, float2* vb) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const unsigned ba = rowoff(y0 + 2 * l) + jj, bb = ba + nx;
        const float s = 0.f;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const float exa = va[q].x, eya = -va[q].y, exb = vb[q].x, eyb = -vb[q].y;
          const float rxA = ax[i][q] * (ax[i][q] * rxa[i][q] - dt * r0a[i][q] * exa) + s;
          const float ryA = aya[i] * (aya[i] * rya[i][q] - dt * r0a[i][q] * eya) + s;
          const float rxB = ax[i][q] * (ax[i][q] * rxb[i][q] - dt * r0b[i][q] * exb) + s;
          const float ryB = ayb[i] * (ayb[i] * ryb[i][q] - dt * r0b[i][q] * eyb) + s;
          W.f2[ba + q * NB] = rxA;
          W.f3[ba + q * NB] = ryA;
          W.f2[bb + q * NB] = rxB;
          W.f3[bb + q * NB] = ryB;
          va[q] = make_float2(rxA + ryA, rxB + ryB);
          vb[q] = make_float2(r0a[i][q] * (ax[i][q] * exa + aya[i] * eya), r0b[i][q] * (ax[i][q] * exb + ayb[i] * eyb));
        }
      };
      float2* r = fft_fused2<NF, IP>(bufA, bufB, rt, tw, inl, outl, pw);
      store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
      store_rowpair_spectra<NF, TG>(r + half * LS, M, W.s1, tile);
    } else if constexpr (BM == RM_A2 && row_fusable<NF>() && PAIRS) {
      // the eta / tau lines (rows 2l, 2l+1 packed) in, each row's line out
      const bool first = (n == M.nt - 2);
      constexpr int R = plan_radix(NF, 0), NB = NF / R, MB = fused_slots<NF>();
      const int half = rt / 2;
      float qv[MB][R], x0[MB][R], y0v[MB][R], r0[MB][R], ax[MB][R], ay[MB];
      RowPairRegs S0, S1;
      TwRegs TW;
      fetch_rowpair<NF>(S0, M, W.s0, tile);
      fetch_rowpair<NF>(S1, M, W.s1, tile);
      if constexpr (!TG) fetch_tw(TW, M.twx, nx);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (wave_base() + i * B < rt * NB) {
          const unsigned it = min(unsigned(threadIdx.x + i * B), unsigned(rt * NB) - 1u);
          const unsigned p = it >> 1, l = p / NB, jj = p % NB;
          const int y = y0 + 2 * int(l) + int(it & 1u);
          const unsigned base = rowoff(y) + jj;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            qv[i][q] = W.q[base + q * NB];
            x0[i][q] = W.f2[base + q * NB];
            y0v[i][q] = W.f3[base + q * NB];
            r0[i][q] = M.rho0[base + q * NB];
            ax[i][q] = M.arx[jj + q * NB];
          }
          ay[i] = M.ary[y];
        }
      }
      put_rowpair<NF>(S0, bufA, M);
      put_rowpair<NF>(S1, bufA + half * LS, M);
      if constexpr (!TG) put_tw(TW, twl, nx);
      __syncthreads();
      auto inl = [&](int l, int sd) { return sd * half + l; };
      auto outl = [&](int l, int sd) { return 2 * l + sd; };
      auto pw = [&](int i, int l, int sd, int jj, float2* v, bool active) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const unsigned base = rowoff(y0 + 2 * l + sd) + jj;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          // row 2l holds the eta line (yd of rows 2l, 2l+1), row 2l+1 the tau
          // line (ya of rows 2l, 2l+1): each sends the value the other's row needs
          const float got = lane_pair_swap(sd ? v[q].x : -v[q].y);
          const float yd = sd ? got : v[q].x, ya = sd ? -v[q].y : got;
          const float sb = qv[i][q] - yd;
          const float rbx = (first ? 0.f : x0[i][q]) + sb, rby = (first ? 0.f : y0v[i][q]) + sb;
          v[q] = make_float2(r0[i][q] * ax[i][q] * (ya - dt * rbx), r0[i][q] * ay[i] * (ya - dt * rby));
          if (active) {
            W.f2[base + q * NB] = ax[i][q] * ax[i][q] * rbx;
            W.f3[base + q * NB] = ay[i] * ay[i] * rby;
          }
        }
      };
      float2* r = fft_fused_pairs<NF, IP>(bufA, bufB, rt, tw, inl, outl, pw);
      store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
    } else if constexpr (BM == RM_A2 && row_fusable<NF>() && !TG) {
      const bool first = (n == M.nt - 2);
      // the update between the two FFTs in registers: rows 2l and 2l+1 of
      // each position together (they share the input lines)
      constexpr int R = plan_radix(NF, 0), NB = NF / R, MB = fused2_slots<NF>();
      const int half = rt / 2;
      float qa[MB][R], xa[MB][R], ya0[MB][R], r0a[MB][R], qb[MB][R], xb[MB][R], yb0[MB][R], r0b[MB][R];
      float ax[MB][R], aya[MB], ayb[MB];
      RowPairRegs S0, S1;
      TwRegs TW;
      fetch_rowpair<NF>(S0, M, W.s0, tile);
      fetch_rowpair<NF>(S1, M, W.s1, tile);
      if constexpr (!TG) fetch_tw(TW, M.twx, nx);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (wave_base() + i * B < half * NB) {
          const unsigned it = min(unsigned(threadIdx.x + i * B), unsigned(half * NB) - 1u);
          const int l = int(it / NB), jj = int(it % NB), y = y0 + 2 * l;
          const unsigned ba = rowoff(y) + jj, bb = ba + nx;
#pragma unroll
          for (int q = 0; q < R; ++q) {
            qa[i][q] = W.q[ba + q * NB];
            xa[i][q] = W.f2[ba + q * NB];
            ya0[i][q] = W.f3[ba + q * NB];
            r0a[i][q] = M.rho0[ba + q * NB];
            qb[i][q] = W.q[bb + q * NB];
            xb[i][q] = W.f2[bb + q * NB];
            yb0[i][q] = W.f3[bb + q * NB];
            r0b[i][q] = M.rho0[bb + q * NB];
            ax[i][q] = M.arx[jj + q * NB];
          }
          aya[i] = M.ary[y];
          ayb[i] = M.ary[y + 1];
        }
      }
      put_rowpair<NF>(S0, bufA, M);
      put_rowpair<NF>(S1, bufA + half * LS, M);
      if constexpr (!TG) put_tw(TW, twl, nx);
      __syncthreads();
      auto inl = [&](int l, int sd) { return sd * half + l; };
      auto outl = [&](int l, int sd) { return 2 * l + sd; };
      auto pw = [&](int i, int l, int jj, float2* va, float2* vb) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const unsigned ba = rowoff(y0 + 2 * l) + jj, bb = ba + nx;
#pragma unroll
        for (int q = 0; q < R; ++q) {
          // rows 2l and 2l+1 of the (conjugated) inverse transforms
          const float yda = va[q].x, ydb = -va[q].y, yaa = vb[q].x, yab = -vb[q].y;
          const float sba = qa[i][q] - yda, sbb = qb[i][q] - ydb;
          const float rbxa = (first ? 0.f : xa[i][q]) + sba, rbya = (first ? 0.f : ya0[i][q]) + sba;
          const float rbxb = (first ? 0.f : xb[i][q]) + sbb, rbyb = (first ? 0.f : yb0[i][q]) + sbb;
          va[q] = make_float2(r0a[i][q] * ax[i][q] * (yaa - dt * rbxa), r0a[i][q] * aya[i] * (yaa - dt * rbya));
          vb[q] = make_float2(r0b[i][q] * ax[i][q] * (yab - dt * rbxb), r0b[i][q] * ayb[i] * (yab - dt * rbyb));
          W.f2[ba + q * NB] = ax[i][q] * ax[i][q] * rbxa;
          W.f3[ba + q * NB] = aya[i] * aya[i] * rbya;
          W.f2[bb + q * NB] = ax[i][q] * ax[i][q] * rbxb;
          W.f3[bb + q * NB] = ayb[i] * ayb[i] * rbyb;
        }
      };
      float2* r = fft_fused2<NF, IP>(bufA, bufB, rt, tw, inl, outl, pw);
      store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
    }
  } else if constexpr (BM == RM_F2 || BM == RM_F2L) {
    // eq num-rho with the additive source of eq s1 (dt s = p0 / (2 d c^2), d = 2)
    const bool skip = (n == -1);  // v^{-1/2} = 0 and rho^{-1} = 0
    const bool inject = (n <= 0);
    float rxo[kMaxPer], ryo[kMaxPer], r0[kMaxPer], ax[kMaxPer], ay[kMaxPer], src[kMaxPer], c2[kMaxPer];
    PairRegs S;
    TwRegs TW;
    TapStage T{};
    if constexpr (BM == RM_F2L) taps_range(T, M, tap_base, y0, rt);
    if (!skip) fetch_pair<NF>(S, M, W.s0, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx, y = y0 + j;
        const unsigned idx = rowoff(y) + x;
        rxo[k] = W.f2[idx];
        ryo[k] = W.f3[idx];
        r0[k] = M.rho0[idx];
        ax[k] = M.arx[x];
        ay[k] = M.ary[y];
        if constexpr (BM == RM_F2L) c2[k] = M.c2[idx];
      }
    }
    if (inject) {  // first two iterates only (kept apart so the loads above issue back to back)
      FOR_K_LD {
        const int it = min(int(threadIdx.x) + k * B, tot - 1);
        {
          const int j = rowdiv(it), x = it - j * nx;
          const unsigned idx = rowoff(y0 + j) + x;
          if constexpr (BM != RM_F2L) c2[k] = M.c2[idx];
          src[k] = X.in[idx];
        }
      }
    }
    if (!skip) put_pair<NF>(S, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    if constexpr (BM == RM_F2L) taps_fetch(T, M, nullptr, 0);
    float2* r = nullptr;
    float2* o = bufA;
    if (!skip) {
      r = fft_any<NF, IP, !U>(bufA, bufB, rt, nx, LS, M.radx, M.nstx, tw);
      o = other(r, bufA, bufB);
    }
    float2 zr[kMaxPer];
    if (!skip) {
      FOR_K {
        const int it = threadIdx.x + k * B;
        if (it < tot) {
          const int j = rowdiv(it), x = it - j * nx;
          zr[k] = r[j * LS + px(x)];
        }
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        float ex = 0.f, ey = 0.f;
        if (!skip) {
          const float2 z = zr[k];
          ex = z.x;
          ey = -z.y;
        } else {
          W.f0[idx] = 0.f;  // the state z_0 holds v^{-1/2} = 0
          W.f1[idx] = 0.f;
        }
        const float s = inject ? src[k] * (0.25f / c2[k]) : 0.f;
        const float rx = ax[k] * (ax[k] * (skip ? 0.f : rxo[k]) - dt * r0[k] * ex) + s;
        const float ry = ay[k] * (ay[k] * (skip ? 0.f : ryo[k]) - dt * r0[k] * ey) + s;
        W.f2[idx] = rx;
        W.f3[idx] = ry;
        if constexpr (BM == RM_F2) {
          // S = sum_i rho_i and u = rho0 sum_i A_i d/dr_i^- v_i feed eq num-p.
          // Each is transformed with its own rows paired (S and u differ by
          // orders of magnitude, so they must not share one complex FFT).
          pcomp(o, j, x, nx) = rx + ry;
          pcomp(o + (rt / 2) * LS, j, x, nx) = r0[k] * (ax[k] * ex + ay[k] * ey);
        } else {
          const float p = c2[k] * (rx + ry);
          pcomp(o, j, x, nx) = p;
          if (flags & FL_STORE_P) W.q[idx] = p;
          if constexpr (XS) sens[idx] = 2.f * p * rsqrtf(c2[k]);  // d(c^2 S)/dc
        }
      }
    }
    if constexpr (BM == RM_F2L) taps_put(T, false);
    __syncthreads();
    if constexpr (BM == RM_F2) {
      r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
      store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
      store_rowpair_spectra<NF, TG>(r + (rt / 2) * LS, M, W.s1, tile);
    } else {
      if (!(flags & FL_NO_SENSORS)) sensor_partials(M, T, o, y0, W.part, n + 1);
      r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt / 2, nx, LS, M.radx, M.nstx, tw);
      store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
    }
  } else if constexpr (BM == RM_F3) {
    // eq num-p: p = c^2 (S - eta Y_dis S + tau Y_abs u)
    float rxo[kMaxPer], ryo[kMaxPer], c2[kMaxPer], ce[kMaxPer], ctau[kMaxPer];
    TapStage T;
    taps_range(T, M, tap_base, y0, rt);
    RowPairRegs S0, S1;
    TwRegs TW;
    fetch_rowpair<NF>(S0, M, W.s0, tile);
    fetch_rowpair<NF>(S1, M, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        rxo[k] = W.f2[idx];
        ryo[k] = W.f3[idx];
        c2[k] = M.c2[idx];
        ce[k] = M.c2eta[idx];
        ctau[k] = M.c2tau[idx];
      }
    }
    put_rowpair<NF>(S0, bufA, M);
    put_rowpair<NF>(S1, bufA + (rt / 2) * LS, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    taps_fetch(T, M, nullptr, 0);
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt, nx, LS, M.radx, M.nstx, tw);
    float2* o = other(r, bufA, bufB);
    float ysr[kMaxPer], yur[kMaxPer];
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        ysr[k] = rowpair_val(r, j, x, nx);
        yur[k] = rowpair_val(r + (rt / 2) * LS, j, x, nx);
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        const float ys = ysr[k], yu = yur[k];
        const float p = c2[k] * (rxo[k] + ryo[k]) - ce[k] * ys + ctau[k] * yu;
        pcomp(o, j, x, nx) = p;
        const unsigned idx = rowoff(y0 + j) + x;
        if (flags & FL_STORE_P) W.q[idx] = p;
        if constexpr (XS) {
          // eq Twelve: c^2 eta ~ c^(y+2) and c^2 tau ~ c^(y+1), so each term of
          // eq num-p differentiates to its power over c
          const float S = rxo[k] + ryo[k];
          sens[idx] = (2.f * c2[k] * S - (M.ypow + 2.f) * ce[k] * ys + (M.ypow + 1.f) * ctau[k] * yu) * rsqrtf(c2[k]);
        }
      }
    }
    taps_put(T, false);
    __syncthreads();
    if (!(flags & FL_NO_SENSORS)) sensor_partials(M, T, o, y0, W.part, n + 1);
    r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt / 2, nx, LS, M.radx, M.nstx, tw);
    store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
  } else if constexpr (BM == RM_A1 || BM == RM_A1L) {
    // transpose of eqs num-m and num-p: p* += M^T r_{n+1}; q = c^2 p*
    const bool first = (n == M.nt - 2);
    const int half = rt / 2;
    float c2[kMaxPer], ce[kMaxPer], ctau[kMaxPer], rbx0[kMaxPer], rby0[kMaxPer], r0[kMaxPer];
    float ax[kMaxPer], ay[kMaxPer], gacc[kMaxPer];
    TapStage T;
    taps_range(T, M, tap_base, y0, rt, true);
    RowPairRegs S0;
    TwRegs TW;
    if (!first) fetch_rowpair<NF>(S0, M, W.s0, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx, y = y0 + j;
        const unsigned idx = rowoff(y) + x;
        c2[k] = M.c2[idx];
        if constexpr (BM == RM_A1) {
          ce[k] = M.c2eta[idx];
          ctau[k] = M.c2tau[idx];
        } else {
          rbx0[k] = W.f2[idx];
          rby0[k] = W.f3[idx];
          r0[k] = M.rho0[idx];
          ax[k] = M.arx[x];
          ay[k] = M.ary[y];
        }
      }
    }
    float sv[kMaxPer];
    double gprev[kMaxPer];
    if constexpr (XS) {
      FOR_K_LD {
        const int it = min(int(threadIdx.x) + k * B, tot - 1);
        {
          const int j = rowdiv(it), x = it - j * nx;
          const unsigned idx = rowoff(y0 + j) + x;
          sv[k] = sens[idx];
          gprev[k] = first ? 0.0 : X.gc[idx];
        }
      }
    }
    if constexpr (BM == RM_A1L) {
      if (n == -1 && M.nt >= 2) {  // the gradient accumulated at n = 0
        FOR_K_LD {
          const int it = min(int(threadIdx.x) + k * B, tot - 1);
          {
            const int j = rowdiv(it), x = it - j * nx;
            gacc[k] = X.out[rowoff(y0 + j) + x];
          }
        }
      }
    }
    if (!first) put_rowpair<NF>(S0, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    taps_fetch(T, M, W.part, n + 1);
    nodes_fetch(T, M);
    float2* r = bufA;
    if (!first) {
      r = fft_any<NF, IP, !U>(bufA, bufB, half, nx, LS, M.radx, M.nstx, tw);
      // p* = -(grad_x^- g_x + grad_y^- g_y): negate the (conjugated) inverse
#pragma unroll 4
      for (int it = threadIdx.x; it < half * LS; it += B) {
        const float2 z = r[it];
        r[it] = make_float2(-z.x, z.y);
      }
    } else {
      for (int it = threadIdx.x; it < half * LS; it += B) r[it] = make_float2(0.f, 0.f);
    }
    taps_put(T, true);
    __syncthreads();
    sensor_scatter(M, T, r, y0, W.part, n + 1);
    __syncthreads();
    float2* o = other(r, bufA, bufB);
    float pbr[kMaxPer];
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        pbr[k] = pcomp(r, j, x, nx);
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        const float pb = pbr[k];
        if constexpr (XS) X.gc[idx] = gprev[k] + double(pb) * double(sv[k]);
        if constexpr (BM == RM_A1) {
          // eta q and tau q, each with its own rows paired (see RM_F2)
          W.q[idx] = c2[k] * pb;
          pcomp(o, j, x, nx) = ce[k] * pb;
          pcomp(o + half * LS, j, x, nx) = ctau[k] * pb;
        } else {
          // lossless: S* = q, u* = 0, then the transposed mass update
          const float q = c2[k] * pb;
          const float rbx = (first ? 0.f : rbx0[k]) + q, rby = (first ? 0.f : rby0[k]) + q;
          if (n == 0) X.out[idx] = rbx + rby;
          if (n == -1) {
            X.out[idx] = (rbx + rby + (M.nt >= 2 ? gacc[k] : 0.f)) * (0.25f / c2[k]);
          } else {
            o[j * LS + px(x)] = make_float2(-dt * r0[k] * ax[k] * rbx, -dt * r0[k] * ay[k] * rby);
            W.f2[idx] = ax[k] * ax[k] * rbx;
            W.f3[idx] = ay[k] * ay[k] * rby;
          }
        }
      }
    }
    __syncthreads();
    if constexpr (BM == RM_A1) {
      r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
      store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
      store_rowpair_spectra<NF, TG>(r + half * LS, M, W.s1, tile);
    } else if (n != -1) {
      r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
      store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
    }
  } else if constexpr (BM == RM_A2) {
    // transpose of the mass update and of the Y terms of eq num-p
    const bool first = (n == M.nt - 2);
    float qv[kMaxPer], rbx0[kMaxPer], rby0[kMaxPer], r0[kMaxPer], ax[kMaxPer], ay[kMaxPer];
    float c2[kMaxPer], gacc[kMaxPer];
    RowPairRegs S0, S1;
    TwRegs TW;
    fetch_rowpair<NF>(S0, M, W.s0, tile);
    fetch_rowpair<NF>(S1, M, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx, y = y0 + j;
        const unsigned idx = rowoff(y) + x;
        qv[k] = W.q[idx];
        rbx0[k] = W.f2[idx];
        rby0[k] = W.f3[idx];
        r0[k] = M.rho0[idx];
        ax[k] = M.arx[x];
        ay[k] = M.ary[y];
      }
    }
    if (n == -1) {  // the last iterate: gradient scaling and the sum accumulated at n = 0
      FOR_K_LD {
        const int it = min(int(threadIdx.x) + k * B, tot - 1);
        {
          const int j = rowdiv(it), x = it - j * nx;
          const unsigned idx = rowoff(y0 + j) + x;
          c2[k] = M.c2[idx];
          gacc[k] = M.nt >= 2 ? X.out[idx] : 0.f;
        }
      }
    }
    put_rowpair<NF>(S0, bufA, M);
    put_rowpair<NF>(S1, bufA + (rt / 2) * LS, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt, nx, LS, M.radx, M.nstx, tw);
    float2* o = other(r, bufA, bufB);
    float ydr[kMaxPer], yar[kMaxPer];
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        ydr[k] = rowpair_val(r, j, x, nx);
        yar[k] = rowpair_val(r + (rt / 2) * LS, j, x, nx);
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        const float yd = ydr[k], ya = yar[k];
        const float sb = qv[k] - yd;
        const float rbx = (first ? 0.f : rbx0[k]) + sb, rby = (first ? 0.f : rby0[k]) + sb;
        if (n == 0) X.out[idx] = rbx + rby;
        if (n == -1) {
          X.out[idx] = (rbx + rby + gacc[k]) * (0.25f / c2[k]);
        } else {
          o[j * LS + px(x)] = make_float2(r0[k] * ax[k] * (ya - dt * rbx), r0[k] * ay[k] * (ya - dt * rby));
          W.f2[idx] = ax[k] * ax[k] * rbx;
          W.f3[idx] = ay[k] * ay[k] * rby;
        }
      }
    }
    __syncthreads();
    if (n != -1) {
      r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
      store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
    }
  } else if constexpr (BM == RM_A3) {
    // transpose of eq num-vel
    const bool first = (n == M.nt - 2);
    float vbx0[kMaxPer], vby0[kMaxPer], bx[kMaxPer], by[kMaxPer], ax[kMaxPer], ay[kMaxPer];
    PairRegs S;
    TwRegs TW;
    fetch_pair<NF>(S, M, W.s0, W.s1, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx, y = y0 + j;
        const unsigned idx = rowoff(y) + x;
        vbx0[k] = W.f0[idx];
        vby0[k] = W.f1[idx];
        bx[k] = M.bx[idx];
        by[k] = M.by[idx];
        ax[k] = M.avx[x];
        ay[k] = M.avy[y];
      }
    }
    put_pair<NF>(S, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt, nx, LS, M.radx, M.nstx, tw);
    float2* o = other(r, bufA, bufB);
    float2 zr[kMaxPer];
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        zr[k] = r[j * LS + px(x)];
      }
    }
    if constexpr (IP) __syncthreads();  // the loop below writes the buffer just read
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
#pragma clang fp contract(off)  // the same rounding fused or not (no cross-path contraction choices)
        const int j = rowdiv(it), x = it - j * nx;
        const unsigned idx = rowoff(y0 + j) + x;
        const float2 z = zr[k];
        const float vbx = (first ? 0.f : vbx0[k]) - z.x;
        const float vby = (first ? 0.f : vby0[k]) + z.y;
        o[j * LS + px(x)] = make_float2(-ax[k] * bx[k] * vbx, -ay[k] * by[k] * vby);
        W.f0[idx] = ax[k] * ax[k] * vbx;
        W.f1[idx] = ay[k] * ay[k] * vby;
      }
    }
    __syncthreads();
    r = fft_any<NF, IP, !U>(o, other(o, bufA, bufB), rt, nx, LS, M.radx, M.nstx, tw);
    store_pair_spectra<NF, TG>(r, M, W.s0, W.s1, tile);
  } else if constexpr (BM == RM_FWD1) {
    const float* src = X.in;
    TwRegs TW;
    float v[kMaxPer];
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    FOR_K_LD {
      const int it = min(int(threadIdx.x) + k * B, tot - 1);
      {
        const int j = rowdiv(it), x = it - j * nx;
        v[k] = src[rowoff(y0 + j) + x];
      }
    }
    FOR_K {
      const int it = threadIdx.x + k * B;
      if (it < tot) {
        const int j = rowdiv(it), x = it - j * nx;
        pcomp(bufA, j, x, nx) = v[k];
      }
    }
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt / 2, nx, LS, M.radx, M.nstx, tw);
    store_rowpair_spectra<NF, TG>(r, M, W.s0, tile);
  } else if constexpr (BM == RM_INV1) {
    RowPairRegs S0;
    TwRegs TW;
    fetch_rowpair<NF>(S0, M, W.s0, tile);
    if constexpr (!TG) fetch_tw(TW, M.twx, nx);
    put_rowpair<NF>(S0, bufA, M);
    if constexpr (!TG) put_tw(TW, twl, nx);
    __syncthreads();
    float2* r = fft_any<NF, IP, !U>(bufA, bufB, rt / 2, nx, LS, M.radx, M.nstx, tw);
    float* dst = X.out;
#pragma unroll 4
    for (int it = threadIdx.x; it < tot; it += B) {
      const int j = rowdiv(it), x = it - j * nx;
      dst[rowoff(y0 + j) + x] = rowpair_val(r, j, x, nx);
    }
  }
}

// ---------------------------------------------------------------- column pass
// Multipliers of a launch are either the staggered gradients (kappa times a
// 1-D symbol in x or y) or the fractional-Laplacian tables; the values a
// thread needs are prefetched into registers in the load phase.
struct MultPre {
  float a, b;     // table A / B at (kx, ky): kappa (or Y_dis) and Y_abs
  float an, bn;   // the same at the Nyquist column (packed column 0 only)
  float2 sx, sxn; // x symbol at kx and at the Nyquist column
  float2 sy;      // y symbol at ky
};

__device__ __forceinline__ float2 mult_of(int code, const MultPre& P, bool nyq) {
  switch (code) {
    case MC_DXP:
    case MC_DXM: return cscale(nyq ? P.sxn : P.sx, nyq ? P.an : P.a);
    case MC_DYP:
    case MC_DYM: return cscale(P.sy, nyq ? P.an : P.a);
    case MC_LDIS: return make_float2(nyq ? P.an : P.a, 0.f);
    case MC_LABS: return make_float2(nyq ? P.bn : P.b, 0.f);
    default: return make_float2(0.f, 0.f);
  }
}

// Column-pass kinds: multiplier codes (out_o = sum_i M[o][i] in_i), inputs, outputs.
__device__ constexpr int kColCode[kColModes] = {
    mpack(MC_DXP, 0, MC_DYP, 0),    // CM_GRADP1: d/dx^+ p, d/dy^+ p
    mpack(MC_DXM, 0, 0, MC_DYM),    // CM_GRADM2: d/dx^- v_x, d/dy^- v_y
    mpack(MC_LDIS, 0, 0, MC_LABS),  // CM_FRAC:   Y_dis S, Y_abs u
    mpack(MC_DXP, 0, 0, MC_DYP),    // CM_GRADP2: d/dx^+ e_x, d/dy^+ e_y
    mpack(MC_DXM, MC_DYM, 0, 0),    // CM_DIVM:   d/dx^- g_x + d/dy^- g_y
    0};                             // CM_APPLY:  one operator given at launch
__device__ constexpr int kColIn[kColModes] = {1, 2, 2, 2, 2, 1};
__device__ constexpr int kColOut[kColModes] = {2, 2, 2, 2, 1, 1};

// Column pass of the lengths without a compile-time plan (8 to 24): the tile
// goes through LDS between every phase.
template <int CM>
__device__ __forceinline__ void col_generic(const Medium& M, const Work& W, int tile, int mcode, float2* lds) {
  constexpr int nin = kColIn[CM], nout = kColOut[CM];
  const int ny = M.ny, nxh = M.nxh, ct = M.ct, ls = col_lstride(ny);
  const int c0 = tile * ct;
  const int B = blockDim.x;
  const int nsl = 2;
  float2* bufA = lds;
  float2* bufB = lds + nsl * ct * ls;
  float2* const tw = lds + 2 * nsl * ct * ls;
  // which tables this launch uses
  int xcode = 0, ycode = 0;
  bool frac = false, labs = false;
  for (int e = 0; e < 4; ++e) {
    const int c = (mcode >> (4 * e)) & 15;
    if (c == MC_DXP || c == MC_DXM) xcode = c;
    if (c == MC_DYP || c == MC_DYM) ycode = c;
    if (c == MC_LDIS) frac = true;
    if (c == MC_LABS) { frac = true; labs = true; }
  }
  const float* tabA = frac ? M.ldis : M.kap;
  const float2* symx = xcode == MC_DXP ? M.dxp : M.dxm;
  const float2* symy = ycode == MC_DYP ? M.dyp : M.dym;
  // load phase: the tile (transposed into lines), twiddles, multiplier values
  // memory order: field, tile row ty, element (iy, c) of the srt x ct tile
  const float rny = 1.0f / static_cast<float>(ny);
  const int rc = M.srt * ct;
  // (a tile holds nin*ct*ny <= nin*kColPer*B elements: all loads are issued
  // into registers before the first LDS write)
  constexpr int kIt = nin * kColPer;
  const unsigned ncol = unsigned(ct) * ny, ntot = nin * ncol;     // elements per field / tile
  const unsigned rowstep = unsigned(nxh) * M.srt, tbase = unsigned(tile) * rc;  // tile row ty at ty * rowstep
  const int lsh = M.lsrt + M.lct;
  float2 tv[kIt];
#pragma unroll
  for (int k = 0; k < kIt; ++k) {
    const unsigned it = threadIdx.x + k * B;
    if (it < ntot) {
      const bool f = it >= ncol;
      const unsigned rem = f ? it - ncol : it;
      tv[k] = (f ? W.s1 : W.s0)[mul24(rem >> lsh, rowstep) + tbase + (rem & (rc - 1))];
    }
  }
  TwRegsK<kColPer> TW;  // ny <= kColPer * B
  fetch_tw(TW, M.twy, ny);
  const int tot = ct * ny;
  MultPre P[kColPer];
#pragma unroll
  for (int k = 0; k < kColPer; ++k) {
    const int it = threadIdx.x + k * B;
    if (it < tot) {
      const int c = ct == 1 ? 0 : fdiv(it, ny, rny), ky = it - c * ny, kx = c0 + c;
      const unsigned t = mul24(kx, ny) + ky, tn = mul24(nxh, ny) + ky;   // tables are [kx][ky]
      MultPre& p = P[k];
      p.a = tabA[t];
      p.b = labs ? M.labs[t] : 0.f;
      p.sx = xcode ? symx[kx] : make_float2(0.f, 0.f);
      p.sy = ycode ? symy[ky] : make_float2(0.f, 0.f);
      if (kx == 0) {
        p.an = tabA[tn];
        p.bn = labs ? M.labs[tn] : 0.f;
        p.sxn = xcode ? symx[nxh] : make_float2(0.f, 0.f);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kIt; ++k) {
    const unsigned it = threadIdx.x + k * B;
    if (it < ntot) {
      const bool f = it >= ncol;
      const unsigned rem = f ? it - ncol : it, w = rem & (rc - 1);
      const unsigned ky = ((rem >> lsh) << M.lsrt) + (w >> M.lct), c = w & (ct - 1);
      bufA[mul24((f ? ct : 0) + c, ls) + px(ky)] = tv[k];
    }
  }
  put_tw(TW, tw, ny);
  __syncthreads();
  float2* r = fft_lines(bufA, bufB, nin * ct, ny, ls, M.rady, M.nsty, tw);
  float2* o = other(r, bufA, bufB);
#pragma unroll
  for (int k = 0; k < kColPer; ++k) {
    const int it = threadIdx.x + k * B;
    if (it < tot) {
      const int c = ct == 1 ? 0 : fdiv(it, ny, rny), ky = it - c * ny;
      const int kx = c0 + c;
      const MultPre& p = P[k];
      // (loops over fields have compile-time bounds so the arrays stay in registers)
      if (kx == 0) {
        // packed column: DC (real part) and Nyquist (imaginary part) columns
        const int km = ky ? ny - ky : 0;
        float2 f0[2], fn[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          if (f < nin) {
            const float2 z = r[mul24(f * ct + c, ls) + px(ky)], zm = cconj(r[mul24(f * ct + c, ls) + px(km)]);
            f0[f] = cscale(cadd(z, zm), 0.5f);
            fn[f] = mul_mi(cscale(csub(z, zm), 0.5f));
          } else {
            f0[f] = fn[f] = make_float2(0.f, 0.f);
          }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (q < nout) {
            float2 g0 = make_float2(0.f, 0.f), gn = make_float2(0.f, 0.f);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              const int code = (mcode >> (4 * (2 * q + f))) & 15;
              if (code) {
                g0 = cadd(g0, cmul(mult_of(code, p, false), f0[f]));
                gn = cadd(gn, cmul(mult_of(code, p, true), fn[f]));
              }
            }
            // W = G0 + i GN, stored conjugated for the inverse transform
            o[mul24(q * ct + c, ls) + px(ky)] = cconj(make_float2(g0.x - gn.y, g0.y + gn.x));
          }
        }
      } else {
        float2 in[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) in[f] = f < nin ? r[mul24(f * ct + c, ls) + px(ky)] : make_float2(0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (q < nout) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              const int code = (mcode >> (4 * (2 * q + f))) & 15;
              if (code) acc = cadd(acc, cmul(mult_of(code, p, false), in[f]));
            }
            o[mul24(q * ct + c, ls) + px(ky)] = cconj(acc);
          }
        }
      }
    }
  }
  __syncthreads();
  r = fft_lines(o, other(o, bufA, bufB), nout * ct, ny, ls, M.rady, M.nsty, tw);
  for (unsigned it = threadIdx.x; it < nout * ncol; it += B) {
    const bool f = it >= ncol;
    const unsigned rem = f ? it - ncol : it, w = rem & (rc - 1), ty = rem >> lsh;
    const unsigned ky = (ty << M.lsrt) + (w >> M.lct), c = w & (ct - 1);
    (f ? W.s1 : W.s0)[mul24(ty, rowstep) + tbase + w] = cconj(r[mul24((f ? ct : 0) + c, ls) + px(ky)]);
  }
}

// Value of one multiplier code applied to z at (ky, kx): a = kappa (or Y_dis),
// b = Y_abs, sx / sy the 1-D staggered symbols at kx / ky.
__device__ __forceinline__ float2 mult_apply(int code, float a, float b, float2 sx, float2 sy, float2 z) {
  switch (code) {
    case MC_DXP:
    case MC_DXM: return cmul(cscale(sx, a), z);
    case MC_DYP:
    case MC_DYM: return cmul(cscale(sy, a), z);
    case MC_LDIS: return cscale(z, a);
    case MC_LABS: return cscale(z, b);
    default: return make_float2(0.f, 0.f);
  }
}

// Conjugated products of the packed DC / Nyquist column at row ky: z[f] is
// field f's forward spectrum there, zm[f] the conjugate at the mirror row
// ny - ky; the two real columns are separated, multiplied with their own
// tables (a, b at kx = 0; an, bn at the Nyquist column) and packed again.
template <int CM>
__device__ __forceinline__ void packed_products(int mcode, float a, float b, float an, float bn, float2 sx,
                                                float2 sxn, float2 sy, const float2* z, const float2* zm,
                                                float2* g) {
  constexpr int nin = kColIn[CM], nout = kColOut[CM];
  float2 f0[2], fn[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    if (f < nin) {
      f0[f] = cscale(cadd(z[f], zm[f]), 0.5f);
      fn[f] = mul_mi(cscale(csub(z[f], zm[f]), 0.5f));
    } else {
      f0[f] = fn[f] = make_float2(0.f, 0.f);
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (q < nout) {
      float2 g0 = make_float2(0.f, 0.f), gn = make_float2(0.f, 0.f);
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int code = (mcode >> (4 * (2 * q + f))) & 15;
        if (code) {
          g0 = cadd(g0, mult_apply(code, a, b, sx, sy, f0[f]));
          gn = cadd(gn, mult_apply(code, an, bn, sxn, sy, fn[f]));
        }
      }
      g[q] = cconj(make_float2(g0.x - gn.y, g0.y + gn.x));
    }
  }
}

// Multiply phase through LDS for the first `ncols` columns of the tile
// (including the packed DC / Nyquist column, whose two real columns are
// separated with the mirror element ny - ky): r holds the forward spectra, o
// receives the conjugated products.  Loads its multiplier values itself.
template <int CM>
__device__ __forceinline__ void col_mult_lds(const Medium& M, int tile, int mcode, int ls, int ncols,
                                             const float2* r, float2* o) {
  constexpr int nin = kColIn[CM], nout = kColOut[CM];
  const int ny = M.ny, nxh = M.nxh, ct = M.ct, c0 = tile * ct, B = blockDim.x;
  int xcode = 0, ycode = 0;
  bool frac = false, labs = false;
  for (int e = 0; e < 4; ++e) {
    const int c = (mcode >> (4 * e)) & 15;
    if (c == MC_DXP || c == MC_DXM) xcode = c;
    if (c == MC_DYP || c == MC_DYM) ycode = c;
    if (c == MC_LDIS) frac = true;
    if (c == MC_LABS) { frac = true; labs = true; }
  }
  const float* tabA = frac ? M.ldis : M.kap;
  const float2* symx = xcode == MC_DXP ? M.dxp : M.dxm;
  const float2* symy = ycode == MC_DYP ? M.dyp : M.dym;
  const float rny = 1.0f / static_cast<float>(ny);
  for (int it = threadIdx.x; it < ncols * ny; it += B) {
    const int c = ncols == 1 ? 0 : fdiv(it, ny, rny), ky = it - c * ny, kx = c0 + c;
    const unsigned t = mul24(kx, ny) + ky, tn = mul24(nxh, ny) + ky;   // tables are [kx][ky]
    const float a = tabA[t], b = labs ? M.labs[t] : 0.f;
    const float2 sx = xcode ? symx[kx] : make_float2(0.f, 0.f), sy = ycode ? symy[ky] : make_float2(0.f, 0.f);
    if (kx == 0) {
      const float an = tabA[tn], bn = labs ? M.labs[tn] : 0.f;
      const float2 sxn = xcode ? symx[nxh] : make_float2(0.f, 0.f);
      const int km = ky ? ny - ky : 0;
      float2 z[2], zm[2], g[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        z[f] = f < nin ? r[mul24(f * ct + c, ls) + px(ky)] : make_float2(0.f, 0.f);
        zm[f] = f < nin ? cconj(r[mul24(f * ct + c, ls) + px(km)]) : make_float2(0.f, 0.f);
      }
      packed_products<CM>(mcode, a, b, an, bn, sx, sxn, sy, z, zm, g);
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < nout) o[mul24(q * ct + c, ls) + px(ky)] = g[q];
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (q < nout) {
          float2 acc = make_float2(0.f, 0.f);
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            const int code = (mcode >> (4 * (2 * q + f))) & 15;
            if (code && f < nin) acc = cadd(acc, mult_apply(code, a, b, sx, sy, r[mul24(f * ct + c, ls) + px(ky)]));
          }
          o[mul24(q * ct + c, ls) + px(ky)] = cconj(acc);
        }
      }
    }
  }
}

// The multiply phase of the packed column (column 0 of tile 0) in place: lines
// f ct hold the forward spectra, lines q ct receive the conjugated products.
// Every thread reads its rows and their mirrors before any is overwritten.
template <int CM>
__device__ __forceinline__ void col_mult_packed_ip(const Medium& M, int mcode, int ls, float2* a) {
  constexpr int nin = kColIn[CM], nout = kColOut[CM];
  const int ny = M.ny, nxh = M.nxh, ct = M.ct, B = blockDim.x, tid = threadIdx.x;
  int xcode = 0, ycode = 0;
  bool frac = false, labs = false;
  for (int e = 0; e < 4; ++e) {
    const int c = (mcode >> (4 * e)) & 15;
    if (c == MC_DXP || c == MC_DXM) xcode = c;
    if (c == MC_DYP || c == MC_DYM) ycode = c;
    if (c == MC_LDIS) frac = true;
    if (c == MC_LABS) { frac = true; labs = true; }
  }
  const float* tabA = frac ? M.ldis : M.kap;
  const float2* symx = xcode == MC_DXP ? M.dxp : M.dxm;
  const float2* symy = ycode == MC_DYP ? M.dyp : M.dym;
  float2 z[kColPer][2], zm[kColPer][2];  // ny <= kColPer * B
#pragma unroll
  for (int k = 0; k < kColPer; ++k) {
    const int ky = tid + k * B;
    if (ky < ny) {
      const int km = ky ? ny - ky : 0;
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        z[k][f] = f < nin ? a[mul24(f * ct, ls) + px(ky)] : make_float2(0.f, 0.f);
        zm[k][f] = f < nin ? cconj(a[mul24(f * ct, ls) + px(km)]) : make_float2(0.f, 0.f);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kColPer; ++k) {
    const int ky = tid + k * B;
    if (ky < ny) {
      const unsigned tn = mul24(nxh, ny) + ky;   // tables are [kx][ky]; kx = 0 here
      const float va = tabA[ky], vb = labs ? M.labs[ky] : 0.f;
      const float an = tabA[tn], bn = labs ? M.labs[tn] : 0.f;
      const float2 sx = xcode ? symx[0] : make_float2(0.f, 0.f), sxn = xcode ? symx[nxh] : make_float2(0.f, 0.f);
      const float2 sy = ycode ? symy[ky] : make_float2(0.f, 0.f);
      float2 g[2];
      packed_products<CM>(mcode, va, vb, an, bn, sx, sxn, sy, z[k], zm[k], g);
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (q < nout) a[mul24(q * ct, ls) + px(ky)] = g[q];
    }
  }
}

// One Stockham stage in place on `nlines` lines a + l lstep (at most two
// lines of N <= kColPer B points): all butterflies are read and transformed
// in registers, then the block synchronises and writes them back.
template <int R, int NS, int NB, int OFF>
__device__ __forceinline__ void stage_ip(float2* a, int nlines, int lstep, const float2* tw) {
  constexpr int MB = (2 * kColPer + R - 1) / R;
  const unsigned total = unsigned(nlines) * NB;
  float2 v[MB][R];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const unsigned line = it / NB, j = it % NB;
      stage_load<R, NB>(v[i], a + line * lstep, j);
      stage_regs<R, NS, OFF, NB>(v[i], j, tw);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const unsigned it = threadIdx.x + i * blockDim.x;
    if (it < total) {
      const unsigned line = it / NB, j = it % NB;
      stage_store<R, NS, NB>(v[i], a + line * lstep, j);
    }
  }
}

// Column pass for line lengths N with a compile-time plan.  The
// forward transform's first stage is computed straight from the global loads
// and the inverse transform (the same plan in reverse order, so that its
// first stage takes the butterfly outputs one thread already holds) writes
// its last stage straight to global memory; in between, the forward
// transform's last stage, the multipliers and the inverse transform's first
// stage stay in registers.  The tile with the packed DC / Nyquist column
// (tile 0) takes its multiply phase through LDS.
// IP: the FFT stages run in place in one LDS line buffer (each exchange
// stage gathers its butterflies into registers, synchronises, scatters), which
// halves the block's LDS and lets more blocks share a CU.
template <int CM, int N, bool TG, bool IP = false>
__device__ __forceinline__ void col_fused(const Medium& M, const Work& W, int tile, int mcode, float2* lds) {
  constexpr int nin = kColIn[CM], nout = kColOut[CM];
  constexpr int NST = plan_nst(N), LS = col_lstride(N);
  constexpr int R1 = radix_of<N, false>(0), NB1 = N / R1;        // first forward = last inverse stage
  constexpr int RS = radix_of<N, false>(NST - 1), NBS = N / RS;  // last forward = first inverse stage
  static_assert(RS == radix_of<N, true>(0) && R1 == radix_of<N, true>(NST - 1), "plan reversal");
  constexpr int OFFS = NBS - R1;  // twiddles of the last forward stage (Ns = NBS)
  constexpr int OFFL = NB1 - RS;  // twiddles of the last inverse stage (Ns = NB1)
  constexpr int kQ = (nin * kColPer + R1 - 1) / R1;  // first-stage butterflies per thread (bound)
  constexpr int kP = (kColPer + RS - 1) / RS;         // middle butterflies per thread (bound)
  const int nxh = M.nxh, ct = M.ct, c0 = tile * ct, B = blockDim.x, lct = M.lct, lsrt = M.lsrt;
  const int tid = threadIdx.x;
  float2* bufA = lds;
  float2* bufB = IP ? lds : lds + 2 * ct * LS;
  float2* const twl = lds + (IP ? 2 : 4) * ct * LS;  // LDS copies: forward-plan twiddles, then reversed-plan ones
  const float2* const tw = TG ? static_cast<const float2*>(M.twy) : twl;
  const float2* const twr = TG ? static_cast<const float2*>(M.twyr) : twl + N;
  int xcode = 0, ycode = 0;
  bool frac = false, labs = false;
  for (int e = 0; e < 4; ++e) {
    const int c = (mcode >> (4 * e)) & 15;
    if (c == MC_DXP || c == MC_DXM) xcode = c;
    if (c == MC_DYP || c == MC_DYM) ycode = c;
    if (c == MC_LDIS) frac = true;
    if (c == MC_LABS) { frac = true; labs = true; }
  }
  const float* tabA = frac ? M.ldis : M.kap;
  const float2* symx = xcode == MC_DXP ? M.dxp : M.dxm;
  const float2* symy = ycode == MC_DYP ? M.dyp : M.dym;
  // element ky of column c of the tile: (ky / srt) rowstep + tbase + (ky mod srt) ct + c;
  // inputs r and r + 1 of a first-stage butterfly are step1 apart where srt
  // divides NB1: always at powers of two of 128 and more (a row tile of such a
  // grid has at most ny / 8 rows), else tested (block-uniform)
  const unsigned rowstep = unsigned(nxh) * M.srt, tbase = unsigned(tile) * (M.srt * ct);
  const unsigned step1 = mul24(NB1 >> lsrt, rowstep);
  auto elem = [&](unsigned j, unsigned c) { return mul24(j >> lsrt, rowstep) + tbase + ((j & (M.srt - 1)) << lct) + c; };
  constexpr bool kStepped = N >= 128 && (N & (N - 1)) == 0;
  const bool stepped = kStepped || (NB1 & (M.srt - 1)) == 0;

  // ---- load phase: first-stage inputs, both twiddle tables, middle multipliers
  const unsigned nq = unsigned(nin * ct) * NB1;
  float2 v1[kQ][R1];
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    if (wave_base() + i * B < nq) {
      const unsigned q = min(unsigned(tid + i * B), nq - 1);
      const unsigned l = q / NB1, j = q % NB1, f = l >> lct, c = l & (ct - 1);
      const float2* src = f ? W.s1 : W.s0;
      if (stepped) {
        src += elem(j, c);
#pragma unroll
        for (int r = 0; r < R1; ++r) v1[i][r] = src[r * step1];
      } else {
#pragma unroll
        for (int r = 0; r < R1; ++r) v1[i][r] = src[elem(j + r * NB1, c)];
      }
    }
  }
  TwRegsK<kColPer> TW, TWR;  // N <= kColPer * B (ct >= 1)
  if constexpr (!TG) {
    fetch_tw(TW, M.twy, N);
    fetch_tw(TWR, M.twyr, N);
  }
  const unsigned np = unsigned(ct) * NBS;
  const unsigned tstep = unsigned(NBS);   // tables are [kx][ky]: a column's entries are contiguous
  float ma[kP][RS], mb[kP][RS];
  float2 msy[kP][RS], msx[kP];
#pragma unroll
  for (int i = 0; i < kP; ++i) {
    if (wave_base() + i * B < np) {
      const unsigned pp = min(unsigned(tid + i * B), np - 1);
      const unsigned c = pp / NBS, j = pp % NBS, kx = c0 + c;
      const unsigned t0 = mul24(kx, N) + j;
      msx[i] = xcode ? symx[kx] : make_float2(0.f, 0.f);
#pragma unroll
      for (int r = 0; r < RS; ++r) {
        ma[i][r] = tabA[t0 + r * tstep];
        mb[i][r] = labs ? M.labs[t0 + r * tstep] : 0.f;
        msy[i][r] = ycode ? symy[j + r * NBS] : make_float2(0.f, 0.f);
      }
    }
  }
  // ---- forward first stage from registers
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const unsigned q = tid + i * B;
    if (q < nq) {
      const unsigned l = q / NB1, j = q % NB1;
      stage_regs<R1, 1, 0, NB1>(v1[i], j, tw);
      stage_store<R1, 1, NB1>(v1[i], bufA + l * LS, j);
    }
  }
  if constexpr (!TG) {
    put_tw(TW, twl, N);
    put_tw(TWR, twl + N, N);
  }
  __syncthreads();
  // ---- forward stages 2 .. NST-1
  float2* r;
  if constexpr (IP) r = fft_range_ip<N, LS, 1, NST - 1, R1>(bufA, nin * ct, tw);
  else r = fft_stages<N, false, LS, 1, NST - 1, R1>(bufA, bufB, nin * ct, tw);
  float2* o = IP ? r : other(r, bufA, bufB);
  // column 0 of tile 0 holds the packed DC / Nyquist column: its last forward
  // stage goes to LDS (into its own lines of o) for the mirror-element
  // multiply; every other column stays in registers.  A column takes the
  // same path whatever the tile shape, so results do not depend on it.
  const bool packed = c0 == 0;
  if (packed) {
    if constexpr (IP) {
      stage_ip<RS, NBS, NBS, OFFS>(r, nin, ct * LS, tw);  // lines f ct; the loop below reads other lines
    } else {
      for (unsigned it = tid; it < unsigned(nin) * NBS; it += B) {
        const unsigned f = it / NBS, j = it % NBS;
        stockham_c<RS, NBS, NBS, OFFS>(r + f * ct * LS, o + f * ct * LS, j, tw);
      }
    }
  }
  {
    // last forward stage, multipliers, first inverse stage: registers only
    float2 z[kP][nin][RS];
#pragma unroll
    for (int i = 0; i < kP; ++i) {
      const unsigned pp = tid + i * B;
      if (pp < np && !(packed && pp < NBS)) {
        const unsigned c = pp / NBS, j = pp % NBS;
#pragma unroll
        for (int f = 0; f < nin; ++f) {
          stage_load<RS, NBS>(z[i][f], r + (f * ct + c) * LS, j);
          stage_regs<RS, NBS, OFFS, NBS>(z[i][f], j, tw);
        }
      }
    }
    if constexpr (IP) __syncthreads();  // the stores below overwrite lines just read
#pragma unroll
    for (int i = 0; i < kP; ++i) {
      const unsigned pp = tid + i * B;
      if (pp < np && !(packed && pp < NBS)) {
        const unsigned c = pp / NBS, j = pp % NBS;
#pragma unroll
        for (int q = 0; q < nout; ++q) {
          float2 w[RS];
#pragma unroll
          for (int rr = 0; rr < RS; ++rr) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int f = 0; f < nin; ++f) {
              const int code = (mcode >> (4 * (2 * q + f))) & 15;
              if (code) acc = cadd(acc, mult_apply(code, ma[i][rr], mb[i][rr], msx[i], msy[i][rr], z[i][f][rr]));
            }
            w[rr] = cconj(acc);
          }
          stage_regs<RS, 1, 0, NBS>(w, j, twr);
          stage_store<RS, 1, NBS>(w, o + (q * ct + c) * LS, j);
        }
      }
    }
    __syncthreads();
  }
  if (packed) {
    if constexpr (IP) {
      // column 0 lines, in place: products (q ct), then the first inverse stage
      col_mult_packed_ip<CM>(M, mcode, LS, o);
      __syncthreads();
      stage_ip<RS, 1, NBS, 1 - RS>(o, nout, ct * LS, twr);
    } else {
      // column 0 lines: o (f ct) -> products r (q ct) -> first inverse stage o (q ct)
      col_mult_lds<CM>(M, tile, mcode, LS, 1, o, r);
      __syncthreads();
      for (unsigned it = tid; it < unsigned(nout) * NBS; it += B) {
        const unsigned q = it / NBS, j = it % NBS;
        stockham_c<RS, 1, NBS, 1 - RS>(r + q * ct * LS, o + q * ct * LS, j, twr);
      }
    }
    __syncthreads();
  }
  // ---- inverse stages 2 .. NST-1, then the last one straight to global memory
  float2* r2;
  if constexpr (IP) r2 = fft_range_ip<N, LS, 1, NST - 1, RS, true>(o, nout * ct, twr);
  else r2 = fft_stages<N, true, LS, 1, NST - 1, RS>(o, other(o, bufA, bufB), nout * ct, twr);
  const unsigned nq2 = unsigned(nout * ct) * NB1;
  for (unsigned q = tid; q < nq2; q += B) {
    const unsigned l = q / NB1, j = q % NB1, f = l >> lct, c = l & (ct - 1);
    float2 v[R1];
    stage_load<R1, NB1>(v, r2 + l * LS, j);
    stage_regs<R1, NB1, OFFL, NB1>(v, j, twr);
    float2* dst = f ? W.s1 : W.s0;
    if (stepped) {
      dst += elem(j, c);
#pragma unroll
      for (int rr = 0; rr < R1; ++rr) st_spec<TG>(dst + rr * step1, cconj(v[rr]));
    } else {
#pragma unroll
      for (int rr = 0; rr < R1; ++rr) st_spec<TG>(dst + elem(j + rr * NB1, c), cconj(v[rr]));
    }
  }
}

template <bool U, int CM, int NF, bool TG = false>
__global__ void __launch_bounds__(kMaxThreads)
col_kernel(const Launch L, int ntile, int chunk, int mcode_arg, int n) {
  const int mcode = CM == CM_APPLY ? mcode_arg : kColCode[CM];
  extern __shared__ float2 lds[];
  if constexpr (U) col_args_batch<CM>(L, ntile, chunk, n);
  else launch_args_batch(L, ntile, chunk, n, mcode_arg);
  int item, tile;
  if (!locate<U>(L, ntile, chunk, item, tile)) return;
  const MediumOf<U> M = medium_of<U>(L, item);
  const Work W = U ? shift_work(L.w0, item * L.wstride) : table_work(L, item);
  if constexpr (!U) col_fields_batch<CM>(M, W);
  if (n > M.nt - 2) return;  // this problem has finished (uneven batches)
  // Lengths with a compile-time plan take the fused pass, in their own
  // instance or, where a table launch holds several lengths, in this one; the
  // generic pass serves the short lengths 8 to 24.
  if constexpr (NF > 0) {
    col_fused<CM, NF, TG, !TG>(M, W, tile, mcode, lds);  // in place unless twiddles are read from global memory
  } else {
#define QPAT_COL_CASE(N)                        \
  case N:                                       \
    col_fused<CM, N, TG>(M, W, tile, mcode, lds); \
    return;
    if constexpr (!U) {
      switch (M.ny) {
        QPAT_FOR_LENGTHS(QPAT_COL_CASE)
        default: break;
      }
    }
#undef QPAT_COL_CASE
    col_generic<CM>(M, W, tile, mcode, lds);
  }
}


}  // namespace qpat

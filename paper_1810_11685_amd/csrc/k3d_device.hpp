// Device helpers shared by the two forms of the 3-D passes (k3d.hip: Stockham
// FFTs in LDS; k3d_dense.hip: DFTs as matrix products).
#pragma once

#include "k3d_internal.hpp"

namespace qpat3 {

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// floor(a / d) for 0 <= a < 2^21, d >= 1, from rd = 1/d: (a + 1/2) / d lies at
// least 1/(2d) from an integer and the float product errs by less than that.
__device__ __forceinline__ int udiv(int a, float rd) { return int((float(a) + 0.5f) * rd); }
__device__ __forceinline__ float rcp(int d) { return 1.0f / float(d); }

// ---------------------------------------------------------------- block -> (item, tile)
// Consecutive tiles of one item go to one XCD (work-groups are dispatched to
// the XCDs round-robin).
__device__ __forceinline__ bool locate(int nitems, int ntile, int chunk, int& item, int& tile) {
  const int b = blockIdx.x;
  const int i = (b & (kXcds - 1)) * chunk + (b / kXcds);
  if (i >= nitems * ntile) return false;
  item = i / ntile;
  tile = i - item * ntile;
  return true;
}

__device__ __forceinline__ Work3 shift(const Work3& w, long long off) {
  Work3 r;
  r.f = reinterpret_cast<float*>(reinterpret_cast<char*>(w.f) + off);
  r.s = reinterpret_cast<float2*>(reinterpret_cast<char*>(w.s) + off);
  r.part = reinterpret_cast<float*>(reinterpret_cast<char*>(w.part) + off);
  return r;
}

__device__ __forceinline__ size_t spec_index(const Medium3& M, int f, int c, int l) {
  return size_t(f) * M.ctiles * M.ct * M.nlines + size_t(c / M.ct) * (M.nlines * M.ct) + size_t(l) * M.ct +
         (c % M.ct);
}

// ---------------------------------------------------------------- passes
// incoming and outgoing spectra of a row pass at iterate n
template <int MODE>
__device__ __forceinline__ void row_counts(const Medium3& M, int n, int& nin, int& nout) {
  const bool first = (n == M.nt - 2);
  switch (MODE) {
    case R3_F1: nin = 3; nout = 3; break;
    case R3_F2: nin = n == -1 ? 0 : 3; nout = 2; break;
    case R3_F2L: nin = n == -1 ? 0 : 3; nout = 1; break;
    case R3_F3: nin = 2; nout = 1; break;
    case R3_A1: nin = first ? 0 : 1; nout = 2; break;
    case R3_A1L: nin = first ? 0 : 1; nout = n == -1 ? 0 : 3; break;
    case R3_A2: nin = 2; nout = n == -1 ? 0 : 3; break;
    case R3_A3: nin = 3; nout = 3; break;
    case R3_FWD1: nin = 0; nout = 1; break;
    default: nin = 1; nout = 0; break;  // R3_INV1
  }
}

// The scalar cache is cold when a kernel starts, so every kernel-argument
// load is a memory round trip, and the compiler issues each where its value is
// first needed: behind the prologue's early-exit branch and the twiddle
// staging loops.  These empty asm statements take the fields the prologue and
// the load phase read (and the block size, an implicit argument) as SGPR
// operands, so their loads issue as one batch at the top of the kernel.
__device__ __forceinline__ void args3_batch(const Launch3& L, int ntile, int chunk, int n) {
  const Medium3& m = L.m;
  asm volatile("" ::"s"(ntile), "s"(chunk), "s"(n), "s"(blockDim.x), "s"(L.nitems), "s"(L.wstride), "s"(L.io),
               "s"(L.w0.f), "s"(L.w0.s), "s"(L.w0.part), "s"(m.nx), "s"(m.ny), "s"(m.nz), "s"(m.nxh1),
               "s"(m.nlines), "s"(m.nt), "s"(m.rt), "s"(m.ct), "s"(m.ctiles));
}

template <int MODE>
__host__ __device__ __forceinline__ int plane_code(int f, int code) {
  switch (MODE) {
    case P3_GRADP1:
    case P3_GRADP2: return f == 0 ? OP_DXP : f == 1 ? OP_DYP : OP_DZP;
    case P3_GRADM2: return f == 0 ? OP_DXM : f == 1 ? OP_DYM : OP_DZM;
    case P3_FRAC: return f == 0 ? OP_LDIS : OP_LABS;
    default: return code;
  }
}

}  // namespace qpat3

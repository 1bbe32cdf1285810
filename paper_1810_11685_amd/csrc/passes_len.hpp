// Launches of the pass kernels of one compile-time line length N.  The device
// code of a length is instanced in its own translation unit (passes<N>.hip, one
// explicit instantiation each of the templates below), so that the lengths
// compile side by side and a process loads only the code objects of the
// lengths it uses.
#pragma once

#include "qpat_internal.hpp"

namespace qpat {

// How a launch finds its items, and where its FFT twiddles are.
enum LaunchKind : int {
  LK_UNIFORM = 0,     // uniform launch, twiddles staged in LDS
  LK_UNIFORM_TG = 1,  // uniform launch, twiddles read from global memory
  LK_TABLE = 2        // table launch whose items share the length
};

template <int N>
hipError_t launch_row_len(int mode, LaunchKind kind, const Launch& L, int ntile, int chunk, int nblocks, int threads,
                          size_t lds, int n, int flags, hipStream_t st);
template <int N>
hipError_t launch_col_len(int cm, LaunchKind kind, int mcode, const Launch& L, int ntile, int chunk, int nblocks,
                          int threads, size_t lds, int n, hipStream_t st);
// Let the row (col false) or column kernels of this length use up to `bytes`
// of dynamic LDS.
template <int N>
hipError_t allow_lds_len(bool col, size_t bytes);
// Whether the RM_FZ instances of this length exist for launches reading
// global twiddles (tg) or not.
template <int N>
bool row_fused_len(bool tg);

}  // namespace qpat

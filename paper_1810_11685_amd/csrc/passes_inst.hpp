// Definitions of passes_len.hpp for the length QPAT_LEN (included once by each
// passes<length>.hip, which defines it).
#include "passes.hpp"
#include "passes_len.hpp"

namespace qpat {

#define QPAT_FOR_ROW_MODES(X)                                                                            \
  X(RM_F1) X(RM_F2) X(RM_F2L) X(RM_F3) X(RM_A1) X(RM_A1L) X(RM_A2) X(RM_A3) X(RM_FWD1) X(RM_INV1)        \
  X(RM_F2L | RM_X) X(RM_F3 | RM_X) X(RM_A1 | RM_X) X(RM_A1L | RM_X)
#define QPAT_FOR_FUSED_MODES(X) X(RM_F2 | RM_FZ) X(RM_A2 | RM_FZ)
#define QPAT_FOR_COL_MODES(X) X(CM_GRADP1) X(CM_GRADM2) X(CM_FRAC) X(CM_GRADP2) X(CM_DIVM) X(CM_APPLY)

template <typename K>
static hipError_t allow_fn(K* k, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                             int(bytes));
}

// Whether the RM_FZ instances exist, by where the twiddles are: with radix-4 ends
// the fused update is only built on LDS twiddles.
template <int N>
constexpr bool row_fused(bool tg) {
  return row_fusable<N>() && (plan_radix(N, 0) > 4 || !tg);
}
template <int N>
bool row_fused_len(bool tg) {
  return row_fused<N>(tg);
}

template <int N>
hipError_t launch_row_len(int mode, LaunchKind kind, const Launch& L, int ntile, int chunk, int nblocks, int threads,
                          size_t lds, int n, int flags, hipStream_t st) {
  const dim3 g(nblocks), t(threads);
#define QPAT_MODE(m)                                                                                              \
  case m:                                                                                                         \
    if (kind == LK_TABLE)                                                                                         \
      hipLaunchKernelGGL((row_kernel<m, false, N>), g, t, lds, st, L, ntile, chunk, n, flags);                    \
    else if (kind == LK_UNIFORM)                                                                                  \
      hipLaunchKernelGGL((row_kernel<m, true, N>), g, t, lds, st, L, ntile, chunk, n, flags);                     \
    else if constexpr (((m) & RM_FZ) == 0 || row_fused<N>(true))                                                  \
      hipLaunchKernelGGL((row_kernel<m, true, N, true>), g, t, lds, st, L, ntile, chunk, n, flags);               \
    else                                                                                                          \
      return hipErrorInvalidValue;                                                                                \
    break;
  if constexpr (row_fusable<N>()) {
    if (mode & RM_FZ) {
      switch (mode) {
        QPAT_FOR_FUSED_MODES(QPAT_MODE)
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
  }
  switch (mode) {
    QPAT_FOR_ROW_MODES(QPAT_MODE)
    default: return hipErrorInvalidValue;
  }
#undef QPAT_MODE
  return hipGetLastError();
}

template <int N>
hipError_t launch_col_len(int cm, LaunchKind kind, int mcode, const Launch& L, int ntile, int chunk, int nblocks,
                          int threads, size_t lds, int n, hipStream_t st) {
  const dim3 g(nblocks), t(threads);
#define QPAT_MODE(c)                                                                                    \
  case c:                                                                                               \
    if (kind == LK_TABLE)                                                                               \
      hipLaunchKernelGGL((col_kernel<false, c, N>), g, t, lds, st, L, ntile, chunk, mcode, n);          \
    else if (kind == LK_UNIFORM)                                                                        \
      hipLaunchKernelGGL((col_kernel<true, c, N>), g, t, lds, st, L, ntile, chunk, mcode, n);           \
    else                                                                                                \
      hipLaunchKernelGGL((col_kernel<true, c, N, true>), g, t, lds, st, L, ntile, chunk, mcode, n);     \
    break;
  switch (cm) {
    QPAT_FOR_COL_MODES(QPAT_MODE)
    default: return hipErrorInvalidValue;
  }
#undef QPAT_MODE
  return hipGetLastError();
}

template <int N>
hipError_t allow_lds_len(bool col, size_t bytes) {
  hipError_t e = hipSuccess;
  if (col) {
#define QPAT_MODE(c)                                                                \
  if (e == hipSuccess) e = allow_fn(&col_kernel<true, c, N>, bytes);              \
  if (e == hipSuccess) e = allow_fn(&col_kernel<true, c, N, true>, bytes);        \
  if (e == hipSuccess) e = allow_fn(&col_kernel<false, c, N>, bytes);
    QPAT_FOR_COL_MODES(QPAT_MODE)
#undef QPAT_MODE
    return e;
  }
#define QPAT_MODE(m)                                                     \
  if (e == hipSuccess) e = allow_fn(&row_kernel<m, true, N>, bytes);   \
  if (e == hipSuccess) e = allow_fn(&row_kernel<m, false, N>, bytes);
#define QPAT_MODE_TG(m) \
  if (e == hipSuccess) e = allow_fn(&row_kernel<m, true, N, true>, bytes);
  QPAT_FOR_ROW_MODES(QPAT_MODE)
  QPAT_FOR_ROW_MODES(QPAT_MODE_TG)
  if constexpr (row_fusable<N>()) {
    QPAT_FOR_FUSED_MODES(QPAT_MODE)
  }
  if constexpr (row_fused<N>(true)) {
    QPAT_FOR_FUSED_MODES(QPAT_MODE_TG)
  }
#undef QPAT_MODE
#undef QPAT_MODE_TG
  return e;
}

template bool row_fused_len<QPAT_LEN>(bool);
template hipError_t launch_row_len<QPAT_LEN>(int, LaunchKind, const Launch&, int, int, int, int, size_t, int, int,
                                             hipStream_t);
template hipError_t launch_col_len<QPAT_LEN>(int, LaunchKind, int, const Launch&, int, int, int, int, size_t, int,
                                             hipStream_t);
template hipError_t allow_lds_len<QPAT_LEN>(bool, size_t);

}  // namespace qpat

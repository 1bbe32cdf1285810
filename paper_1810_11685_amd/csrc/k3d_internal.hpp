// Internal structures of the 3-D solver shared by its kernels (k3d.hip) and
// its host runtime (plan3d.cpp).  Not part of the public ABI.
//
// Layout: fields are [nz][ny][nx] (x fastest); "lines" are the nz*ny x-lines,
// line l = z*ny + y.  A field's half spectrum along x has nxh1 = nx/2 + 1
// columns and is stored in column tiles of ct columns: element (c, l) sits at
// (c / ct) * (nlines * ct) + l * ct + c % ct, so a y-z plane pass reads one
// contiguous chunk per tile and a row pass writes runs of ct elements.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qpat3 {

constexpr int kBlock = 256;          // threads per block of the helper kernels
constexpr int kRowMax = 512;         // most threads of a row block
constexpr int kPlaneMax = 1024;      // most threads of a plane block
constexpr int kMaxN = 128;           // longest axis
constexpr int kMaxStages = 8;        // FFT stages per axis
constexpr size_t kMaxLds = 163840;   // gfx950 LDS per work-group
constexpr int kXcds = 8;
constexpr int kCus = 256;            // MI355X compute units

// FFT plan of one axis: the radices in stage order (2, 3, 4, 5, 7, 8 have
// their own butterflies; any other prime runs as a direct DFT stage).
struct AxisPlan {
  int n, nst;
  int r[kMaxStages];
};

// One trilinear tap line of a sensor: the sensor's contribution from line
// `line` is wl * f[line][ixl] + wr * f[line][ixr]; slot 0..3 names which of
// the sensor's four lines it is.  Sorted by line.
struct Tap3 {
  int s, slot, line, ixl, ixr;
  float wl, wr;
  int pad;
};

// One grid node that receives the transposed measurement M^T r: the sum of
// w * r[s] over its entries [e0, e1) of the scatter list; sorted by (line, ix).
struct ScatterNode {
  int line, ix, e0, e1;
};
struct ScatterEntry {
  int s;
  float w;
};

struct Medium3 {
  int nx, ny, nz, nxh1, nlines, nt, ns, lossy;
  float dt;
  int rt, ct, ctiles;                 // lines per row tile, columns per plane tile, column tiles
  int rthr, pthr;                     // threads per row / plane block
  AxisPlan px, py, pz;
  const float *c2, *c2eta, *c2tau, *rho0;      // [N]
  const float *bx, *by, *bz;                   // dt / rho0 at the staggered positions [N]
  const float *avx, *arx, *avy, *ary, *avz, *arz;  // PML diagonals [nx] / [ny] / [nz]
  const float2 *dxp, *dxm, *dyp, *dym, *dzp, *dzm;  // 1-D symbols i k e^{+-i k d/2}: [nxh1] / [ny] / [nz]
  const float *kap, *ldis, *labs;              // [nxh1][nz][ny] (a column's lines contiguous), each / N
  const float2 *twx, *twy, *twz;               // e^{-2 pi i m / n}, m < n
  const float *dfx, *dfxi, *dfy, *dfz, *dfzc;         // DFT matrices of axes up to kDenseMax, see dense3
  const int* tap_off;                          // [nlines + 1]
  const Tap3* taps;
  const int* node_off;                         // [nlines + 1] into nodes
  const ScatterNode* nodes;
  const ScatterEntry* entries;
};

// Per-vector work buffers.
struct Work3 {
  float* f;       // 7 fields of N: forward v_x v_y v_z rho_x rho_y rho_z p; adjoint their adjoints, q
  float2* s;      // 4 half spectra, each ctiles * ct * nlines (3: the pressure of the forward)
  float* part;    // forward: sensor partials [nt][ns][4]
};

struct IO3 {
  const float* in;   // forward: p0 [N]; adjoint: residual [nt][ns]; apply: field
  float* out;        // forward: data [nt][ns]; adjoint: gradient [N]; apply: field
};

struct Launch3 {
  Medium3 m;
  Work3 w0;
  long long wstride;   // bytes between the work buffers of consecutive items
  int nitems;
  const IO3* io;
};

enum Row3 : int {
  R3_F1 = 0,    // forward: d_i^+ p -> velocity update -> spectra of v_x, v_y, v_z
  R3_F2 = 1,    // forward lossy: d_i^- v_i -> density update (+ source) -> spectra of S, u
  R3_F2L = 2,   // forward lossless: density update -> p, sensors, spectrum of p
  R3_F3 = 3,    // forward lossy: Y_dis S, Y_abs u -> p, sensors, spectrum of p
  R3_A1 = 4,    // adjoint lossy: p* + M^T r -> q, spectra of eta q, tau q
  R3_A1L = 5,   // adjoint lossless: p* + M^T r -> transposed density update -> spectra of e*_i
  R3_A2 = 6,    // adjoint lossy: Y terms -> transposed density update -> spectra of e*_i
  R3_A3 = 7,    // adjoint: transposed velocity update -> spectra of g*_i
  R3_FWD1 = 8,  // field -> spectrum 0
  R3_INV1 = 9   // spectrum 0 -> field
};

enum Plane3 : int {
  P3_GRADP1 = 0,  // 1 -> 3: d_x^+, d_y^+, d_z^+ of spectrum 3 into spectra 0..2
  P3_GRADM2 = 1,  // 3 -> 3: d_i^- of field i
  P3_FRAC = 2,    // 2 -> 2: Y_dis of field 0, Y_abs of field 1
  P3_GRADP2 = 3,  // 3 -> 3: d_i^+ of field i
  P3_APPLY = 5    // 1 -> 1: one operator (code in the launch)
};

enum OpCode3 : int { OP_DXP = 0, OP_DXM, OP_DYP, OP_DYM, OP_DZP, OP_DZM, OP_LDIS, OP_LABS };

// LDS bytes of a row block (two buffers of 3 x rt/2 lines + twiddles) and of
// a plane block (twiddles + two buffers of ct columns x nlines: a block
// transforms one field).
inline size_t row3_lds(int nx, int rt) { return (size_t(2) * 3 * (rt / 2) * nx + nx) * sizeof(float2); }
inline size_t plane3_lds(int ny, int nz, int ct) { return (size_t(2) * ct * ny * nz + ny + nz) * sizeof(float2); }

// ---- axes transformed as dense DFTs on the matrix cores (k3d_dense.hip)
// A length in [kDenseMin, kDenseMax] takes the symmetric DFT as matrix
// products: with e_r = x_r + x_{n-r} and o_r = x_r - x_{n-r} (1 <= r <= n/2),
// output q is x_0 + sum_r cos(2 pi q r / n) e_r -+ i sum_r sin(2 pi q r / n) o_r
// and output n - q takes the other sign; r = n/2 counts half (its mirror is
// itself).
constexpr int kDenseMin = 18, kDenseMax = 63;
constexpr int kDenseTiles = 2;   // 16-row tiles of outputs q
constexpr int kDenseSteps = 8;   // steps of four inputs r
inline __host__ __device__ bool dense3(int n) { return n >= kDenseMin && n <= kDenseMax; }
// Radix of the lengths that FFT kernels of their own transform in two equal
// stages, 7 x 7 and 8 x 8 (0: none).
inline __host__ __device__ constexpr int staged3(int n) { return n == 7 * 7 ? 7 : n == 8 * 8 ? 8 : 0; }
// Planes transformed as matrix products: both axes in the dense range, unless both
// have one such FFT: two radix-7 stages cost as much as the products at up to four
// vectors and less above (a J^T J v of 31 steps, FFT / products: 49^3 x 1 2759 / 2762
// us, x 4 4163 / 4112, x 8 5385 / 5981, x 16 8644 / 9630; 30 x 49 x 49 x 16 5363 / 6035).
// Radix 5 has too little in a stage: 25^3 x 1 1830 / 1753, x 16 2307 / 2259.  x-lines
// take the products at 49 too: a pass of one vector 6.8 us against 8.1, of 16 26.3
// against 28.4.
inline __host__ __device__ bool dense3_plane(int ny, int nz) {
  return dense3(ny) && dense3(nz) && !(ny == nz && staged3(ny));
}
// length classes of the kernels and their steps of four inputs
inline __host__ __device__ constexpr int dense3_class(int n) { return n <= 31 ? 0 : n <= 33 ? 1 : n <= 49 ? 2 : 3; }
inline __host__ __device__ constexpr int dense3_steps(int cls) { return cls <= 1 ? 4 : cls == 2 ? 6 : 8; }
// A matrix as the matrix instruction's first operand, [tile][step / 2][lane]
// [step % 2][cos, sin]: lane l of step s holds row q = 16 tile + l % 16 and
// input r = dense3_input(s, l / 16) + 1: the inputs of a step are neighbours and
// grow over the steps (what a sum loses depends on it, see chain_step in
// k3d_dense.hip).  The chained form takes its inputs from the accumulators of a preceding product (register i of row tile t
// in step 4 t + i) with r = dense3_input(4 t + i, l / 16), from r = 0, which counts
// half too; the rows of that preceding product are in the order that gives this.
inline __host__ __device__ constexpr int dense3_input(int s, int g) { return 4 * s + g; }
// The inputs of a y transform, whose lanes load them in pairs (r, r + 1 with
// r = 8 p + 2 g + 1 for steps 2 p and 2 p + 1) and trade one of each between the
// halves of the wave: the same inputs a step, in another order of the lanes.
inline __host__ __device__ constexpr int dense3_input_y(int s, int g) { return 4 * s + (g % 2 * 2 + g / 2); }
// Size in floats:
constexpr size_t kDenseTable = size_t(kDenseTiles) * kDenseSteps * 2 * 64;
static_assert(4 * kDenseTiles == kDenseSteps, "the chained form has four steps a tile");

hipError_t launch_row3_dense(int mode, const Launch3& L, int ntile, int chunk, int n, hipStream_t st);
hipError_t launch_plane3_dense(int mode, int code, const Launch3& L, int ntile, int chunk, int n, hipStream_t st);

hipError_t launch_row3(int mode, const Launch3& L, int ntile, int chunk, int n, hipStream_t st);
// blocks per column tile of a plane pass: one per field of the diagonal
// passes and one per output of the gradient (one-field blocks are small
// enough in LDS that several share a CU and hide each other's barrier waits)
__host__ __device__ constexpr int plane3_split(int mode) {
  return (mode == P3_GRADM2 || mode == P3_GRADP2 || mode == P3_GRADP1) ? 3 : mode == P3_FRAC ? 2 : 1;
}
hipError_t launch_plane3(int mode, int code, const Launch3& L, int ntile, int chunk, int n, hipStream_t st);
hipError_t launch_combine3(const Launch3& L, hipStream_t st);
hipError_t k3d_allow_lds(size_t bytes);

}  // namespace qpat3

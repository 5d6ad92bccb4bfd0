// Variable-coefficient system operator (host-callable launcher and its argument block).
#pragma once
#include "common.h"

namespace tbs {

constexpr int kVcMaxQ = 8;   // Gauss points per cell and axis: ceil((3n + 1) / 2) <= 8 for n <= 5
constexpr int kVcMaxB = 6;   // B-splines per cell and axis: n + 1 <= 6

constexpr int kVcHalfQ = 4;  // Gauss points up to the middle of a cell
constexpr int kVcHalfB = 3;  // B-spline pairs of a cell (t, n - t), or pairs and the middle one

// Basis tables of a unit cell in the arithmetic precision.  v, d: value and derivative of the t-th
// B-spline at the q-th Gauss point; pv, pdy, pdz: the same for the projections, times the point's weight
// (and h_y^-2, h_z^-2 for the derivatives).  The x-axis tables hold the parts even and odd under
// t <-> n - t of the points q up to the middle (the cell is symmetric: the point Q - 1 - q has the same
// parts, the odd one with the other sign); an even degree's middle B-spline is the even part's last entry.
template <typename T> struct VarcoefTab {
  T v[kVcMaxQ][kVcMaxB], d[kVcMaxQ][kVcMaxB], pv[kVcMaxQ][kVcMaxB], pdy[kVcMaxQ][kVcMaxB], pdz[kVcMaxQ][kVcMaxB];
  T xve[kVcHalfQ][kVcHalfB], xvo[kVcHalfQ][kVcHalfB], xde[kVcHalfQ][kVcHalfB], xdo[kVcHalfQ][kVcHalfB];
  T pve[kVcHalfQ][kVcHalfB], pvo[kVcHalfQ][kVcHalfB], pde[kVcHalfQ][kVcHalfB], pdo[kVcHalfQ][kVcHalfB];
};

// One launch of F(c)_l = sum_k sum_m c_k (m_m f^{klm} + d_m w^{klm}) (all arrays [z][y][x]).
struct VarcoefArgs {
  int nx, ny, nz, zc;
  int tiles_x, tiles_y, nchunks, nblocks;
  const void* c;
  const void* d;
  const void* m;
  void* y;
  // value and derivative of the t-th B-spline of a cell at its q-th Gauss point (unit cell), the
  // point's weight, and h_d^-2; the launcher forms the kernel's tables of them
  double bv[kVcMaxQ * kVcMaxB];
  double bd[kVcMaxQ * kVcMaxB];
  double w[kVcMaxQ];
  double ihx2, ihy2, ihz2;
};

constexpr int kVcWaves = 4;  // waves of a strip, one z-point of a cell each at a time
// Rows of outputs per strip (its y-extent): taller strips recompute fewer halo cells, but their LDS (the
// waves' rows and the output planes, 48 KB for both) must leave room for three workgroups per CU.
// Measured, cubic: FP32 400^3 14.8 ms with 16 rows, 17.2 with 8.
constexpr int vc_tile_y(int dt) { return dt == 0 ? 8 : 16; }
// z-chunk plan (plan_zc): workgroups per CU below which the latency of a wave's march counts.  Two, eight
// waves per CU.  Measured in FP32 with one / two / three: cubic 192^3 3.58 / 2.14 / 2.13 ms, 128x100x90
// 0.93 / 0.77 / 0.88, quartic 128^3 4.07 / 3.71 / 3.49, quintic 100^3 4.70 / 5.08 / 6.74.
constexpr double kVcLatencyLoad = 2.0;
// Output columns of one strip: the 64 lanes hold the strip's coefficient columns and an n-column halo.
constexpr int vc_tile_x(int n) { return 64 - 2 * n; }

// dt 0: FP64 arrays and arithmetic, 1: FP32.  bc: BC_PERIODIC or BC_DIRICHLET.
hipError_t launch_varcoef(const VarcoefArgs& a, int n, int bc, int dt, hipStream_t st);

}  // namespace tbs

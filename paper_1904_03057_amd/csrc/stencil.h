// Launchers of the stencil tile engine and the vector/reduction kernels (host-callable).
#pragma once
#include "common.h"

#ifndef STENCIL_APPLY_WX
#define STENCIL_APPLY_WX 1
#endif

#ifndef STENCIL_CG_TY
#define STENCIL_CG_TY 16
#endif
#ifndef STENCIL_CGF_TY
#define STENCIL_CGF_TY 48
#endif
#ifndef STENCIL_CG_PF
#define STENCIL_CG_PF 1
#endif
#ifndef STENCIL_RESID_TY
#define STENCIL_RESID_TY 16
#endif
#ifndef STENCIL_RESID_WY
#define STENCIL_RESID_WY 8
#endif
#ifndef STENCIL_F64_WY
#define STENCIL_F64_WY 8
#endif

namespace tbs {

constexpr int kLdsMax = 160 * 1024;  // LDS one workgroup may hold on gfx950

// LDS of the one-kernel CG iteration (degree n, tile height ty, 64 columns, es-byte compute type):
// staged plane (x halo of at most 8 columns a side: one 16-byte vector of bf16), the two x-pass
// planes, the p and r rings, the reduction slots of up to 16 waves, and the Robin corner tables and z-accumulators
// (one-element placeholders otherwise).  An upper bound of what the kernel declares (it asserts so).
constexpr int cgf_lds_bytes(int n, int ty, int bc, int es) {
  return es * ((ty + 2 * n) * (64 + 16) + 2 * (ty + 2 * n) * 64 + (2 * n + 3) * ty * 64) +
         8 * 4 * 16 +
         (bc == BC_ROBIN ? es * (4 * kRobinMaxZ * kRobinMaxZ + (2 * (n / 2) + 1) * ty * 64) : 2 * es);
}

// The one-kernel CG iteration's tile height: in FP32 the tallest of STENCIL_CGF_TY, 32 and 16 rows
// whose LDS fits one workgroup (row waves of four rows each: the registers per thread do not grow
// with the height, and a taller tile re-reads fewer halo rows of r, q and p); in FP64 16 rows, or 8
// where 16 do not fit (Robin quartic and quintic).
constexpr int cgf_tile_y(int n, int bc, int es) {
  return es == 4 ? (cgf_lds_bytes(n, STENCIL_CGF_TY, bc, 4) <= kLdsMax
                        ? STENCIL_CGF_TY
                        : (cgf_lds_bytes(n, 32, bc, 4) <= kLdsMax ? 32 : 16))
                 : (cgf_lds_bytes(n, 16, bc, 8) <= kLdsMax ? 16 : 8);
}

// Shapes of the one-kernel CG iteration.  Shape 0 is the tile above.  On smaller grids its few, large
// workgroups leave CUs idle, and where every workgroup has a CU to itself the time per plane is the
// instructions of one wave: shape 1 is 32 rows in FP32, and 8 in FP64 with one row per wave; shape 2 is 16
// rows of two per wave in FP32.  The plan takes the cheapest (stencil_plan_zc).  Measured, cubic
// periodic, us per iteration with shapes 0 / 1 / 2 in FP32: 32^3 25.5 / 22.7 / 19.5, 100^3 32.1 / 30.1 / 29.1,
// 192^3 58.5 / 55.3 / 60.7, 256^3 131.8 / 124.0 / 146.1; with 0 / 1 in FP64: 32^3 22.2 / 19.2, 64^3 24.8 / 22.9,
// 100^3 33.5 / 36.0.  Robin boxes and the bf16-stored direction have shape 0 only.
constexpr int kCgfShapes = 3;
// tile height of a shape, 0 if there is none
constexpr int cgf_shape_ty(int shape, int n, int bc, int es) {
  return shape == 0 ? cgf_tile_y(n, bc, es)
                    : (bc == BC_ROBIN ? 0
                                      : (es == 4 ? (shape == 2 ? 16 : (cgf_tile_y(n, bc, 4) > 32 ? 32 : 0))
                                                 : (shape == 1 ? 8 : 0)));
}
constexpr int cgf_shape_rows_per_wave(int shape, int es) {
  return es == 4 ? (shape == 2 ? 2 : 4) : (shape == 1 ? 1 : 2);
}
// A plane's time in a lone workgroup (us, cubic; between the value on an idle chip and on a busy one)
constexpr double cgf_plane_time(int shape, int es) {
  return es == 4 ? (shape == 0 ? 2.9 : (shape == 1 ? 2.25 : 1.65)) : (shape == 0 ? 2.3 : 1.65);
}

// Tile height per (mode, compute precision, degree, boundary): taller tiles re-read fewer halo
// rows.  The FP64 kernels take 16 rows in eight row waves of two rows (the FP64 ring and column
// windows of two rows leave room for more waves per SIMD than four rows in four waves).  shape: of
// the one-kernel CG iteration.
constexpr int stencil_tile_y(int mode, int compute_bytes, int n, int bc, int shape = 0) {
  return mode == M_CGF ? cgf_shape_ty(shape, n, bc, compute_bytes)
                       : (compute_bytes == 4 ? (mode == M_APPLY ? 32 : (mode == M_CG1 ? STENCIL_CG_TY : 16))
                                             : ((mode == M_RESID || mode == M_RHSRES) ? STENCIL_RESID_TY : 16));
}
// Row waves per workgroup: four for the FP32 kernels, except the one-kernel CG iteration; eight for the
// other FP64 kernels.
constexpr int stencil_tile_wy(int mode, int compute_bytes, int n, int bc, int shape = 0) {
  return mode == M_CGF ? stencil_tile_y(mode, compute_bytes, n, bc, shape) / cgf_shape_rows_per_wave(shape, compute_bytes)
                       : ((mode == M_RESID || mode == M_RHSRES) ? STENCIL_RESID_WY
                                                                   : (compute_bytes == 8 ? STENCIL_F64_WY : 4));
}
// Columns per lane of the x-pass.  Two: the LDS reads of a row drop from 2N + 1 values per output to
// N + 1 or N + 2 per two outputs (in pairs), which is what bounds the FP64 kernels of high degree and
// saves instruction slots in FP32: measured FP64 apply, quartic 385x259x201, 144 against 168 us, FP32 apply
// cubic 928^3 1.69 against 1.74 ms, FP64 CG iteration quadratic 400^3 762 against 833 us.  One where
// the pairs read no less (linear) or the copy rate already bounds the launch (FP64 quadratic apply 308
// against 294 us, residual 425 against 405 us at 400^3).
constexpr int stencil_x_cols(int mode, int compute_bytes, int n) {
  return n >= 3 || compute_bytes == 4 || (n == 2 && (mode == M_CG1 || mode == M_CGF)) ? 2 : 1;
}
// Waves per SIMD the register allocation must leave room for.  Robin kernels: two.  The linear FP64
// kernels of eight waves: six, three workgroups per CU; they need 74 to 82 registers and six waves
// have 80 (residual at 400^3: 280 against 394 us at 82 registers; right-hand side 214 against 274 us at 81).
constexpr int stencil_min_waves(int mode, int compute_bytes, int n, int bc) {
  return bc == BC_ROBIN ? 2 : (n == 1 && compute_bytes == 8 && (mode == M_APPLY || mode == M_RHS || mode == M_RESID) ? 6 : 1);
}

// Planes per z-chunk of a launch.  A workgroup marches zc + 2n planes; with W workgroups the busiest
// of the 256 CUs gets ceil(W / 256) of them, and a CU's time per plane grows with that number from
// the value at which it is busy (below it, the plane's latency counts).  The plan takes the chunk
// count with the smallest (zc + 2n) max(latency load, ceil(W / 256)): one chunk per plane on the
// smallest grids, all CUs evenly loaded on the middle ones, long chunks on the largest.  Above four
// workgroups per CU they no longer start and end together: W / 256 plus a share for the uneven end
// replaces the ceiling (which took four chunks for the FP32 apply at 928^3: 1.81 against 1.72 ms); 0.75,
// or 1.5 for the FP32 apply, which is bound by its arithmetic and not by the halo planes' traffic (with
// 1.5 for all, twelve chunks instead of eight, the FP32 CG step at 928^3 took 292 against 280 ms).
constexpr double stencil_latency_load(int mode, int compute_bytes) {
  return mode == M_CGF ? 1.0 : (compute_bytes == 4 ? 1.8 : ((mode == M_RESID || mode == M_RHSRES) ? 1.5 : 1.3));
}
int plan_zc(int64_t tiles, int64_t nz, int halo, int slots, int64_t most_blocks, double lat, double tail,
            double* cost = nullptr);
// Chunks of at least 4 (2n+1) planes for about 8192 workgroups: what a launch takes where the plan is not worth it.
int long_zc(int64_t nx, int64_t ny, int64_t nz, int n);
// The estimate is good to about 10 % only, and one latency load per kernel is a mean over degrees and grids: the
// light kernels (low degrees, FP32) hide more latency in more workgroups, and the plan, long chunks at just that
// load, lost to long_zc by more than 3 % on one launch in eight (FP64) to two in three (FP32 right-hand side: 512^3
// linear 281 against 218 us, 385x259x201 64 against 37; FP32 apply 16x2048x2048 linear 380 against 240; two-kernel
// FP32 CG there 929 against 651).  So the plan stands only where it is kPlanGain cheaper with this load too.  Of
// 488 launches (ten grids, degrees 1 to 5), 6 % are then more than 3 % behind long_zc (the worst 1.21) and 3 % more
// than 3 % behind the plan (1.12).
constexpr double kPlanGain = 0.95;
constexpr double clamp_load(double v, double lo, double hi) { return v < lo ? lo : (v > hi ? hi : v); }
constexpr double stencil_settled_load(int mode, int compute_bytes, int n, int bc) {
  const double heavy = 0.3 * (n + (bc == BC_ROBIN ? 2 : 0));  // more arithmetic per plane, less latency to hide
  if (compute_bytes == 8) return clamp_load((mode == M_CG1 ? 2.0 : 2.5) - heavy, 1.0, 2.0);
  return mode == M_APPLY ? clamp_load(3.25 - heavy, 1.75, 3.25) : (mode == M_CG1 ? 2.4 : 4.0 - 0.3 * n);
}
// The linear FP64 kernels are bound by memory traffic, of which a tile that overhangs the grid has less: their
// latency loads grow by this (fill: the share of the tiles inside the grid).  One-kernel CG iteration 16x2048x2048
// 1206 against 1565 us, 16x16x8192 47 against 55; FP64 apply 16x2048x2048 510 against 617.
constexpr double stencil_fill_factor(double root_fill, int compute_bytes, int n) {
  return compute_bytes == 8 && n == 1 && root_fill < 0.9 ? 0.9 / root_fill : 1.0;
}
// FP64 CG on a Robin box of degree 2 or more: its nearly empty corner functions take hundreds to thousands
// of iterations, and sums grouped in another way moved its solutions by up to 4e-8 of their RMS.  So its
// sums keep the grouping of long_zc.  Where the plan's own chunks are faster by more than kRobinDotsGain, the
// iteration runs with those and leaves the sums to a second launch that adds them in that grouping
// (cg_dots_kernel, which reads r, p and q again): cubic 121x104x90, 36 + 22 us per iteration against 105 with
// the long chunks.
constexpr double kRobinDotsGain = 1.7;
bool robin_dots_apart(int64_t nx, int64_t ny, int64_t nz, int n, int zc);
// zchunk > 0: the caller's own chunk length.  *shape (M_CGF): the shape the plan takes, the one with the
// smallest cost times its time per plane (0 with a caller's chunk length).
int stencil_plan_zc(int64_t nx, int64_t ny, int64_t nz, int mode, int compute_bytes, int n, int bc, int zchunk,
                    int* shape);

// One stencil launch of degree N for a (mode, input, compute, output) type combination and
// boundary condition BC; defined in stencil_kernel.h and instantiated per degree and boundary
// condition by stencil_inst.hip.
template <int N, int MODE, typename Tin, typename Tc, typename Tout, int BC>
hipError_t launch_bcx(const StencilArgs& a, bool vec, hipStream_t st);

template <int N, int BC>
hipError_t launch_rhsres_bc(const StencilArgs& a, bool vec, hipStream_t st);

template <int N, int MODE, typename Tin, typename Tc, typename Tout>
inline hipError_t launch_bc(const StencilArgs& a, int bc, bool vec, hipStream_t st) {
  if (bc == BC_PERIODIC) return launch_bcx<N, MODE, Tin, Tc, Tout, BC_PERIODIC>(a, vec, st);
  if (bc == BC_ROBIN) return launch_bcx<N, MODE, Tin, Tc, Tout, BC_ROBIN>(a, vec, st);
  return launch_bcx<N, MODE, Tin, Tc, Tout, BC_DIRICHLET>(a, vec, st);
}

// Number of workgroups (= partial sums written) of a stencil launch of this mode.
int stencil_blocks(const StencilArgs& a, int mode, int compute_bytes, int n, int bc);

// stencil.hip
hipError_t launch_apply(const StencilArgs& a, int n, int bc, int in_dt, int out_dt, hipStream_t st);
hipError_t launch_rhs(const StencilArgs& a, int n, int bc, int dt, hipStream_t st);
hipError_t launch_cg1(const StencilArgs& a, int n, int bc, int dt, hipStream_t st);
// CGF (one-kernel CG iteration): dt = 1 (all f32), 2 (f32 with p stored as bf16)
hipError_t launch_cgf(const StencilArgs& a, int n, int bc, int dt, hipStream_t st);
// the sums of a Robin FP64 CGF launch that was given no partial-sum arrays (in0 = r, in1 = p, in2 = q)
hipError_t launch_cg_dots(const StencilArgs& a, int n, hipStream_t st);
hipError_t launch_resid(const StencilArgs& a, int n, int bc, int r_dt, hipStream_t st);
// RHSRES: u (f64, in0) -> b = M u (f64, out1) and r = (b - A u) rscale (f32, out0), with the partial
// sums of r.r and (b rscale).(b rscale); periodic and Dirichlet only (hipErrorInvalidValue on Robin)
hipError_t launch_rhs_resid(const StencilArgs& a, int n, int bc, hipStream_t st);

// vector.hip
constexpr int kVecBlocks = 2048;   // grid of the elementwise kernels (= partial sums they write)
hipError_t launch_cg2(void* r, const void* q, int64_t n, int dt, double* part, const Scalars* s, hipStream_t st);
hipError_t launch_sub_norm(void* r, const void* b, const void* q, int64_t n, int dt, double* p0, double* p1,
                           hipStream_t st);
hipError_t launch_flush(void* x, const void* p0, const void* p1, int64_t n, int dt, const Scalars* s, hipStream_t st);
hipError_t launch_dot(const void* a, const void* b, int64_t n, int dt, double* part, hipStream_t st);
hipError_t launch_convert(const void* src, int sdt, void* dst, int ddt, int64_t n, hipStream_t st);
hipError_t launch_add_f32_to_f64(double* x, const float* d, int64_t n, hipStream_t st);
hipError_t launch_fill(void* x, int dt, int64_t n, hipStream_t st);  // zero fill
hipError_t launch_stream_copy(const void* src, void* dst, int64_t nbytes, hipStream_t st);
hipError_t launch_guess_combine(double* x, const double* u, const float* du, int64_t n, double scale,
                                hipStream_t st);  // x = u + scale du

// finalize kernels (single block, fixed-order reduction of partial sums)
enum FinOp { FIN_INIT = 0, FIN_ALPHA = 1, FIN_BETA = 2, FIN_DOT = 3, FIN_NORMS = 4, FIN_CLEAR_PENDING = 5,
             FIN_INIT_XZERO = 6 };  // FIN_INIT_XZERO: FIN_INIT for x = 0 left unwritten
// Reduces the per-block partial sums p0 (and p1 where the op uses it) in a fixed order and updates the
// CG scalars (a CGF launch does this itself).
hipError_t launch_finalize(int op, const double* p0, const double* p1, int count, Scalars* s, double rtol,
                           hipStream_t st);
// out[0] = sqrt(s->out), out[1] = sqrt(s->out2) (the norms of a FIN_NORMS reduction) in device memory
hipError_t launch_norms_out(const Scalars* s, double* out, hipStream_t st);

}  // namespace tbs

// Dispatch of the stencil launches: (mode, dtype) combinations, basis degree n and boundary -> the
// kernel instances of stencil_kernel.h that stencil_inst.hip compiles per degree and boundary.
#include <algorithm>
#include <cmath>

#include "cg_finish.h"
#include "common.h"
#include "stencil.h"

namespace tbs {

template <int MODE, typename Tin, typename Tc, typename Tout>
static hipError_t launch_n(const StencilArgs& a, int n, int bc, hipStream_t st) {
  // 16-byte vector staging needs rows made of whole vectors: Nx divisible by the vector width
  constexpr int ve = 16 / sizeof(Tin);
  const bool vec = (a.nx % ve) == 0;
  switch (n) {
    case 1: return launch_bc<1, MODE, Tin, Tc, Tout>(a, bc, vec, st);
    case 2: return launch_bc<2, MODE, Tin, Tc, Tout>(a, bc, vec, st);
    case 3: return launch_bc<3, MODE, Tin, Tc, Tout>(a, bc, vec, st);
    case 4: return launch_bc<4, MODE, Tin, Tc, Tout>(a, bc, vec, st);
    case 5: return launch_bc<5, MODE, Tin, Tc, Tout>(a, bc, vec, st);
  }
  return hipErrorInvalidValue;
}

int stencil_blocks(const StencilArgs& a, int mode, int compute_bytes, int n, int bc) {
  const int ty = stencil_tile_y(mode, compute_bytes, n, bc, a.shape);
  const int wx = (mode == M_APPLY && compute_bytes == 4) ? STENCIL_APPLY_WX : 1;
  return ((a.nx + 64 * wx - 1) / (64 * wx)) * ((a.ny + ty - 1) / ty) * a.nchunks;
}

static double chunk_cost(int64_t tiles, int64_t nz, int64_t zc, int halo, int slots, double lat, double tail) {
  const double load = (double)(tiles * ((nz + zc - 1) / zc)) / slots;
  return (double)(zc + halo) * std::max(lat, load <= 4.0 ? std::ceil(load) : load + tail);
}

// The planes per chunk with the smallest (zc + halo) max(lat, load), load the workgroups of the busiest of
// `slots` equal processors; at most most_blocks workgroups, or one chunk.
int plan_zc(int64_t tiles, int64_t nz, int halo, int slots, int64_t most_blocks, double lat, double tail,
            double* least) {
  const int64_t most = std::min<int64_t>(nz, std::max<int64_t>(1, most_blocks / tiles));
  int64_t best = nz;
  double cost = 0.0;
  for (int64_t want = 1; want <= most; ++want) {
    const int64_t zc = (nz + want - 1) / want;
    const double t = chunk_cost(tiles, nz, zc, halo, slots, lat, tail);
    if (want == 1 || t < cost) {
      cost = t;
      best = zc;
    }
  }
  if (least) *least = cost;
  return (int)best;
}

int long_zc(int64_t nx, int64_t ny, int64_t nz, int n) {
  const int64_t tiles = ((nx + 63) / 64) * ((ny + 15) / 16), least = std::max(16, 4 * (2 * n + 1));
  const int64_t chunks = std::max<int64_t>(1, std::min((8192 + tiles - 1) / tiles, nz / least));
  return (int)((nz + chunks - 1) / chunks);
}

bool robin_dots_apart(int64_t nx, int64_t ny, int64_t nz, int n, int zc) {
  const int ty = stencil_tile_y(M_CGF, 8, n, BC_ROBIN);
  const int64_t tiles = ((nx + 63) / 64) * ((ny + ty - 1) / ty);
  const double lat = stencil_latency_load(M_CGF, 8);
  return chunk_cost(tiles, nz, long_zc(nx, ny, nz, n), 2 * n, 256, lat, 0.75) >
         kRobinDotsGain * chunk_cost(tiles, nz, zc, 2 * n, 256, lat, 0.75);
}

int stencil_plan_zc(int64_t nx, int64_t ny, int64_t nz, int mode, int compute_bytes, int n, int bc, int zchunk,
                    int* shape) {
  if (shape) *shape = 0;
  if (zchunk > 0) return (int)std::min<int64_t>(zchunk, nz);
  const int wx = (mode == M_APPLY && compute_bytes == 4) ? STENCIL_APPLY_WX : 1;
  const int64_t tiles_x = (nx + 64 * wx - 1) / (64 * wx);
  if (compute_bytes == 8 && mode == M_CG1 && bc == BC_ROBIN && n >= 2) return long_zc(nx, ny, nz, n);
  int zc = 0;
  double least = 0.0;
  for (int sh = 0; sh < (mode == M_CGF && shape ? kCgfShapes : 1); ++sh) {
    const int ty = stencil_tile_y(mode, compute_bytes, n, bc, sh);
    if (ty == 0) continue;
    const int64_t tiles = tiles_x * ((ny + ty - 1) / ty);
    const double fill = stencil_fill_factor(std::sqrt((double)nx * ny / (64.0 * ty * tiles)), compute_bytes, n);
    const double lat = stencil_latency_load(mode, compute_bytes) * (mode == M_CGF ? fill : 1.0);
    double cost;
    int z = plan_zc(tiles, nz, 2 * n, 256, 16384, lat, mode == M_APPLY && compute_bytes == 4 ? 1.5 : 0.75, &cost);
    if (mode != M_CGF) {
      const int zl = long_zc(nx, ny, nz, n);
      const double load = stencil_settled_load(mode, compute_bytes, n, bc) * fill;
      if (chunk_cost(tiles, nz, z, 2 * n, 256, load, 0.75) > kPlanGain * chunk_cost(tiles, nz, zl, 2 * n, 256, load, 0.75))
        z = zl;
    }
    cost *= cgf_plane_time(sh, compute_bytes);
    if (zc == 0 || cost < least) {
      zc = z;
      least = cost;
      if (shape) *shape = sh;
    }
  }
  return zc;
}

// dtype codes: 0 = f64, 1 = f32, 2 = bf16
hipError_t launch_apply(const StencilArgs& a, int n, int bc, int in_dt, int out_dt, hipStream_t st) {
  if (in_dt == 0 && out_dt == 0) return launch_n<M_APPLY, double, double, double>(a, n, bc, st);
  if (in_dt == 1 && out_dt == 1) return launch_n<M_APPLY, float, float, float>(a, n, bc, st);
  if (in_dt == 2 && out_dt == 1) return launch_n<M_APPLY, uint16_t, float, float>(a, n, bc, st);
  if (in_dt == 1 && out_dt == 0) return launch_n<M_APPLY, float, double, double>(a, n, bc, st);
  if (in_dt == 2 && out_dt == 0) return launch_n<M_APPLY, uint16_t, double, double>(a, n, bc, st);
  return hipErrorInvalidValue;
}

hipError_t launch_rhs(const StencilArgs& a, int n, int bc, int dt, hipStream_t st) {
  if (dt == 0) return launch_n<M_RHS, double, double, double>(a, n, bc, st);
  if (dt == 1) return launch_n<M_RHS, float, float, float>(a, n, bc, st);
  return hipErrorInvalidValue;
}

// CG1: dt = 0 (all f64), 1 (all f32), 2 (f32 with p stored as bf16)
hipError_t launch_cg1(const StencilArgs& a, int n, int bc, int dt, hipStream_t st) {
  if (dt == 0) return launch_n<M_CG1, double, double, double>(a, n, bc, st);
  if (dt == 1) return launch_n<M_CG1, float, float, float>(a, n, bc, st);
  if (dt == 2) return launch_n<M_CG1, uint16_t, float, float>(a, n, bc, st);
  return hipErrorInvalidValue;
}

hipError_t launch_cgf(const StencilArgs& a, int n, int bc, int dt, hipStream_t st) {
  if (dt == 0) return launch_n<M_CGF, double, double, double>(a, n, bc, st);
  if (dt == 1) return launch_n<M_CGF, float, float, float>(a, n, bc, st);
  if (dt == 2) return launch_n<M_CGF, uint16_t, float, float>(a, n, bc, st);
  return hipErrorInvalidValue;
}

// The sums of a one-kernel FP64 CG iteration from the arrays it has written (in0 = r, in1 = p, in2 = q),
// with the additions of a launch of that kernel with this z-chunk, bit for bit: thread for thread the same
// points in the same order, then the same reduction.  kPlanes planes of loads are in flight at a
// time; a chunk's planes are one chain of additions per thread.
template <int TY, int WY, int VE>
__global__ __launch_bounds__(64 * WY) void cg_dots_kernel(StencilArgs a) {
  constexpr int NT = 64 * WY, RPW = TY / WY, kPlanes = 5;
  constexpr int CORE = TY * (64 / VE), NVC = CORE / NT;
  static_assert(CORE % NT == 0, "whole vectors per thread");
  __shared__ double red[4][WY];
  __shared__ bool last;
  if (a.scal->done) {
    if (a.status && blockIdx.x == 0 && threadIdx.x == 0) cg_publish(a.status, a.gen, a.scal);
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bid = xcd_remap(blockIdx.x, a.nblocks);
  int txi, tyi, czi;
  if (a.order == 0) {
    txi = bid % a.tiles_x;
    tyi = bid / a.tiles_x % a.tiles_y;
    czi = bid / a.tiles_x / a.tiles_y;
  } else {
    tyi = bid % a.tiles_y;
    txi = bid / a.tiles_y % a.tiles_x;
    czi = bid / a.tiles_y / a.tiles_x;
  }
  const int x0 = txi * 64, y0 = tyi * TY, z0 = czi * a.zc, z1 = min(z0 + a.zc, a.nz);
  const int64_t plane = (int64_t)a.nx * a.ny;
  const double* __restrict__ r = (const double*)a.in0;
  const double* __restrict__ p = (const double*)a.in1;
  const double* __restrict__ q = (const double*)a.in2;
  bool row_ok[RPW], core_ok[NVC];
  int row_off[RPW], core_off[NVC];  // 0 for points outside the grid, whose values are not used
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int gy = y0 + wave * RPW + i;
    row_ok[i] = x0 + lane < a.nx && gy < a.ny;
    row_off[i] = row_ok[i] ? gy * a.nx + x0 + lane : 0;
  }
#pragma unroll
  for (int v = 0; v < NVC; ++v) {
    const int idx = tid + NT * v, gx = x0 + idx % (64 / VE) * VE, gy = y0 + idx / (64 / VE);
    core_ok[v] = gx < a.nx && gy < a.ny;
    core_off[v] = core_ok[v] ? gy * a.nx + gx : 0;
  }
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
  for (int o0 = z0; o0 < z1; o0 += kPlanes) {
    double pv[kPlanes][RPW], qv[kPlanes][RPW], rv[kPlanes][RPW], cv[kPlanes][NVC][VE];
#pragma unroll
    for (int u = 0; u < kPlanes; ++u) {
      const int64_t base = (int64_t)min(o0 + u, z1 - 1) * plane;
#pragma unroll
      for (int i = 0; i < RPW; ++i) {
        pv[u][i] = p[base + row_off[i]];
        qv[u][i] = q[base + row_off[i]];
        rv[u][i] = r[base + row_off[i]];
      }
#pragma unroll
      for (int v = 0; v < NVC; ++v)
#pragma unroll
        for (int e = 0; e < VE; ++e) cv[u][v][e] = r[base + core_off[v] + e];
    }
#pragma unroll
    for (int u = 0; u < kPlanes; ++u) {
      if (o0 + u < z1) {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
          if (row_ok[i]) {
            s0 = fma(pv[u][i], qv[u][i], s0);
            s1 = fma(rv[u][i], qv[u][i], s1);
            s2 = fma(qv[u][i], qv[u][i], s2);
          }
#pragma unroll
        for (int v = 0; v < NVC; ++v)
          if (core_ok[v])
#pragma unroll
            for (int e = 0; e < VE; ++e) s3 = fma(cv[u][v][e], cv[u][v][e], s3);
      }
    }
  }
  cg_finish<WY>(a, s0, s1, s2, s3, red, &last);
}

hipError_t launch_cg_dots(const StencilArgs& a0, int n, hipStream_t st) {
  StencilArgs a = a0;
  const int ty = stencil_tile_y(M_CGF, 8, n, BC_ROBIN);
  a.tiles_x = (a.nx + 63) / 64;
  a.tiles_y = (a.ny + ty - 1) / ty;
  a.nblocks = a.tiles_x * a.tiles_y * a.nchunks;
  const bool vec = a.nx % 2 == 0;  // as launch_cgf
#define CG_DOTS(TY, WY, VE) hipLaunchKernelGGL((cg_dots_kernel<TY, WY, VE>), dim3(a.nblocks), dim3(64 * WY), 0, st, a)
  const int wy = stencil_tile_wy(M_CGF, 8, n, BC_ROBIN);
  if (ty == 16 && wy == 8) {
    if (vec) CG_DOTS(16, 8, 2);
    else CG_DOTS(16, 8, 1);
  } else if (ty == 8 && wy == 4) {
    if (vec) CG_DOTS(8, 4, 2);
    else CG_DOTS(8, 4, 1);
  } else {
    return hipErrorInvalidValue;
  }
#undef CG_DOTS
  return hipGetLastError();
}

// RESID: FP64 x and b; r written as f64 (r_dt 0) or f32 (r_dt 1) when out0 != NULL
hipError_t launch_resid(const StencilArgs& a, int n, int bc, int r_dt, hipStream_t st) {
  if (r_dt == 0) return launch_n<M_RESID, double, double, double>(a, n, bc, st);
  if (r_dt == 1) return launch_n<M_RESID, double, double, float>(a, n, bc, st);
  return hipErrorInvalidValue;
}

hipError_t launch_rhs_resid(const StencilArgs& a, int n, int bc, hipStream_t st) {
  const bool vec = (a.nx % 2) == 0;  // 16-byte staging of the FP64 input
  if (bc == BC_ROBIN) return hipErrorInvalidValue;
  const bool per = bc == BC_PERIODIC;
  switch (n) {
    case 1: return per ? launch_rhsres_bc<1, BC_PERIODIC>(a, vec, st) : launch_rhsres_bc<1, BC_DIRICHLET>(a, vec, st);
    case 2: return per ? launch_rhsres_bc<2, BC_PERIODIC>(a, vec, st) : launch_rhsres_bc<2, BC_DIRICHLET>(a, vec, st);
    case 3: return per ? launch_rhsres_bc<3, BC_PERIODIC>(a, vec, st) : launch_rhsres_bc<3, BC_DIRICHLET>(a, vec, st);
    case 4: return per ? launch_rhsres_bc<4, BC_PERIODIC>(a, vec, st) : launch_rhsres_bc<4, BC_DIRICHLET>(a, vec, st);
    case 5: return per ? launch_rhsres_bc<5, BC_PERIODIC>(a, vec, st) : launch_rhsres_bc<5, BC_DIRICHLET>(a, vec, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace tbs

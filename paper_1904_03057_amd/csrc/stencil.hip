// Dispatch of the stencil launches: (mode, dtype) combinations, basis degree n and boundary -> the
// kernel instances of stencil_kernel.h that stencil_inst.hip compiles per degree and boundary.
#include <algorithm>
#include <cmath>

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

// The planes per chunk with the smallest (zc + halo) max(lat, load), load the workgroups of the busiest of
// `slots` equal processors; at most most_blocks workgroups, or one chunk.
int plan_zc(int64_t tiles, int64_t nz, int halo, int slots, int64_t most_blocks, double lat, double tail,
            double* least) {
  const int64_t most = std::min<int64_t>(nz, std::max<int64_t>(1, most_blocks / tiles));
  int64_t best = nz;
  double cost = 0.0;
  for (int64_t want = 1; want <= most; ++want) {
    const int64_t zc = (nz + want - 1) / want, chunks = (nz + zc - 1) / zc;
    const double load = (double)(tiles * chunks) / slots;
    const double t = (double)(zc + halo) * std::max(lat, load <= 4.0 ? std::ceil(load) : load + tail);
    if (want == 1 || t < cost) {
      cost = t;
      best = zc;
    }
  }
  if (least) *least = cost;
  return (int)best;
}

int stencil_plan_zc(int64_t nx, int64_t ny, int64_t nz, int mode, int compute_bytes, int n, int bc, int zchunk,
                    int* shape) {
  if (shape) *shape = 0;
  if (zchunk > 0) return (int)std::min<int64_t>(zchunk, nz);
  const int wx = (mode == M_APPLY && compute_bytes == 4) ? STENCIL_APPLY_WX : 1;
  const int64_t tiles_x = (nx + 64 * wx - 1) / (64 * wx);
  if (compute_bytes == 8 && (mode == M_CGF || mode == M_CG1) && bc == BC_ROBIN && n >= 2) {
    const int64_t plan_tiles = ((nx + 63) / 64) * ((ny + 15) / 16);
    const int64_t chunks = std::max<int64_t>(1, std::min((8192 + plan_tiles - 1) / plan_tiles, nz / (4 * (2 * n + 1))));
    return (int)((nz + chunks - 1) / chunks);
  }
  int zc = 0;
  double least = 0.0;
  for (int sh = 0; sh < (mode == M_CGF && shape ? kCgfShapes : 1); ++sh) {
    const int ty = stencil_tile_y(mode, compute_bytes, n, bc, sh);
    if (ty == 0) continue;
    double cost;
    const int z = plan_zc(tiles_x * ((ny + ty - 1) / ty), nz, 2 * n, 256, 16384, stencil_latency_load(mode, compute_bytes),
                          mode == M_APPLY && compute_bytes == 4 ? 1.5 : 0.75, &cost);
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

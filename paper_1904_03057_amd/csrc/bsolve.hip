// Banded solves of the direct B-spline transform on gfx950 (Sec. 2.3, Fig. figBspnSignProc: the sampled
// B-spline b^n is inverted along each axis by recursive filtering).  The 1-D operator is a symmetric
// Toeplitz band of half-width W = floor(n / 2) <= 2; with E = L D L^T a line is solved by a forward
// and a backward recursion of W terms,
//   y_i = s_i - l1_i y_{i-1} - l2_i y_{i-2},   w_i = y_i / D_i,   c_i = w_i - l1_{i+1} c_{i+1} - l2_{i+2} c_{i+2}.
// On a truncated band the factor's rows converge to constants within kBandTab rows (the largest pole of
// degree 5 is -0.43, its square the rate).  A circulant band uses the constants everywhere and starts
// each recursion kWarm samples before the line's end, wrapped around: 0.27^32 (W = 1) and 0.43^48 (W = 2)
// are below 1e-17.
//
// One thread owns a line and runs both recursions in place, so a value is read and written twice per
// axis; the backward recursion starts on the values written last.  Along y and z neighbouring lanes are
// neighbouring x: every access of a wave is 512 contiguous bytes, and the values of the next kBatch steps
// are in flight while the current ones are used (one load per step would leave the memory latency on the
// chain).  Along x a wave stages 64 lines x kTile columns in LDS, so that memory sees 256-byte rows.
// Bound by memory: at 256^3 the axes take 86 (x), 75 (y) and 106 us (z, with the addition), 540 MB (z 800)
// read and written each at 6 to 7.5 TB/s with what the caches keep.
#include <algorithm>

#include "bsolve.h"

namespace tbs {

constexpr int kBatch = 16;  // steps per batch of loads (y, z)
constexpr int kTile = 32;   // columns per LDS tile (x)
template <int W> constexpr int kWarm = W == 1 ? 32 : 48;

// coefficients of row i (truncated band) or of the limit
template <int W, bool PER> struct Rows {
  const BandFactor& f;
  double l1, l2, dinv;
  __device__ Rows(const BandFactor& f_) : f(f_), l1(f_.l1[kBandTab - 1]), l2(f_.l2[kBandTab - 1]), dinv(f_.dinv[kBandTab - 1]) {}
  // lo: the smallest row of the batch (uniform): only the first kBandTab rows need the table
  __device__ double fwd(double s, double y1, double y2, int i, int lo) const {
    const bool t = !PER && lo < kBandTab;
    const int r = t ? min(i, kBandTab - 1) : 0;
    double y = __builtin_fma(-(t ? f.l1[r] : l1), y1, s);
    if (W == 2) y = __builtin_fma(-(t ? f.l2[r] : l2), y2, y);
    return y;
  }
  __device__ double scale(double y, int i, int lo) const {
    return y * (!PER && lo < kBandTab ? f.dinv[min(i, kBandTab - 1)] : dinv);
  }
  __device__ double bwd(double w, double c1, double c2, int i, int lo) const {
    const bool t = !PER && lo < kBandTab;
    double c = __builtin_fma(-(t ? f.l1[min(max(i + 1, 0), kBandTab - 1)] : l1), c1, w);
    if (W == 2) c = __builtin_fma(-(t ? f.l2[min(max(i + 2, 0), kBandTab - 1)] : l2), c2, c);
    return c;
  }
};

// Lines along y or z: line k starts at (k / inner) * outer + k % inner, its elements `stride` apart.
template <int W, bool PER>
__global__ __launch_bounds__(64) void solve_strided(double* __restrict__ v, double* __restrict__ dst, int64_t lines,
                                                    int64_t inner, int64_t outer, int64_t stride, int n, BandFactor f) {
  const int64_t k = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (k >= lines) return;
  const int64_t base = k / inner * outer + k % inner;
  double* line = v + base;
  double* out = dst ? dst + base : line;
  const Rows<W, PER> R(f);
  double y1 = 0.0, y2 = 0.0, cur[kBatch], nxt[kBatch];
  if (PER) {
    for (int b = kWarm<W>; b > 0; b -= kBatch) {
      int i = (n - b % n) % n;  // -b modulo n
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        cur[j] = line[(int64_t)i * stride];
        if (++i == n) i = 0;
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const double y = R.fwd(cur[j], y1, y2, 0, 0);
        y2 = y1;
        y1 = y;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kBatch; ++j) cur[j] = line[(int64_t)min(j, n - 1) * stride];
  for (int i0 = 0; i0 < n; i0 += kBatch) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j) nxt[j] = line[(int64_t)min(i0 + kBatch + j, n - 1) * stride];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const double y = R.fwd(cur[j], y1, y2, i0 + j, i0);
      y2 = y1;
      y1 = y;
      if (i0 + j < n) line[(int64_t)(i0 + j) * stride] = R.scale(y, i0 + j, i0);
      cur[j] = nxt[j];
    }
  }
  // backward; the prefetches of the last forward batch past the line's end are not used
  double c1 = 0.0, c2 = 0.0;
  if (PER) {
    for (int b = 0; b < kWarm<W>; b += kBatch) {
      int i = (kWarm<W> - 1 - b) % n;  // n + i modulo n, downwards
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        cur[j] = line[(int64_t)i * stride];
        if (--i < 0) i = n - 1;
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const double c = R.bwd(cur[j], c1, c2, 0, 0);
        c2 = c1;
        c1 = c;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kBatch; ++j) cur[j] = line[(int64_t)max(n - 1 - j, 0) * stride];
  for (int i0 = n - 1; i0 >= 0; i0 -= kBatch) {
    double add[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      nxt[j] = line[(int64_t)max(i0 - kBatch - j, 0) * stride];
      add[j] = dst ? out[(int64_t)max(i0 - j, 0) * stride] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int i = i0 - j;
      const double c = R.bwd(cur[j], c1, c2, i, i0 - kBatch);
      c2 = c1;
      c1 = c;
      if (i >= 0) out[(int64_t)i * stride] = add[j] + c;
      cur[j] = nxt[j];
    }
  }
}

// Lines along x: one wave per 64 lines.
template <int W, bool PER>
__global__ __launch_bounds__(64) void solve_x(double* __restrict__ v, int64_t lines, int n, BandFactor f) {
  __shared__ double t[64][kTile + 1];  // 33 doubles a row: the lanes of a half-wave hit different banks
  const int lane = threadIdx.x;
  const int64_t k0 = (int64_t)blockIdx.x * 64;
  double* row0 = v + k0 * n;
  const int rows = (int)min((int64_t)64, lines - k0);
  const Rows<W, PER> R(f);
  const int lr = lane >> 5, lc = lane & 31;  // two rows of the tile per access
  double pre[kTile];
  // tile columns c0 .. c0 + kTile - 1, taken modulo n (periodic warm-up) or up to the line's ends
  auto fetch = [&](int c0) {
    int c = c0 + lc;
    if (PER) c = ((c % n) + n) % n;
    c = min(max(c, 0), n - 1);
#pragma unroll
    for (int j = 0; j < kTile; ++j) pre[j] = row0[(int64_t)min(2 * j + lr, rows - 1) * n + c];
  };
  auto stash = [&]() {
#pragma unroll
    for (int j = 0; j < kTile; ++j) t[2 * j + lr][lc] = pre[j];
  };
  auto store = [&](int c0) {
    const int c = c0 + lc;
    if (c >= 0 && c < n)
#pragma unroll
      for (int j = 0; j < kTile; ++j)
        if (2 * j + lr < rows) row0[(int64_t)(2 * j + lr) * n + c] = t[2 * j + lr][lc];
  };
  double y1 = 0.0, y2 = 0.0;
  // The wave's own LDS accesses are in order, so no barrier is needed between the steps; the fences
  // keep the compiler from moving them across each other.
  const int w0 = PER ? -((kWarm<W> + kTile - 1) / kTile) * kTile : 0;
  fetch(w0);
  for (int c0 = w0; c0 < n; c0 += kTile) {
    stash();
    __syncthreads();
    // a circulant line's first columns are read by the warm-up of the backward recursion and its last
    // ones by the forward one, before they are overwritten
    if (c0 + kTile < n) fetch(c0 + kTile);
    if (PER && c0 < 0) {
#pragma unroll
      for (int j = 0; j < kTile; ++j) {
        const double y = R.fwd(t[lane][j], y1, y2, 0, 0);
        y2 = y1;
        y1 = y;
      }
      __syncthreads();
      continue;
    }
#pragma unroll
    for (int j = 0; j < kTile; ++j) {
      const double y = R.fwd(t[lane][j], y1, y2, c0 + j, c0);
      if (c0 + j < n) {
        y2 = y1;
        y1 = y;
      }
      t[lane][j] = R.scale(y, c0 + j, c0);
    }
    __syncthreads();
    store(c0);
    __syncthreads();
  }
  double c1 = 0.0, c2 = 0.0;
  const int last = (n - 1) / kTile * kTile;  // first column of the last tile
  if (PER) {
    // columns n .. n + kWarm - 1 modulo n, downwards, in tiles
    for (int c0 = n + (kWarm<W> + kTile - 1) / kTile * kTile - kTile; c0 >= n; c0 -= kTile) {
      fetch(c0);
      stash();
      __syncthreads();
#pragma unroll
      for (int j = kTile - 1; j >= 0; --j) {
        const double c = R.bwd(t[lane][j], c1, c2, 0, 0);
        c2 = c1;
        c1 = c;
      }
      __syncthreads();
    }
  }
  fetch(last);
  for (int c0 = last; c0 >= 0; c0 -= kTile) {
    stash();
    __syncthreads();
    if (c0 > 0) fetch(c0 - kTile);
#pragma unroll
    for (int j = kTile - 1; j >= 0; --j) {
      const double c = R.bwd(t[lane][j], c1, c2, c0 + j, c0);
      if (c0 + j < n) {
        c2 = c1;
        c1 = c;
      }
      t[lane][j] = c;
    }
    __syncthreads();
    store(c0);
    __syncthreads();
  }
}

BandFactor band_factor(const double* b, int W) {
  BandFactor f{};
  double d[kBandTab];
  for (int i = 0; i < kBandTab; ++i) {
    const double l2 = W == 2 && i >= 2 ? b[2] / d[i - 2] : 0.0;
    const double l1 = i >= 1 ? (b[1] - (i >= 2 ? l2 * d[i - 2] * f.l1[i - 1] : 0.0)) / d[i - 1] : 0.0;
    d[i] = b[0] - (i >= 1 ? l1 * l1 * d[i - 1] : 0.0) - (i >= 2 ? l2 * l2 * d[i - 2] : 0.0);
    f.l1[i] = l1;
    f.l2[i] = l2;
    f.dinv[i] = 1.0 / d[i];
  }
  return f;
}

template <int W, bool PER>
static hipError_t solve_axes(double* v, double* dst, const int dims[3], const BandFactor& f, hipStream_t st) {
  const int64_t nx = dims[0], ny = dims[1], nz = dims[2];
  auto blocks = [](int64_t lines) { return dim3((unsigned)((lines + 63) / 64)); };
  hipLaunchKernelGGL((solve_x<W, PER>), blocks(ny * nz), dim3(64), 0, st, v, ny * nz, (int)nx, f);
  hipLaunchKernelGGL((solve_strided<W, PER>), blocks(nx * nz), dim3(64), 0, st, v, (double*)nullptr, nx * nz, nx,
                     nx * ny, nx, (int)ny, f);
  hipLaunchKernelGGL((solve_strided<W, PER>), blocks(nx * ny), dim3(64), 0, st, v, dst, nx * ny, nx * ny, (int64_t)0,
                     nx * ny, (int)nz, f);
  return hipGetLastError();
}

hipError_t launch_band_solve(double* v, double* dst, const int dims[3], int W, int periodic, const BandFactor& f,
                             hipStream_t st) {
  if (W == 1) return periodic ? solve_axes<1, true>(v, dst, dims, f, st) : solve_axes<1, false>(v, dst, dims, f, st);
  if (W == 2) return periodic ? solve_axes<2, true>(v, dst, dims, f, st) : solve_axes<2, false>(v, dst, dims, f, st);
  return hipErrorInvalidValue;
}

}  // namespace tbs

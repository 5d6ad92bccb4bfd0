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

// Thin boxes: few, long lines would leave the chip to a handful of waves, each one serial chain (the cubic 1048576 x 5 x 5
// transform: 131 ms with whole lines, 26 with CG, 1.6 as here; 8192 x 16 x 16: 1.34, 2.4 and 0.20 ms).  There
// each line is cut into segments that run in threads of their own: a recursion started kWarm samples before its
// segment holds the line's values, as on a circulant line; outside a truncated line the samples are zero and so
// are the recursions.  A segment reads its neighbours' values, so the forward and the backward recursion are two
// launches, from one array to another.

// One step of a segment's forward (BWD: backward) recursion; i: position from the segment's start (uniform).
template <int W, bool PER, bool BWD> struct SegStep {
  const BandFactor& f;
  bool first;  // the line's first segment, whose rows the table holds
  double v1, v2;
  __device__ double co(const double* tab, int r, bool t) const {
    return t && first ? tab[min(max(r, 0), kBandTab - 1)] : tab[kBandTab - 1];
  }
  __device__ double operator()(double s, int i) {
    const bool t = !PER && i < kBandTab;
    double y = __builtin_fma(-co(f.l1, BWD ? i + 1 : i, t), v1, s);
    if (W == 2) y = __builtin_fma(-co(f.l2, BWD ? i + 2 : i, t), v2, y);
    v2 = v1;
    v1 = y;
    return BWD ? y : y * co(f.dinv, i, t);
  }
};

// Segments of lines along y or z (as solve_strided), blockIdx.y the segment.  add: dst += instead of dst =.
template <int W, bool PER, bool BWD>
__global__ __launch_bounds__(64) void seg_strided(const double* __restrict__ src, double* __restrict__ dst, int add,
                                                  int64_t lines, int64_t inner, int64_t outer, int64_t stride, int n,
                                                  int len, BandFactor f) {
  const int64_t k = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (k >= lines) return;
  const int64_t base = k / inner * outer + k % inner;
  const int lo = blockIdx.y * len, own = min(len, n - lo), steps = kWarm<W> + own;
  SegStep<W, PER, BWD> step{f, lo == 0, 0.0, 0.0};
  auto pos = [&](int s) { return BWD ? own - 1 + kWarm<W> - s : s - kWarm<W>; };  // from the segment's start
  auto load = [&](int s) -> double {
    int i = lo + pos(min(s, steps - 1));
    if (PER) i = i < 0 ? i + n : (i >= n ? i - n : i);
    return i >= 0 && i < n ? src[base + (int64_t)i * stride] : 0.0;
  };
  double cur[kBatch], nxt[kBatch];
#pragma unroll
  for (int j = 0; j < kBatch; ++j) cur[j] = load(j);
  for (int s0 = 0; s0 < steps; s0 += kBatch) {
    double old[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      nxt[j] = load(s0 + kBatch + j);
      const int s = s0 + j;
      old[j] = add && s >= kWarm<W> && s < steps ? dst[base + (int64_t)(lo + pos(s)) * stride] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int s = s0 + j;
      const double v = step(cur[j], pos(s));
      if (s >= kWarm<W> && s < steps) dst[base + (int64_t)(lo + pos(s)) * stride] = old[j] + v;
      cur[j] = nxt[j];
    }
  }
}

// Segments of lines along x: one wave per 64 of them (as solve_x), nseg consecutive ones to a line; len is a
// multiple of kTile.
template <int W, bool PER, bool BWD>
__global__ __launch_bounds__(64) void seg_x(const double* __restrict__ src, double* __restrict__ dst, int64_t segs, int n,
                                            int nseg, int len, BandFactor f) {
  constexpr int LEAD = (kWarm<W> + kTile - 1) / kTile * kTile;
  __shared__ double t[64][kTile + 1];
  const int lane = threadIdx.x, lr = lane >> 5, lc = lane & 31;
  const int64_t k0 = (int64_t)blockIdx.x * 64;
  const int64_t line0 = (k0 + lr) / nseg;
  const int seg0 = (int)((k0 + lr) % nseg);
  SegStep<W, PER, BWD> step{f, (k0 + lane) % nseg == 0, 0.0, 0.0};
  // every second segment from k0 + lr: element of column c0 + lc, -1 outside the line
  auto each = [&](int c0, auto&& use) {
    int64_t line = line0;
    int seg = seg0;
#pragma unroll
    for (int j = 0; j < kTile; ++j) {
      use(j, line, k0 + 2 * j + lr < segs ? seg * len + c0 + lc : -1);
      seg += 2;
      if (seg >= nseg) {
        seg -= nseg;
        ++line;
      }
    }
  };
  double pre[kTile];
  auto fetch = [&](int c0) {
    each(c0, [&](int j, int64_t line, int i) {
      if (PER && k0 + 2 * j + lr < segs) i = i < 0 ? i + n : (i >= n ? i - n : i);
      pre[j] = i >= 0 && i < n ? src[line * n + i] : 0.0;
    });
  };
  const int c_first = BWD ? len - kTile + LEAD : -LEAD, c_step = BWD ? -kTile : kTile;
  const int tiles = (len + LEAD) / kTile;
  fetch(c_first);
  for (int b = 0; b < tiles; ++b) {
    const int c0 = c_first + b * c_step;
#pragma unroll
    for (int j = 0; j < kTile; ++j) t[2 * j + lr][lc] = pre[j];
    __syncthreads();
    if (b + 1 < tiles) fetch(c0 + c_step);
#pragma unroll
    for (int j = 0; j < kTile; ++j) {
      const int c = BWD ? kTile - 1 - j : j;
      t[lane][c] = step(t[lane][c], c0 + c);
    }
    __syncthreads();
    if (c0 >= 0 && c0 < len)
      each(c0, [&](int j, int64_t line, int i) {
        if (i >= 0 && i < n) dst[line * n + i] = t[2 * j + lr][lc];
      });
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

// Segments a line of n samples is cut into (1: solved whole) and their length.  kFewWaves waves are one per CU, below
// which whole lines leave CUs idle (2048 x 32 x 32, 16 waves: 0.42 ms whole, 0.21 cut; 8192 x 64 x 64, 64 waves: 2.1 and
// 1.2); segments of at least kMinSeg samples keep the lead-in small beside them.
constexpr int64_t kFewWaves = 256, kManyWaves = 1024;
constexpr int kMinSeg = 256;
static int cut(int64_t lines, int n, int* len) {
  const int64_t waves = (lines + 63) / 64;
  int64_t nseg = waves < kFewWaves ? std::min<int64_t>(n / kMinSeg, (kManyWaves + waves - 1) / waves) : 1;
  if (nseg < 2) return 1;
  *len = (int)(((n + nseg - 1) / nseg + kTile - 1) / kTile * kTile);
  return (n + *len - 1) / *len;
}

template <int W, bool PER>
static hipError_t solve_axes(double* v, double* tmp, double* dst, const int dims[3], const BandFactor& f, hipStream_t st) {
  const int64_t nx = dims[0], ny = dims[1], nz = dims[2];
  auto blocks = [](int64_t lines) { return (unsigned)((lines + 63) / 64); };
  int len = 0;
  if (const int nseg = cut(ny * nz, (int)nx, &len); nseg > 1) {
    const int64_t segs = ny * nz * nseg;
    hipLaunchKernelGGL((seg_x<W, PER, false>), dim3(blocks(segs)), dim3(64), 0, st, (const double*)v, tmp, segs, (int)nx,
                       nseg, len, f);
    hipLaunchKernelGGL((seg_x<W, PER, true>), dim3(blocks(segs)), dim3(64), 0, st, (const double*)tmp, v, segs, (int)nx,
                       nseg, len, f);
  } else {
    hipLaunchKernelGGL((solve_x<W, PER>), dim3(blocks(ny * nz)), dim3(64), 0, st, v, ny * nz, (int)nx, f);
  }
  auto strided = [&](double* out, int64_t lines, int64_t inner, int64_t outer, int64_t stride, int n) {
    if (const int nseg = cut(lines, n, &len); nseg > 1) {
      const dim3 grid(blocks(lines), (unsigned)nseg);
      hipLaunchKernelGGL((seg_strided<W, PER, false>), grid, dim3(64), 0, st, (const double*)v, tmp, 0, lines, inner, outer,
                         stride, n, len, f);
      hipLaunchKernelGGL((seg_strided<W, PER, true>), grid, dim3(64), 0, st, (const double*)tmp, out ? out : v,
                         out ? 1 : 0, lines, inner, outer, stride, n, len, f);
    } else {
      hipLaunchKernelGGL((solve_strided<W, PER>), dim3(blocks(lines)), dim3(64), 0, st, v, out, lines, inner, outer, stride,
                         n, f);
    }
  };
  strided(nullptr, nx * nz, nx, nx * ny, nx, (int)ny);
  strided(dst, nx * ny, nx * ny, 0, nx * ny, (int)nz);
  return hipGetLastError();
}

hipError_t launch_band_solve(double* v, double* tmp, double* dst, const int dims[3], int W, int periodic,
                             const BandFactor& f, hipStream_t st) {
  if (W == 1) return periodic ? solve_axes<1, true>(v, tmp, dst, dims, f, st) : solve_axes<1, false>(v, tmp, dst, dims, f, st);
  if (W == 2) return periodic ? solve_axes<2, true>(v, tmp, dst, dims, f, st) : solve_axes<2, false>(v, tmp, dst, dims, f, st);
  return hipErrorInvalidValue;
}

}  // namespace tbs

// Learned initial guess for the implicit step: a 4-layer 3x3x3 CNN (2 -> 16 -> 16 -> 16 -> 1,
// exact-erf GELU) with bf16 operands on the gfx950 matrix cores and FP32 accumulation.  Not in
// the paper (which warm-starts CG from a coarse-grid solution); the network predicts
// u^{k+1} - u^k from (u^k, f) and the solver keeps its guess only if the FP64 residual drops.
//
// Activations are channels-last [voxel][16] bf16 (32 B per voxel); the first layer's input has
// 2 channels, the last layer's output 1.  Every convolution is an implicit GEMM on
// v_mfma_f32_16x16x32_bf16 computing Out^T = W^T In^T: M = 16 output channels (zero padded),
// N = 16 voxels along x, K = 2 taps x 16 input channels per instruction (27 taps padded to 30).
// A workgroup stages its input tile (halo 1) in LDS with 16 channels per voxel and each wave
// accumulates 16-voxel rows.  The same kernel runs the backward data pass with flipped,
// transposed weights; the last layer has a kernel of its own (conv_last).  Weight gradients are a
// deterministic two-stage reduction (per-workgroup partial sums on the matrix cores, then a
// fixed-order sum).  Optimiser: Adam on FP32 master weights.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <type_traits>

#include "../../include/tbs.h"
#include "common.h"
#include "net.h"

namespace tbs {
namespace net {

constexpr int NL = 4;
constexpr int CIN[NL] = {2, 16, 16, 16};
constexpr int COUT[NL] = {16, 16, 16, 1};
constexpr int NSTEP = 15;         // MFMA K-steps of the 16-channel layout (27 taps + 3 zero partners) / 2
constexpr int PACK = NSTEP * 64 * 8;  // bf16 per packed layer
constexpr int WG_PARTS = 6928;    // max partial-gradient row: 16*16*27 weights + 16 biases
constexpr int SMOOTH_PASSES = 2;  // passes of the separable binomial low-pass after the last layer

__host__ __device__ constexpr int woff(int l) {  // offset of W_l in the flat parameter vector
  return l == 0 ? 0 : woff(l - 1) + CIN[l - 1] * COUT[l - 1] * 27 + COUT[l - 1];
}
__host__ __device__ constexpr int boff(int l) { return woff(l) + CIN[l] * COUT[l] * 27; }
static_assert(woff(NL) == TBS_NET_PARAMS, "parameter count");

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// GELU(x) = x Phi(x) = max(x, 0) - |x| Phi(-|x|), with the normal tail Phi(-y) = t 2^(P(t) - y^2 /
// (2 ln 2)), t = 1 / (1 + c y), P of degree 6 fitted by fit_gelu.py (relative error of Phi(-y)
// below 1.3e-6 for all y >= 0), so the negative tail keeps its relative accuracy.
__device__ __forceinline__ float gelu_f(float x) {
  const float y = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(2.700000107e-01f, y, 1.0f));
  float p = 3.957020044e-01f;
  p = fmaf(p, t, -1.359942675e+00f);
  p = fmaf(p, t, 1.348554134e+00f);
  p = fmaf(p, t, -3.906427920e-01f);
  p = fmaf(p, t, 8.047851324e-01f);
  p = fmaf(p, t, 1.414555073e+00f);
  p = fmaf(p, t, -3.213009119e+00f);
  const float q = t * __builtin_amdgcn_exp2f(fmaf(y * y, -0.72134752044448170f, p));  // Phi(-y)
  return fmaf(-y, q, __builtin_amdgcn_fmed3f(x, 0.f, __builtin_inff()));  // max(x, 0) in one instruction
}
// GELU'(x) = Phi(x) + x phi(x) from the tail's side: GELU'(-y) = e (0.5 + y (t P(t) - 1 / sqrt(2 pi))),
// e = 2^(-y^2 / (2 ln 2)), t = 1 / (1 + y / 4), and GELU'(y) = 1 - GELU'(-y).  P of degree 6 fitted by
// fit_gelu.py; every rounding but the last is scaled by e or y: error against 64 bits at most 1.11e-7, rms
// 2.2e-8 on [-8, 8] (1.44e-7 and 2.6e-8 with erff and expf, at three times the instructions).
__device__ __forceinline__ float gelu_grad_f(float x) {
  const float y = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.25f, y, 1.0f));
  float p = 2.358977310e-02f;
  p = fmaf(p, t, -6.521388888e-02f);
  p = fmaf(p, t, 8.545549586e-03f);
  p = fmaf(p, t, -6.954040378e-02f);
  p = fmaf(p, t, -7.072117180e-02f);
  p = fmaf(p, t, -1.006303057e-01f);
  p = fmaf(p, t, -1.249715537e-01f);
  const float e = __builtin_amdgcn_exp2f(y * y * -0.72134752044448170f);
  const float d = fmaf(y, fmaf(t, p, -0.39894228040143268f), 0.5f);
  return fmaf(x > 0.f ? -e : e, d, x > 0.f ? 1.0f : 0.0f);
}

struct Grid3 {
  int nx, ny, nz;
  int periodic;
};

// ------------------------------------------------------------------------------------------
// convolution on the matrix cores

enum Epi { EPI_GELU = 0, EPI_BWD = 2, EPI_RAW = 3, EPI_GELU_Z = 4 };

// Geometry of the z-marching convolution: a workgroup owns a 32 x 8 column of output voxels and
// marches through a chunk of zc planes, keeping the three input planes a output plane needs in an
// LDS ring (one-voxel halo in x and y) and fetching the next plane into registers meanwhile.
constexpr int CTX = 32, CTY = 8;                  // output tile per plane (x, y)
constexpr int SX = CTX + 2, SY = CTY + 2;          // staged plane
constexpr int PLV = SX * SY;                       // voxels per staged plane
constexpr int WROWS = 2 * CTY / 4;                 // 16-voxel rows per wave per plane

struct ConvGeo {
  int tx, ty, nch, zc;
};
// z-chunk length: about `wgs` workgroups on small grids, at most 96 planes per chunk
__host__ __device__ inline ConvGeo conv_geo(const Grid3& g, int wgs = 2048) {
  ConvGeo c;
  c.tx = (g.nx + CTX - 1) / CTX;
  c.ty = (g.ny + CTY - 1) / CTY;
  int64_t zc = (int64_t)g.nz * c.tx * c.ty / wgs;
  c.zc = (int)(zc < 4 ? 4 : (zc > 96 ? 96 : zc));
  c.nch = (g.nz + c.zc - 1) / c.zc;
  return c;
}

// 16-channel K order.  Tap index t = 9 dz + 3 dy + dx.  K-step s holds taps tap16(s, 0) and
// tap16(s, 1): steps 3 dy + dx pair (0, dy, dx) with (1, dy, dx); steps 9 + dy pair (2, dy, 0) with
// (2, dy, 1); steps 12 + dy hold (2, dy, 2) and a zero-weight partner.  For a fixed dz-pair and dx
// the B operand depends only on the staged row y + dy, so one LDS read serves the three output
// rows it touches (dy = 0, 1, 2), each with its own A operand.
__host__ __device__ constexpr int tap16(int s, int half) {
  return s < 9 ? s + 9 * half : (s < 12 ? 18 + 3 * (s - 9) + half : 18 + 3 * (s - 12) + 2);
}
__host__ __device__ constexpr bool pad16(int s, int half) { return s >= 12 && half == 1; }

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
// two floats to packed bf16 (round to nearest even) with the gfx950 conversion instruction
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// in: [voxel][CIS] bf16; wpk: packed A operands [steps][64 lanes][8]; out per epilogue:
//   EPI_GELU:   yout (bf16 [voxel][16]) = GELU(z), z = acc + bias
//   EPI_GELU_Z: as EPI_GELU, and zout (f32 [voxel][16]) = z
//   EPI_BWD:    yout (bf16 [voxel][16]) = acc * GELU'(zprev[voxel][c])       (backward data)
//   EPI_RAW:    fout (f32 [voxel][COS]) = acc (+ bias if bias != NULL)       (parity probes)
// Two K layouts: with 16 input channels each K-step holds 2 taps x 16 channels (15 steps, order
// tap16); with 2 (or 1) input channels it holds 16 taps x 2 (32 taps x 1) channels (2 steps or one,
// 27 taps padded to 32), and the ring keeps only those channels.  Each wave owns 4 consecutive
// rows (y) of 16 voxels (x) per plane; the plane loop is unrolled by the ring period so all LDS
// reads of the B operands use immediate offsets.
//
// The backward data pass moves 96 (1 -> 16 channels) or 128 bytes per voxel, 42 or 56 us at 128^3 at the
// copy rate, and takes 50 or 64 us there; 88 or 83 us with 1 channel padded to 16, GELU' from erff and expf
// and z loaded only after the products.
//
// The launch bound is the occupancy these kernels have anyhow (three or four waves per SIMD); said aloud it
// makes the compiler keep the accumulators out of the accumulation registers, whose contents the epilogue
// would first have to move: 64 against 69 us (16 -> 16 backward), 68 against 71 us (forward, storing z).
template <int CIS, int COS, int EPI>
__global__ __launch_bounds__(256, CIS == 16 ? 3 : 4) void conv_mfma(const uint16_t* __restrict__ in, const uint16_t* __restrict__ wpk,
                                                 const float* __restrict__ bias, Grid3 g,
                                                 float* __restrict__ zout, uint16_t* __restrict__ yout,
                                                 float* __restrict__ fout, const float* __restrict__ zprev) {
  constexpr bool TAPS = (CIS < 16);                 // K runs over taps x CIS channels
  constexpr int STEPS = TAPS ? CIS : NSTEP;
  constexpr int VW = CIS;                           // bf16 per staged voxel
  constexpr int UNITS = CIS == 16 ? 2 * PLV : PLV;  // load units per plane (16 B, or one voxel)
  constexpr int UPT = (UNITS + 255) / 256;          // units per thread
  using Unit = typename std::conditional<CIS == 16, uint4, typename std::conditional<CIS == 2, uint32_t, uint16_t>::type>::type;
  __shared__ __attribute__((aligned(16))) uint16_t st[3 * PLV * VW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const ConvGeo geo = conv_geo(g);
  const int64_t plane = (int64_t)g.nx * g.ny;

  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int bx = bid % geo.tx, by = (bid / geo.tx) % geo.ty, ch = bid / (geo.tx * geo.ty);
  const int x0 = bx * CTX, y0 = by * CTY, z0 = ch * geo.zc;
  const int zc = min(geo.zc, g.nz - z0);
  const bool inside = x0 + CTX <= g.nx && y0 + CTY <= g.ny;

  // A operands (weights) for all K-steps, loaded once and kept in registers
  bf16x8 wa[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) wa[s] = *(const bf16x8*)(wpk + (s * 64 + lane) * 8);
  float bz[4] = {0.f, 0.f, 0.f, 0.f};
  const int grp = lane >> 4;          // K-group of this lane
  const int vx = lane & 15;           // voxel (x) of this lane's B column / D column
  const int c0 = 4 * grp;             // D rows (output channels) held by this lane
  if (bias)
#pragma unroll
    for (int r = 0; r < 4; ++r) bz[r] = (c0 + r < COS) ? bias[c0 + r] : 0.f;

  // this thread's load units: plane-relative global voxel offsets (-1: outside a Dirichlet grid)
  int uoff[UPT];
#pragma unroll
  for (int q = 0; q < UPT; ++q) {
    const int u = tid + 256 * q;
    const int v = CIS == 16 ? (u >> 1) : u;
    int gx = x0 - 1 + v % SX, gy = y0 - 1 + v / SX;
    bool ok = u < UNITS;
    if (g.periodic) {
      gx = (gx + g.nx) % g.nx;
      gy = (gy + g.ny) % g.ny;
    } else {
      ok = ok && gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
    }
    uoff[q] = ok ? gy * g.nx + gx : -1;
  }
  Unit pre[UPT];
  // fetch relative plane j (global plane z0 - 1 + j) into pre
  auto fetch = [&](int j) {
    int gz = z0 - 1 + j;
    bool pv = true;
    if (g.periodic) gz = (gz + g.nz) % g.nz;
    else pv = gz >= 0 && gz < g.nz;
    const int64_t pb = (int64_t)gz * plane;
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      pre[q] = Unit{};
      if (pv && uoff[q] >= 0) {
        if constexpr (CIS == 16) pre[q] = ((const uint4*)(in + (pb + uoff[q]) * 16))[(tid + 256 * q) & 1];
        else if constexpr (CIS == 2) pre[q] = *(const uint32_t*)(in + (pb + uoff[q]) * 2);
        else pre[q] = in[pb + uoff[q]];
      }
    }
  };
  auto stash = [&](int slot) {
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int u = tid + 256 * q;
      if (UNITS % 256 == 0 || u < UNITS) {
        if constexpr (CIS == 16) ((uint4*)st)[slot * PLV * 2 + u] = pre[q];
        else ((Unit*)st)[slot * PLV + u] = pre[q];
      }
    }
  };

  // B operand lane offsets (bf16 elements of st) for the wave's first row: wave w owns rows
  // y = 4 (w >> 1) + r (r = 0..3) of x half w & 1
  const int yb = 4 * (wave >> 1), xh = wave & 1;
  const int lb = yb * SX + xh * 16 + vx;
  constexpr int TPL = 8 / (TAPS ? CIS : 8);  // taps of a lane per K-step
  int loff[TAPS ? 24 : 5];
  if (TAPS) {
    // k = 8 grp + j: tap (32 s + 8 grp + j) / CIS, channel j % CIS; padding taps (> 26) read tap 13
#pragma unroll
    for (int ph = 0; ph < 3; ++ph)
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int t = 0; t < TPL; ++t) {
          int tap = (4 * s + grp) * TPL + t;
          if (tap > 26) tap = 13;
          loff[8 * ph + TPL * s + t] = (lb + ((ph + tap / 9) % 3) * PLV + ((tap / 3) % 3) * SX + tap % 3) * CIS;
        }
  } else {
    // k = 8 grp + j: tap tap16(s, grp >> 1), channel 8 (grp & 1) + j
    const int l0 = lb * 16 + (grp & 1) * 8, h = grp >> 1;
#pragma unroll
    for (int ph = 0; ph < 3; ++ph) loff[ph] = l0 + h * ((ph == 2 ? -2 : 1) * PLV * 16);  // dz 0 -> dz 1
    loff[3] = l0 + h * 16;                                                           // dx 0 -> dx 1
    loff[4] = l0;                                                                    // partner unused
  }

  // prologue: ring slots 0..2 hold planes z0-1, z0, z0+1; registers hold plane z0+2
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    fetch(j);
    stash(j);
  }
  fetch(3);

  for (int i0 = 0; i0 < zc; i0 += 3) {
#pragma unroll
    for (int ph = 0; ph < 3; ++ph) {
      const int i = i0 + ph;
      if (i < zc) {  // uniform
        __syncthreads();  // plane z0 + i + 1 is in the ring
        const int gz = z0 + i;
        f32x4 acc[WROWS];
#pragma unroll
        for (int r = 0; r < WROWS; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
        float4 zp[EPI == EPI_BWD ? WROWS : 1];  // in flight during the products (lanes outside: the last voxel)
        if constexpr (EPI == EPI_BWD)
#pragma unroll
          for (int r = 0; r < WROWS; ++r) {
            const int gx = min(x0 + xh * 16 + vx, g.nx - 1), gy = min(y0 + yb + r, g.ny - 1);
            zp[r] = *(const float4*)(zprev + ((int64_t)gz * plane + (int64_t)gy * g.nx + gx) * 16 + c0);
          }
        if constexpr (TAPS) {
#pragma unroll
          for (int r = 0; r < WROWS; ++r)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
              Unit w4[TPL];
#pragma unroll
              for (int t = 0; t < TPL; ++t) w4[t] = *(const Unit*)(st + loff[8 * ph + TPL * s + t] + r * SX * CIS);
              bf16x8 bv;
              __builtin_memcpy(&bv, w4, 16);
              acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[s], bv, acc[r], 0, 0, 0);
            }
        } else {
          // staged rows yb + yy, yy = 0..5, feed output rows r = yy - dy
#pragma unroll
          for (int yy = 0; yy < WROWS + 2; ++yy) {
#pragma unroll
            for (int q = 0; q < 5; ++q) {
              // q < 3: planes (k-1, k) at dx = q; q = 3: plane k+1 at dx (0, 1); q = 4: plane k+1 at dx 2
              const int pl = q < 3 ? ph : (ph + 2) % 3;
              const int dx = q < 3 ? q : (q == 3 ? 0 : 2);
              const int lo = q < 3 ? loff[ph] : loff[q];
              const bf16x8 bv = *(const bf16x8*)(st + lo + (pl * PLV + yy * SX + dx) * 16);
#pragma unroll
              for (int dy = 0; dy < 3; ++dy) {
                const int r = yy - dy;
                if (r >= 0 && r < WROWS) {
                  const int sidx = q < 3 ? 3 * dy + q : (q == 3 ? 9 + dy : 12 + dy);
                  acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[sidx], bv, acc[r], 0, 0, 0);
                }
              }
            }
          }
        }
        // D layout: acc[r] = Out[channel 4 grp + r][voxel vx]
        auto emit = [&](int r) {
          const f32x4 A = acc[r];
          const int gx = x0 + xh * 16 + vx, gy = y0 + yb + r;
          const int64_t vi = (int64_t)gz * plane + (int64_t)gy * g.nx + gx;
          if constexpr (EPI == EPI_GELU || EPI == EPI_GELU_Z) {
            float z[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) z[c] = A[c] + bz[c];
            if (EPI == EPI_GELU_Z) *(float4*)(zout + vi * 16 + c0) = make_float4(z[0], z[1], z[2], z[3]);
            uint2 packed;
            packed.x = pack_bf16x2(gelu_f(z[0]), gelu_f(z[1]));
            packed.y = pack_bf16x2(gelu_f(z[2]), gelu_f(z[3]));
            *(uint2*)(yout + vi * 16 + c0) = packed;
          } else if (EPI == EPI_BWD) {
            uint2 packed;
            packed.x = pack_bf16x2(A[0] * gelu_grad_f(zp[r].x), A[1] * gelu_grad_f(zp[r].y));
            packed.y = pack_bf16x2(A[2] * gelu_grad_f(zp[r].z), A[3] * gelu_grad_f(zp[r].w));
            *(uint2*)(yout + vi * 16 + c0) = packed;
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
              if (c0 + c < COS) fout[vi * COS + c0 + c] = A[c] + bz[c];
          }
        };
        // a tile inside the grid has no lane to mask: its four rows' epilogues form one block of
        // instructions, in which the long chains of the activation overlap
        if (inside) {
#pragma unroll
          for (int r = 0; r < WROWS; ++r) emit(r);
        } else {
#pragma unroll
          for (int r = 0; r < WROWS; ++r)
            if (x0 + xh * 16 + vx < g.nx && y0 + yb + r < g.ny) emit(r);
        }
        __syncthreads();  // every wave is done with slot ph (plane z0 + i - 1)
        if (i + 3 <= zc + 1) {
          stash(ph);                         // plane z0 + i + 2 (relative plane i + 3)
          if (i + 4 <= zc + 1) fetch(i + 4);
        }
      }
    }
  }
}

// The last layer, 16 channels -> 1: fout (f32 [voxel]) = (acc + bias[0]) * (*scale), or acc + bias[0] without
// a scale.  With one output channel the 16 rows of the A operand hold taps instead: row 4 dz + dy (dz, dy
// = 0..2; the others zero) contracts the 3 taps along x (two K-steps: dx 0 and 1, then dx 2 and a
// zero-weight partner), so an input row gives nine partial sums, which the vector ALU adds to the output
// rows they belong to: 12 matrix instructions per 64 voxels of an input plane, where a row per output
// channel takes 60 and keeps three planes in LDS.  Lane group dz of the D layout holds the sums of output
// plane z + 1 - dz (z: the input plane), four rows in its registers; after a plane, group 2's are complete
// and the others move on by one group.
//
// 256^3: 146 us (4.1 TB/s; 126 us at the copy rate) against 237 with a row per output channel, 128^3: 23
// against 36 us.
//
// z-chunks for 1024 workgroups, four per CU of the six that registers allow: longer chunks read fewer halo
// planes, 149 us at 256^3 against 156 (2048 workgroups) and 159 us (4096).
constexpr int kLastWgs = 1024;

__global__ __launch_bounds__(256, 6) void conv_last(const uint16_t* __restrict__ in, const uint16_t* __restrict__ wpk,
                                                 const float* __restrict__ bias, Grid3 g, float* __restrict__ fout,
                                                 const double* __restrict__ scale) {
  constexpr int UNITS = 2 * PLV, UPT = (UNITS + 255) / 256;  // 16-byte load units per plane, per thread
  __shared__ __attribute__((aligned(16))) uint16_t st[2 * PLV * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ConvGeo geo = conv_geo(g, kLastWgs);
  const int64_t plane = (int64_t)g.nx * g.ny;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int bx = bid % geo.tx, by = (bid / geo.tx) % geo.ty, ch = bid / (geo.tx * geo.ty);
  const int x0 = bx * CTX, y0 = by * CTY, z0 = ch * geo.zc;
  const int zc = min(geo.zc, g.nz - z0);

  bf16x8 wa[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) wa[s] = *(const bf16x8*)(wpk + (s * 64 + lane) * 8);
  const float b0 = bias[0];
  const int grp = lane >> 4, vx = lane & 15;

  // this thread's load units: plane-relative global voxel offsets (-1: outside a Dirichlet grid)
  int uoff[UPT];
#pragma unroll
  for (int q = 0; q < UPT; ++q) {
    const int u = tid + 256 * q, v = u >> 1;
    int gx = x0 - 1 + v % SX, gy = y0 - 1 + v / SX;
    bool ok = u < UNITS;
    if (g.periodic) {
      gx = (gx + g.nx) % g.nx;
      gy = (gy + g.ny) % g.ny;
    } else {
      ok = ok && gx >= 0 && gx < g.nx && gy >= 0 && gy < g.ny;
    }
    uoff[q] = ok ? gy * g.nx + gx : -1;
  }
  uint4 pre[UPT];
  auto fetch = [&](int j) {  // relative plane j (global plane z0 - 1 + j)
    int gz = z0 - 1 + j;
    bool pv = true;
    if (g.periodic) gz = (gz + g.nz) % g.nz;
    else pv = gz >= 0 && gz < g.nz;
    const int64_t pb = (int64_t)gz * plane;
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      pre[q] = make_uint4(0, 0, 0, 0);
      if (pv && uoff[q] >= 0) pre[q] = ((const uint4*)(in + (pb + uoff[q]) * 16))[tid & 1];
    }
  };
  auto stash = [&](int slot) {
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      const int u = tid + 256 * q;
      if (u < UNITS) ((uint4*)st)[slot * UNITS + u] = pre[q];
    }
  };
  // wave w owns rows y = 4 (w >> 1) + r (r = 0..3) of x half w & 1; k = 8 grp + j: dx grp >> 1 (step 0) or 2
  // (step 1; its partner reads the same voxel), channel 8 (grp & 1) + j
  const int yb = 4 * (wave >> 1), xh = wave & 1;
  const int l1 = (yb * SX + xh * 16 + vx) * 16 + (grp & 1) * 8, l0 = l1 + (grp >> 1) * 16;

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};  // rows yb + r of output plane z + 1 - grp
  fetch(0);
  stash(0);
  fetch(1);
  for (int j = 0; j < zc + 2; ++j) {
    __syncthreads();  // plane j is in its slot, and the other slot has been read
    if (j < zc + 1) stash((j + 1) & 1);
    if (j < zc) fetch(j + 2);
    const uint16_t* sp = st + (j & 1) * PLV * 16;
    f32x4 p[WROWS + 2];
#pragma unroll
    for (int yy = 0; yy < WROWS + 2; ++yy) {
      p[yy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[0], *(const bf16x8*)(sp + l0 + yy * SX * 16),
                                                      f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      p[yy] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[1], *(const bf16x8*)(sp + l1 + (yy * SX + 2) * 16), p[yy], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < WROWS; ++r) acc[r] += (p[r][0] + p[r + 1][1]) + p[r + 2][2];
    if (j >= 2 && grp == 2) {
      const int gx = x0 + xh * 16 + vx;
      float* o = fout + (int64_t)(z0 + j - 2) * plane + (int64_t)(y0 + yb) * g.nx + gx;
#pragma unroll
      for (int r = 0; r < WROWS; ++r)
        if (gx < g.nx && y0 + yb + r < g.ny)
          o[(int64_t)r * g.nx] = scale ? (float)(((double)acc[r] + (double)b0) * scale[0]) : acc[r] + b0;
    }
#pragma unroll
    for (int r = 0; r < WROWS; ++r) {
      const float v = __shfl_up(acc[r], 16);
      acc[r] = grp == 0 ? 0.f : v;
    }
  }
}

// ------------------------------------------------------------------------------------------
// weight gradient on the matrix cores: dW[co][ci][tap] = sum_v X[v + off(tap)][ci] G[v][co],
// dB[co] = sum_v G[v][co], with bf16 X and G (exact products) and FP32 accumulation.
//
// One v_mfma_f32_16x16x32_bf16 contracts 32 voxels of a row: A = G (M = 16 output channels), B = X
// (N = 16 input channels), one accumulator per tap (27, and one for the biases with B = 1).  Both
// operands need consecutive voxels per lane while the arrays are channels-last, so they are read
// from LDS with the transposing ds_read_b64_tr_b16: a tap's x offset is then only a row offset.  A
// workgroup owns tiles of 32 (x) x 4 x 4 X rows (wave w: plane w); an X row in registers serves its
// nine G rows (y and z neighbours), which keeps the LDS reads at 0.2 KB per matrix instruction, and
// the row pairs need no halo work: X outside the grid contributes nothing.  Layers with 2 input
// channels or 1 output channel run with the other channels zero in LDS.
//
// The arrays read once take 28 us for 16 -> 16 channels at 128^3 and the matrix instructions 12 us;
// the vector-ALU form this replaced took 2335 us there (16 -> 1: 298 us, 2 -> 16: 128 us), this one
// 62 (41, 45) us.  What bounds it is the latency of a tile (fetch, two barriers, 112 matrix
// instructions in one wave per SIMD): 85 us without the register prefetch of the next tile at two
// workgroups per CU, 225 us with both (the prefetch spills).
//
// The narrow layers use 1 or 2 of an accumulator's 4 values and have more tiles to a workgroup's chain than the
// vector-ALU form had voxels, so each tile is summed by itself and then added: error against 64 bits at
// 128^3 9.1e-8 to 9.9e-8, 1.8e-7 to 2.0e-7 with one chain per workgroup (38 and 42 us), 1.0e-7 to 1.2e-7 in the
// vector-ALU form.
//
// Each workgroup sums its tiles (grid stride) in registers and writes one row of partial sums (its
// waves added in a fixed order); a second kernel adds the rows in a fixed order in FP64.

constexpr int WTX = 32, WTY = 4, WTZ = 4;      // X rows of a tile: WTY x WTZ, 32 voxels long
constexpr int WXV = (WTX + 2) * WTY * WTZ;     // staged X voxels (one-voxel halo in x)
constexpr int WGV = WTX * (WTY + 2) * (WTZ + 2);  // staged G voxels (one-row halo in y and z)
constexpr int WACC = 28;                       // accumulators: 27 taps and the biases

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
// The 8 voxels 8 (lane >> 4) + j of a 32-voxel row at p (channels-last, 16 channels), channel lane & 15.
__device__ __forceinline__ bf16x8 read_row_tr(const uint16_t* p, int lane) {
  typedef __attribute__((address_space(3))) s16x4* lds;
  const uint16_t* q = p + (8 * (lane >> 4) + ((lane & 15) >> 2)) * 16 + (lane & 3) * 4;
  s16x4 v[2] = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)q), __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds)(q + 64))};
  return __builtin_bit_cast(bf16x8, v);
}

template <int CIS, int COS>
__global__ __launch_bounds__(256, CIS * COS == 256 ? 1 : 2) void wgrad_partial(const uint16_t* __restrict__ xin,
                                                        const uint16_t* __restrict__ gin, Grid3 g,
                                                        float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) uint16_t st[(WXV + WGV) * 16];  // staged X, then G
  static_assert(sizeof(st) >= WACC * 65 * 4 * sizeof(float), "the wave reduction reuses the stage");
  uint16_t* xs = st;
  uint16_t* gs = st + WXV * 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: matrix instructions ignore the lane mask
  const int tx = (g.nx + WTX - 1) / WTX, ty = (g.ny + WTY - 1) / WTY, tz = (g.nz + WTZ - 1) / WTZ;
  const int ntiles = tx * ty * tz;
  const int64_t plane = (int64_t)g.nx * g.ny;
  // index along one axis one past either end: wrapped (periodic) or outside (-1, as anything beyond)
  auto fold = [&](int i, int n) -> int {
    if (g.periodic) i = i == -1 ? n - 1 : (i == n ? 0 : i);
    return i >= 0 && i < n ? i : -1;
  };
  // D layout: acc[t][r] = dW[co = 4 (lane >> 4) + r][ci = lane & 15]; with 2 input channels the operands change
  // places, dW[co = lane & 15][ci = 4 (lane >> 4) + r].  A narrow layer's gradients are in the first KEEP values
  // of a lane.  There each tile is summed by itself and then added, which keeps the FP32 chains short.
  constexpr int KEEP = COS == 1 ? 1 : (CIS == 2 ? 2 : 4);
  constexpr bool NARROW = KEEP < 4;
  f32x4 acc[WACC];
#pragma unroll
  for (int t = 0; t < WACC; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mma = [](bf16x8 gv, bf16x8 xv, f32x4 c) {
    return CIS == 2 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, gv, c, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_16x16x32_bf16(gv, xv, c, 0, 0, 0);
  };
  if (CIS < 16 || COS < 16)  // channels the layer does not have stay zero
    for (int i = tid; i < (WXV + WGV) * 2; i += 256) ((uint4*)st)[i] = make_uint4(0, 0, 0, 0);

  // A thread's load units (16 bytes of a voxel, or a voxel of a narrow layer) are fetched into registers
  // while the previous tile is multiplied.
  constexpr int XU = CIS == 16 ? 2 * WXV : WXV, GU = COS == 16 ? 2 * WGV : WGV;
  constexpr int XN = (XU + 255) / 256, GN = (GU + 255) / 256;
  using XUnit = typename std::conditional<CIS == 16, uint4, uint32_t>::type;
  using GUnit = typename std::conditional<COS == 16, uint4, uint16_t>::type;
  static_assert((CIS == 16 || CIS == 2) && (COS == 16 || COS == 1), "channel counts");
  XUnit px[XN];
  GUnit pg[GN];
  // tiles in turn over the XCDs' own ranges: neighbours that share halo rows meet in one L2
  auto locate = [&](int tile, int& x0, int& y0, int& z0) {
    tile = xcd_remap(tile, ntiles);
    x0 = tile % tx * WTX;
    y0 = tile / tx % ty * WTY;
    z0 = tile / (tx * ty) * WTZ;
  };
  auto fetch = [&](int tile) {
    int x0, y0, z0;
    locate(tile, x0, y0, z0);
    // X: rows of the grid only (y0 + r < ny, z0 + r < nz)
#pragma unroll
    for (int q = 0; q < XN; ++q) {
      const int u = tid + 256 * q, v = CIS == 16 ? u >> 1 : u;
      const int gx = fold(x0 - 1 + v % (WTX + 2), g.nx);
      const int gy = y0 + (v / (WTX + 2)) % WTY, gz = z0 + v / ((WTX + 2) * WTY);
      px[q] = XUnit{};
      if (u < XU && gx >= 0 && gy < g.ny && gz < g.nz) {
        const uint16_t* p = xin + ((int64_t)gz * plane + (int64_t)gy * g.nx + gx) * CIS;
        px[q] = ((const XUnit*)p)[CIS == 16 ? u & 1 : 0];
      }
    }
    // G: x inside the grid only
#pragma unroll
    for (int q = 0; q < GN; ++q) {
      const int u = tid + 256 * q, v = COS == 16 ? u >> 1 : u;
      const int gx = x0 + v % WTX;
      const int gy = fold(y0 - 1 + (v / WTX) % (WTY + 2), g.ny), gz = fold(z0 - 1 + v / (WTX * (WTY + 2)), g.nz);
      pg[q] = GUnit{};
      if (u < GU && gx < g.nx && gy >= 0 && gz >= 0) {
        const uint16_t* p = gin + ((int64_t)gz * plane + (int64_t)gy * g.nx + gx) * COS;
        pg[q] = ((const GUnit*)p)[COS == 16 ? u & 1 : 0];
      }
    }
  };

  if ((int)blockIdx.x < ntiles) fetch(blockIdx.x);
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    int x0, y0, z0;
    locate(tile, x0, y0, z0);
    __syncthreads();  // the previous tile's reads (and the zero fill) are done
#pragma unroll
    for (int q = 0; q < XN; ++q) {
      const int u = tid + 256 * q;
      if (XU % 256 == 0 || u < XU) *(XUnit*)(xs + u * (CIS == 16 ? 8 : 16)) = px[q];
    }
#pragma unroll
    for (int q = 0; q < GN; ++q) {
      const int u = tid + 256 * q;
      if (GU % 256 == 0 || u < GU) *(GUnit*)(gs + u * (COS == 16 ? 8 : 16)) = pg[q];
    }
    if (tile + (int)gridDim.x < ntiles) fetch(tile + gridDim.x);
    __syncthreads();
    // X row (wave, y), tap (dz, dy, dx): G row (wave + 2 - dz, y + 2 - dy) of the stage
    if constexpr (NARROW) {
      // one G plane (dz) at a time, so that nine accumulators are in use beside the sums; the next plane's rows
      // are read during the products
      bf16x8 a[WTY + 2], nxt[WTY + 2];
      auto rows = [&](int dz) {
#pragma unroll
        for (int r = 0; r < WTY + 2; ++r) nxt[r] = read_row_tr(gs + ((wave + 2 - dz) * (WTY + 2) + r) * WTX * 16, lane);
      };
      rows(0);
#pragma unroll
      for (int dz = 0; dz < 3; ++dz) {
        __builtin_amdgcn_sched_barrier(0);  // not two planes ahead: the registers are full
#pragma unroll
        for (int r = 0; r < WTY + 2; ++r) a[r] = nxt[r];
        if (dz < 2) rows(dz + 1);
        f32x4 part[10];
#pragma unroll
        for (int t = 0; t < 10; ++t) part[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int y = 0; y < WTY; ++y) {
          bf16x8 b[3];
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) b[dx] = read_row_tr(xs + ((wave * WTY + y) * (WTX + 2) + dx) * 16, lane);
#pragma unroll
          for (int t = 0; t < 9; ++t) part[t] = mma(a[y + 2 - t / 3], b[t % 3], part[t]);
          if (dz == 1) {  // biases, as below
            const __bf16 one = (__bf16)(y0 + y < g.ny && z0 + wave < g.nz ? 1.0f : 0.0f);
            part[9] = mma(a[y + 1], bf16x8{one, one, one, one, one, one, one, one}, part[9]);
          }
        }
#pragma unroll
        for (int t = 0; t < (dz == 1 ? 10 : 9); ++t)
#pragma unroll
          for (int r = 0; r < KEEP; ++r) acc[t < 9 ? 9 * dz + t : 27][r] += part[t][r];
      }
    } else {
      bf16x8 a[3][WTY + 2];
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int r = 0; r < 2; ++r) a[dz][r] = read_row_tr(gs + ((wave + 2 - dz) * (WTY + 2) + r) * WTX * 16, lane);
#pragma unroll
      for (int y = 0; y < WTY; ++y) {
        bf16x8 b[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) b[dx] = read_row_tr(xs + ((wave * WTY + y) * (WTX + 2) + dx) * 16, lane);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
          a[dz][y + 2] = read_row_tr(gs + ((wave + 2 - dz) * (WTY + 2) + y + 2) * WTX * 16, lane);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
              const int t = 9 * dz + 3 * dy + dx;
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[dz][y + 2 - dy], b[dx], acc[t], 0, 0, 0);
            }
        // biases: the tile's own G rows (dz = dy = 1) times one, times zero for a row beyond the grid
        const __bf16 one = (__bf16)(y0 + y < g.ny && z0 + wave < g.nz ? 1.0f : 0.0f);
        const bf16x8 ones = {one, one, one, one, one, one, one, one};
        acc[27] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][y + 1], ones, acc[27], 0, 0, 0);
      }
    }
  }
  // add the four waves in a fixed order
  float* red = (float*)st;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if (wave == w) {
#pragma unroll
      for (int t = 0; t < WACC; ++t) {
        f32x4* p = (f32x4*)(red + (t * 65 + lane) * 4);  // 65: taps a bank apart
        *p = w == 0 ? acc[t] : *p + acc[t];
      }
    }
  }
  __syncthreads();
  float* row = part + (int64_t)blockIdx.x * WG_PARTS;
  for (int j = tid; j < COS * CIS * 27 + COS; j += 256) {
    const int t = j < COS * CIS * 27 ? j % 27 : 27;
    const int co = j < COS * CIS * 27 ? j / (27 * CIS) : j - COS * CIS * 27;
    const int ci = j < COS * CIS * 27 ? (j / 27) % CIS : 0;
    row[j] = red[CIS == 2 ? (t * 65 + co) * 4 + ci : (t * 65 + (co >> 2) * 16 + ci) * 4 + (co & 3)];
  }
}

// grad[j] (+)= sum over the partial rows, FP64 in a fixed order: a workgroup takes 64 columns, its 16
// waves every 16th row each: 5.5 us for 256 rows of 6928 columns (268 us for 1024 rows with each column's
// rows in one thread's chain).
__global__ __launch_bounds__(1024) void wgrad_reduce(const float* __restrict__ part, int rows, int count,
                                                     float* __restrict__ grad, int accumulate) {
  __shared__ double red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (j < count) {
#pragma unroll 4
    for (int r = wave; r < rows; r += 16) s += part[(int64_t)r * WG_PARTS + j];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && j < count) {
#pragma unroll
    for (int w = 1; w < 16; ++w) s += red[w][lane];
    grad[j] = accumulate ? (float)((double)grad[j] + s) : (float)s;
  }
}

// ------------------------------------------------------------------------------------------
// inputs, loss, optimiser, weight packing

// sum of squares of u (and q) into sc[0], sc[1] (fixed order: per-block partials then one block)
template <typename T>
__global__ __launch_bounds__(256) void sumsq_partial(const T* __restrict__ a, const T* __restrict__ b, int64_t n,
                                                     double* part) {
  __shared__ double red[2][4];
  double s0 = 0, s1 = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double x = (double)a[i];
    s0 = fma(x, x, s0);
    if (b) { const double y = (double)b[i]; s1 = fma(y, y, s1); }
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = s0; red[1][threadIdx.x >> 6] = s1; }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    part[2 * blockIdx.x + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// The sums of the reductions' per-block partials below run in one wave: 64 strided chains, then a fixed
// butterfly (5 us; one thread's chain over the 1024 partials took 92 us for the scales and 58 us for
// the loss, 13 % of a 256^3 forward pass).

// sc[0] = 1/rms(u), sc[1] = 1/rms(q) (1 where the rms is 0), sc[2] = output scale tau*rms(u)*out_scale
__global__ __launch_bounds__(64) void scales_final(const double* __restrict__ part, int blocks, int64_t n, double tau,
                                                   double out_scale, double* sc) {
  double s0 = 0, s1 = 0;
#pragma unroll 8
  for (int i = threadIdx.x; i < blocks; i += 64) {
    const double2 p = ((const double2*)part)[i];
    s0 += p.x;
    s1 += p.y;
  }
  s0 = wave_sum(s0);
  s1 = wave_sum(s1);
  if (threadIdx.x != 0) return;
  const double ru = sqrt(s0 / (double)n), rq = sqrt(s1 / (double)n);
  sc[0] = ru > 0 ? 1.0 / ru : 1.0;
  sc[1] = rq > 0 ? 1.0 / rq : 1.0;
  sc[2] = tau * (ru > 0 ? ru : 1.0) * out_scale;
  sc[3] = 1.0;
}

// x0[v] = (bf16(u * sc0), bf16(q * sc1)): the product is formed in FP64, rounded to fp32, then bf16
template <typename T>
__global__ __launch_bounds__(256) void prep_input(const T* __restrict__ u, const T* __restrict__ q, int64_t n,
                                                  const double* __restrict__ sc, uint32_t* __restrict__ x0) {
  const double a = sc[0], b = sc[1];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const uint32_t c0 = f32_to_bf16((float)((double)u[i] * a));
    const uint32_t c1 = q ? f32_to_bf16((float)((double)q[i] * b)) : 0u;
    x0[i] = c0 | (c1 << 16);
  }
}

// loss partials and output gradient: t = du / sc2, diff = o - t, g = 2 diff / total (fp32; it is
// smoothed by the adjoint of the output filter and rounded to bf16 afterwards)
__global__ __launch_bounds__(256) void mse_grad(const float* __restrict__ o, const float* __restrict__ du, int64_t n,
                                                const double* __restrict__ sc, double inv_total,
                                                float* __restrict__ gout, double* part) {
  __shared__ double red[4];
  const double s = sc[2];
  double acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double d = (double)o[i] - (double)du[i] / s;
    acc = fma(d, d, acc);
    gout[i] = (float)(2.0 * d * inv_total);
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// One pass of the separable binomial low-pass [1/4, 1/2, 1/4] along x, then y, then z (zero
// fill outside a Dirichlet box, wrap-around on a periodic one).  A workgroup owns a 64 x 16
// column of outputs and marches through a chunk of z-planes: each input plane is staged with its
// one-point x and y halo in a double-buffered LDS tile (the next plane is fetched into registers
// while the current one is filtered), the x- and y-passes run from LDS, and the z-pass keeps the
// xy-filtered values of the two previous planes in registers.
constexpr int SMX = 64, SMY = 16, SMR = SMY + 2, SMROWS = (SMR + 3) / 4;

__global__ __launch_bounds__(256) void smooth3(const float* __restrict__ src, float* __restrict__ dst, Grid3 g,
                                               int zc) {
  __shared__ float t[2][SMR][SMX + 2];
  const int tid = threadIdx.x, lx = tid & 63, ly = tid >> 6;
  const int tx = (g.nx + SMX - 1) / SMX, ty = (g.ny + SMY - 1) / SMY;
  int b = blockIdx.x;
  const int x0 = (b % tx) * SMX;
  b /= tx;
  const int y0 = (b % ty) * SMY;
  const int z0 = (b / ty) * zc;
  const int z1 = min(z0 + zc, g.nz);
  const int nplanes = z1 - z0 + 2;  // the chunk plus one halo plane on each side
  const int64_t plane = (int64_t)g.nx * g.ny;
  // wrapped (periodic) or range-checked (Dirichlet) index along one axis; -1 = outside
  auto fold = [&](int i, int n) -> int {
    if (g.periodic) return ((i % n) + n) % n;
    return (i >= 0 && i < n) ? i : -1;
  };
  // staged points this thread loads: its column x0 + lx on rows ly, ly + 4, ... of the tile, and
  // for the first 2 SMR threads one halo column point (left for tid < SMR, right otherwise)
  const int cx = fold(x0 + lx, g.nx);
  int64_t rowoff[SMROWS];
#pragma unroll
  for (int i = 0; i < SMROWS; ++i) {
    const int r = ly + 4 * i;
    const int gy = r < SMR ? fold(y0 + r - 1, g.ny) : -1;
    rowoff[i] = (gy < 0 || cx < 0) ? -1 : (int64_t)gy * g.nx + cx;
  }
  const bool halo = tid < 2 * SMR;
  const int hr = tid % SMR, hc = tid < SMR ? 0 : SMX + 1;
  int64_t hoff = -1;
  if (halo) {
    const int gy = fold(y0 + hr - 1, g.ny), gx = fold(x0 + (hc == 0 ? -1 : SMX), g.nx);
    hoff = (gy < 0 || gx < 0) ? -1 : (int64_t)gy * g.nx + gx;
  }
  float pm[SMROWS], ph = 0.f;
  auto fetch = [&](int k) {
    const int gz = fold(z0 - 1 + k, g.nz);
    const float* sp = src + (int64_t)(gz < 0 ? 0 : gz) * plane;
#pragma unroll
    for (int i = 0; i < SMROWS; ++i) pm[i] = (gz >= 0 && rowoff[i] >= 0) ? sp[rowoff[i]] : 0.f;
    if (halo) ph = (gz >= 0 && hoff >= 0) ? sp[hoff] : 0.f;
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int i = 0; i < SMROWS; ++i)
      if (ly + 4 * i < SMR) t[buf][ly + 4 * i][lx + 1] = pm[i];
    if (halo) t[buf][hr][hc] = ph;
  };
  // output rows 4 ly .. 4 ly + 3 of the column; their xy-filtered values on the two previous planes
  float s0[4] = {0.f, 0.f, 0.f, 0.f}, s1[4] = {0.f, 0.f, 0.f, 0.f};
  const int gxo = x0 + lx;
  fetch(0);
  for (int k = 0; k < nplanes; ++k) {
    const int buf = k & 1;
    stash(buf);
    if (k + 1 < nplanes) fetch(k + 1);
    __syncthreads();
    float xr[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const float* row = &t[buf][4 * ly + i][lx];
      xr[i] = 0.25f * row[0] + 0.5f * row[1] + 0.25f * row[2];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float s2 = 0.25f * xr[j] + 0.5f * xr[j + 1] + 0.25f * xr[j + 2];
      const int gy = y0 + 4 * ly + j;
      if (k >= 2 && gxo < g.nx && gy < g.ny)
        dst[(int64_t)(z0 + k - 2) * plane + (int64_t)gy * g.nx + gxo] = 0.25f * s0[j] + 0.5f * s1[j] + 0.25f * s2;
      s0[j] = s1[j];
      s1[j] = s2;
    }
  }
}

// z-planes per workgroup of the low-pass: enough workgroups to fill the chip several times over
static int smooth_zchunk(Grid3 g) {
  const int64_t cols = (int64_t)((g.nx + SMX - 1) / SMX) * ((g.ny + SMY - 1) / SMY);
  return (int)std::max<int64_t>(8, std::min<int64_t>(64, (int64_t)g.nz * cols / 8192));
}

__global__ __launch_bounds__(256) void f32_to_bf16_kernel(const float* __restrict__ src, uint16_t* __restrict__ dst,
                                                          int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    dst[i] = f32_to_bf16(src[i]);
}

__global__ __launch_bounds__(64) void loss_final(const double* __restrict__ part, int blocks, double inv_total,
                                                 double* loss_acc, int accumulate) {
  double s = 0;
#pragma unroll 8
  for (int i = threadIdx.x; i < blocks; i += 64) s += part[i];
  s = wave_sum(s);
  if (threadIdx.x == 0) loss_acc[0] = (accumulate ? loss_acc[0] : 0.0) + s * inv_total;
}

// Adam (Kingma & Ba 2015) on the FP32 master weights; t is the 1-based step
__global__ __launch_bounds__(256) void adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                                            const float* __restrict__ g, int n, int t, float lr, float b1, float b2,
                                            float eps) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / (1.0f - powf(b1, (float)t));
  const float vh = vi / (1.0f - powf(b2, (float)t));
  w[i] = w[i] - lr * mh / (sqrtf(vh) + eps);
}

// Packed A operands of every layer, one wave per (K-step blockIdx.x, layer blockIdx.y, direction
// blockIdx.z): one launch for the eight that took 25 us each with a wave per layer.  Forward (z = 0):
// A[m][k] = W[m][ci][tap] with tap = tap16(s, k >> 4), ci = k & 15 (zero outside the layer's channels
// and for the padding partners of steps 12-14; one row per tap for the last layer).  Backward data (z = 1): the transposed convolution's
// weights W'[ci][co][tap] = W[co][ci][26 - tap], M = ci, K = (tap, co).
// Lane layout of v_mfma_f32_16x16x32_bf16 A: lane holds row (lane & 15), k = 8 (lane >> 4) + j.
__global__ __launch_bounds__(64) void pack_weights(const float* __restrict__ w, uint16_t* __restrict__ wf,
                                                   uint16_t* __restrict__ wb, float* __restrict__ bias) {
  const int lane = threadIdx.x, s = blockIdx.x, l = blockIdx.y, flip = blockIdx.z;
  const int ci_n = flip ? COUT[l] : CIN[l];   // K-channel count of this convolution
  const int m_n = flip ? CIN[l] : COUT[l];    // output channels
  const float* W = w + woff(l);
  uint16_t* out = (flip ? wb : wf) + l * PACK;
  const int mrow = lane & 15, grp = lane >> 4;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float val = 0.f;
    if (!flip && m_n == 1) {
      // last layer: row 4 dz + dy, k = 8 grp + j -> dx grp / 2 (s = 0) or 2 (s = 1), channel 8 (grp % 2) + j
      const int dz = mrow >> 2, dy = mrow & 3, dx = s == 0 ? grp >> 1 : 2;
      if (dz < 3 && dy < 3 && (s == 0 || (s == 1 && grp < 2)))
        val = W[((grp & 1) * 8 + j) * 27 + 9 * dz + 3 * dy + dx];
    } else if (ci_n < 16) {
      // one or two K channels: k = 8 grp + j -> tap (32 s + k) / ci_n, channel j % ci_n (ci_n steps)
      const int tap = (32 * s + 8 * grp + j) / ci_n, kc = j % ci_n;
      if (s < ci_n && tap < 27 && mrow < m_n)
        val = flip ? W[(kc * CIN[l] + mrow) * 27 + (26 - tap)] : W[(mrow * CIN[l] + kc) * 27 + tap];
    } else {
      const int half = grp >> 1;
      const int tap = tap16(s, half);
      const int kc = (grp & 1) * 8 + j;
      if (!pad16(s, half) && mrow < m_n && kc < ci_n) {
        if (!flip) val = W[(mrow * CIN[l] + kc) * 27 + tap];
        else val = W[(kc * CIN[l] + mrow) * 27 + (26 - tap)];
      }
    }
    out[(s * 64 + lane) * 8 + j] = f32_to_bf16(val);
  }
  if (!flip && s == 0 && lane < 16) bias[l * 16 + lane] = lane < COUT[l] ? w[boff(l) + lane] : 0.f;
}

}  // namespace net
}  // namespace tbs

// ==========================================================================================
// host side

using namespace tbs;
using namespace tbs::net;

namespace {

// weight-gradient workgroups (= partial rows), as many as the chip holds at once: two per CU, or one for
// 16 -> 16 channels, whose prefetch registers fill a SIMD
constexpr int kPartBlocks = 512;
constexpr int kPartBlocks16 = 256;
constexpr int kRedBlocks = 1024;    // blocks of the sum-of-squares / loss reductions

struct NetWs {
  // parameter block
  float* master; float* m; float* v; float* grad;
  uint16_t* wf;     // packed forward A operands, NL x PACK
  uint16_t* wb;     // packed backward-data A operands, NL x PACK
  float* bias;      // NL x 16
  double* sc;       // scales: 1/rms u, 1/rms q, output scale; loss accumulator at sc[4]
  double* red;      // reduction partials (2 x kRedBlocks)
  float* part;      // weight-gradient partial rows kPartBlocks x WG_PARTS
  // activations (per sample)
  uint32_t* x0;     // N x 2 bf16
  uint16_t* y[3];   // N x 16 bf16 (inference uses y[0], y[1] as ping-pong)
  float* z[3];      // N x 16 f32 (training)
  uint16_t* gz[2];  // N x 16 bf16 (training: gradients of pre-activations)
  uint16_t* gout;   // N bf16 (training)
  float* o;         // N f32 (network output / guess)
};

size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t layout(NetWs* L, char* base, int64_t N, int training) {
  size_t o = 0;
  auto take = [&](size_t bytes) { char* p = base ? base + o : nullptr; o += a256(bytes); return p; };
  const size_t P = TBS_NET_PARAMS;
  NetWs w{};
  w.master = (float*)take(P * 4); w.m = (float*)take(P * 4); w.v = (float*)take(P * 4); w.grad = (float*)take(P * 4);
  w.wf = (uint16_t*)take((size_t)NL * PACK * 2); w.wb = (uint16_t*)take((size_t)NL * PACK * 2);
  w.bias = (float*)take(NL * 16 * 4);
  w.sc = (double*)take(8 * 8);
  w.red = (double*)take(2 * kRedBlocks * 8);
  w.part = (float*)take(training ? (size_t)kPartBlocks * WG_PARTS * 4 : 0);
  w.x0 = (uint32_t*)take((size_t)N * 4);
  w.y[0] = (uint16_t*)take((size_t)N * 32);
  w.y[1] = (uint16_t*)take((size_t)N * 32);
  w.y[2] = (uint16_t*)take(training ? (size_t)N * 32 : 0);
  for (int i = 0; i < 3; ++i) w.z[i] = (float*)take(training ? (size_t)N * 64 : 0);
  for (int i = 0; i < 2; ++i) w.gz[i] = (uint16_t*)take(training ? (size_t)N * 32 : 0);
  w.gout = (uint16_t*)take(training ? (size_t)N * 2 : 0);
  w.o = (float*)take((size_t)N * 4);
  if (L) *L = w;
  return o;
}

thread_local char g_err[256];
int err(int code, const char* msg) {
  snprintf(g_err, sizeof(g_err), "%s", msg);
  return code;
}

}  // namespace

struct tbs_net {
  hipStream_t st;
  char* ws;
  size_t ws_bytes;
  int64_t grid[3];
  int batch, training;
  NetWs w;
  int step;           // Adam step count
  double out_scale;
  double lr;
  int weights_set;
};

#define NCHK(expr)                                                        \
  do {                                                                    \
    hipError_t e_ = (expr);                                               \
    if (e_ != hipSuccess) return err(TBS_E_HIP, hipGetErrorString(e_));   \
  } while (0)

static bool aligned256(const void* p) { return p && ((uintptr_t)p & 255u) == 0; }

extern "C" int tbs_net_create(tbs_net** out, void* stream) {
  if (!out) return TBS_E_INVAL;
  tbs_net* n = new (std::nothrow) tbs_net();
  if (!n) return TBS_E_INVAL;
  n->st = (hipStream_t)stream;
  n->out_scale = 1.0;
  n->lr = 1e-3;
  *out = n;
  return TBS_OK;
}

extern "C" void tbs_net_destroy(tbs_net* n) { delete n; }

extern "C" size_t tbs_net_workspace_bytes(const int64_t grid[3], int batch, int training) {
  if (!grid || grid[0] < 1 || grid[1] < 1 || grid[2] < 1 || batch < 1) return 0;
  return layout(nullptr, nullptr, grid[0] * grid[1] * grid[2], training);
}

static int repack(tbs_net* n) {
  hipLaunchKernelGGL(pack_weights, dim3(NSTEP, NL, 2), dim3(64), 0, n->st, (const float*)n->w.master, n->w.wf,
                     n->w.wb, n->w.bias);
  NCHK(hipGetLastError());
  return TBS_OK;
}

extern "C" int tbs_net_bind_workspace(tbs_net* n, const int64_t grid[3], int batch, int training, void* p,
                                      size_t bytes) {
  if (!n || !grid || batch < 1) return TBS_E_INVAL;
  if (!aligned256(p)) return TBS_E_INVAL;
  const size_t need = tbs_net_workspace_bytes(grid, batch, training);
  if (need == 0 || bytes < need) return TBS_E_NOMEM;
  const bool keep = n->ws && n->weights_set;
  float host_params[TBS_NET_PARAMS];
  float host_m[TBS_NET_PARAMS], host_v[TBS_NET_PARAMS];
  if (keep) {
    // carry the parameter block (weights and Adam moments) over to the new workspace
    NCHK(hipMemcpyAsync(host_params, n->w.master, sizeof(host_params), hipMemcpyDeviceToHost, n->st));
    NCHK(hipMemcpyAsync(host_m, n->w.m, sizeof(host_m), hipMemcpyDeviceToHost, n->st));
    NCHK(hipMemcpyAsync(host_v, n->w.v, sizeof(host_v), hipMemcpyDeviceToHost, n->st));
    NCHK(hipStreamSynchronize(n->st));
  }
  n->ws = (char*)p;
  n->ws_bytes = bytes;
  for (int d = 0; d < 3; ++d) n->grid[d] = grid[d];
  n->batch = batch;
  n->training = training;
  layout(&n->w, n->ws, grid[0] * grid[1] * grid[2], training);
  if (keep) {
    NCHK(hipMemcpyAsync(n->w.master, host_params, sizeof(host_params), hipMemcpyHostToDevice, n->st));
    NCHK(hipMemcpyAsync(n->w.m, host_m, sizeof(host_m), hipMemcpyHostToDevice, n->st));
    NCHK(hipMemcpyAsync(n->w.v, host_v, sizeof(host_v), hipMemcpyHostToDevice, n->st));
    int rc = repack(n);
    if (rc) return rc;
    NCHK(hipStreamSynchronize(n->st));
  } else {
    n->weights_set = 0;
  }
  return TBS_OK;
}

extern "C" int tbs_net_set_weights(tbs_net* n, const float* host, size_t count) {
  if (!n || !host || count != TBS_NET_PARAMS) return TBS_E_INVAL;
  if (!n->ws) return TBS_E_NOMEM;
  for (size_t i = 0; i < count; ++i)
    if (!std::isfinite(host[i])) return err(TBS_E_INVAL, "non-finite weight");
  NCHK(hipMemcpyAsync(n->w.master, host, count * 4, hipMemcpyHostToDevice, n->st));
  NCHK(hipMemsetAsync(n->w.m, 0, count * 4, n->st));
  NCHK(hipMemsetAsync(n->w.v, 0, count * 4, n->st));
  n->step = 0;
  int rc = repack(n);
  if (rc) return rc;
  NCHK(hipStreamSynchronize(n->st));
  n->weights_set = 1;
  return TBS_OK;
}

extern "C" int tbs_net_get_weights(const tbs_net* n, float* host, size_t count) {
  if (!n || !host || count != TBS_NET_PARAMS) return TBS_E_INVAL;
  if (!n->ws || !n->weights_set) return TBS_E_STATE;
  NCHK(hipMemcpyAsync(host, n->w.master, count * 4, hipMemcpyDeviceToHost, n->st));
  NCHK(hipStreamSynchronize(n->st));
  return TBS_OK;
}

extern "C" int tbs_net_set_hparams(tbs_net* n, double out_scale, double lr) {
  if (!n || !(out_scale > 0) || !(lr > 0) || !std::isfinite(out_scale) || !std::isfinite(lr)) return TBS_E_INVAL;
  n->out_scale = out_scale;
  n->lr = lr;
  return TBS_OK;
}

static int check_grid(const tbs_net* n, const int64_t grid[3]) {
  if (!n->ws) return err(TBS_E_NOMEM, "no workspace bound");
  if (!n->weights_set) return err(TBS_E_STATE, "weights not set");
  for (int d = 0; d < 3; ++d)
    if (grid[d] != n->grid[d]) return err(TBS_E_INVAL, "grid differs from the bound workspace");
  return TBS_OK;
}

// one workgroup per (32 x 8 column, z-chunk)
static int conv_blocks(const int64_t grid[3], int wgs = 2048) {
  const Grid3 g{(int)grid[0], (int)grid[1], (int)grid[2], 0};
  const ConvGeo c = conv_geo(g, wgs);
  return c.tx * c.ty * c.nch;
}

static int smooth(tbs_net* n, const float* src, float* tmp, float* dst, Grid3 g);

// forward of one sample; x0 already prepared.  keep = training (store z and all y, and leave the
// network output unscaled for the loss); otherwise the output is the guess du = o * sc[2].  It goes to
// `out` (w.o or the caller's array).
static int forward_layers(tbs_net* n, Grid3 g, int keep, float* out) {
  const int64_t grid[3] = {g.nx, g.ny, g.nz};
  const int nb = conv_blocks(grid);
  NetWs& w = n->w;
  uint16_t* y2 = keep ? w.y[2] : w.y[0];
#define GELU_LAYER(CI, IN, L, Y)                                                                                       \
  if (keep)                                                                                                            \
    hipLaunchKernelGGL((conv_mfma<CI, 16, EPI_GELU_Z>), dim3(nb), dim3(256), 0, n->st, (const uint16_t*)(IN),          \
                       w.wf + (L) * PACK, w.bias + 16 * (L), g, w.z[L], Y, nullptr, nullptr);                          \
  else                                                                                                                 \
    hipLaunchKernelGGL((conv_mfma<CI, 16, EPI_GELU>), dim3(nb), dim3(256), 0, n->st, (const uint16_t*)(IN),            \
                       w.wf + (L) * PACK, w.bias + 16 * (L), g, nullptr, Y, nullptr, nullptr)
  GELU_LAYER(2, w.x0, 0, w.y[0]);
  GELU_LAYER(16, w.y[0], 1, w.y[1]);
  GELU_LAYER(16, w.y[1], 2, y2);
#undef GELU_LAYER
  hipLaunchKernelGGL(conv_last, dim3(conv_blocks(grid, kLastWgs)), dim3(256), 0, n->st, (const uint16_t*)y2,
                     w.wf + 3 * PACK, w.bias + 48, g, w.o, (const double*)(w.sc + (keep ? 3 : 2)));
  NCHK(hipGetLastError());
  // output low-pass (linear, so it commutes with the output scale); scratch: a free activation buffer
  return smooth(n, w.o, keep ? (float*)w.gz[0] : (float*)w.y[1], out, g);
}

// dst <- B^2 src with B = Bx By Bz the binomial low-pass; tmp is scratch of N floats, dst may be src
static int smooth(tbs_net* n, const float* src, float* tmp, float* dst, Grid3 g) {
  static_assert(SMOOTH_PASSES == 2, "through tmp");
  const int zc = smooth_zchunk(g);
  const int sblocks = ((g.nx + SMX - 1) / SMX) * ((g.ny + SMY - 1) / SMY) * ((g.nz + zc - 1) / zc);
  hipLaunchKernelGGL(smooth3, dim3(sblocks), dim3(256), 0, n->st, src, tmp, g, zc);
  hipLaunchKernelGGL(smooth3, dim3(sblocks), dim3(256), 0, n->st, (const float*)tmp, dst, g, zc);
  NCHK(hipGetLastError());
  return TBS_OK;
}

template <typename T>
static int prepare(tbs_net* n, const T* u, const T* q, int64_t N, double tau, double out_scale) {
  NetWs& w = n->w;
  hipLaunchKernelGGL(sumsq_partial<T>, dim3(kRedBlocks), dim3(256), 0, n->st, u, q, N, w.red);
  hipLaunchKernelGGL(scales_final, dim3(1), dim3(64), 0, n->st, (const double*)w.red, kRedBlocks, N, tau, out_scale,
                     w.sc);
  hipLaunchKernelGGL(prep_input<T>, dim3(2048), dim3(256), 0, n->st, u, q, N, (const double*)w.sc, w.x0);
  NCHK(hipGetLastError());
  return TBS_OK;
}

extern "C" int tbs_net_forward(tbs_net* n, const void* u, const void* q, int dtype, float* du, int periodic,
                               double tau) {
  if (!n || !aligned256(u) || !aligned256(du) || (q && !aligned256(q))) return TBS_E_INVAL;
  if (dtype != TBS_F64 && dtype != TBS_F32) return TBS_E_INVAL;
  if (!(tau > 0)) return TBS_E_INVAL;
  int rc = check_grid(n, n->grid);
  if (rc) return rc;
  const int64_t N = n->grid[0] * n->grid[1] * n->grid[2];
  Grid3 g{(int)n->grid[0], (int)n->grid[1], (int)n->grid[2], periodic ? 1 : 0};
  rc = dtype == TBS_F64 ? prepare(n, (const double*)u, (const double*)q, N, tau, n->out_scale)
                        : prepare(n, (const float*)u, (const float*)q, N, tau, n->out_scale);
  if (rc) return rc;
  return forward_layers(n, g, 0, du);
}

int tbs_net_guess_internal(tbs_net* n, const int64_t grid[3], int periodic, double tau, hipStream_t st,
                           const double* u_prev, const double* q, const float** du_out) {
  if (!n) return TBS_E_INVAL;
  int rc = check_grid(n, grid);
  if (rc) return rc;
  if (n->st != st) return err(TBS_E_INVAL, "network and solver must share one stream");
  const int64_t N = grid[0] * grid[1] * grid[2];
  Grid3 g{(int)grid[0], (int)grid[1], (int)grid[2], periodic ? 1 : 0};
  rc = prepare(n, u_prev, q, N, tau, n->out_scale);
  if (rc) return rc;
  rc = forward_layers(n, g, 0, n->w.o);
  if (rc) return rc;
  *du_out = n->w.o;
  return TBS_OK;
}

extern "C" int tbs_net_train_step(tbs_net* n, const float* u, const float* q, const float* du_t, int batch,
                                  int periodic, double tau, float* loss_out) {
  if (!n || !aligned256(u) || !aligned256(du_t) || (q && !aligned256(q)) || batch < 1) return TBS_E_INVAL;
  if (!(tau > 0)) return TBS_E_INVAL;
  int rc = check_grid(n, n->grid);
  if (rc) return rc;
  if (!n->training) return err(TBS_E_STATE, "workspace bound without training buffers");
  const int64_t N = n->grid[0] * n->grid[1] * n->grid[2];
  Grid3 g{(int)n->grid[0], (int)n->grid[1], (int)n->grid[2], periodic ? 1 : 0};
  NetWs& w = n->w;
  const int nb = conv_blocks(n->grid);
  const double inv_total = 1.0 / ((double)N * batch);
  const int wblocks = kPartBlocks;
  for (int b = 0; b < batch; ++b) {
    const float* ub = u + (size_t)b * N;
    const float* qb = q ? q + (size_t)b * N : nullptr;
    const float* tb = du_t + (size_t)b * N;
    rc = prepare(n, ub, qb, N, tau, n->out_scale);
    if (rc) return rc;
    rc = forward_layers(n, g, 1, w.o);
    if (rc) return rc;
    float* gtmp = (float*)w.gz[0];
    hipLaunchKernelGGL(mse_grad, dim3(kRedBlocks), dim3(256), 0, n->st, (const float*)w.o, tb, N,
                       (const double*)w.sc, inv_total, gtmp, w.red);
    rc = smooth(n, gtmp, (float*)w.gz[1], gtmp, g);  // adjoint of the output filter (it is symmetric)
    if (rc) return rc;
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(2048), dim3(256), 0, n->st, (const float*)gtmp, w.gout, N);
    hipLaunchKernelGGL(loss_final, dim3(1), dim3(64), 0, n->st, (const double*)w.red, kRedBlocks, inv_total,
                       w.sc + 4, b > 0);
    const int acc = b > 0;
    // layer 4: dW4 = sum y3 (x) g ; dZ3 = convT(g, W4) * GELU'(z3)
    hipLaunchKernelGGL((wgrad_partial<16, 1>), dim3(wblocks), dim3(256), 0, n->st, (const uint16_t*)w.y[2],
                       (const uint16_t*)w.gout, g, w.part);
    hipLaunchKernelGGL(wgrad_reduce, dim3((16 * 27 + 1 + 63) / 64), dim3(1024), 0, n->st, (const float*)w.part,
                       wblocks, 16 * 27 + 1, w.grad + woff(3), acc);
    hipLaunchKernelGGL((conv_mfma<1, 16, EPI_BWD>), dim3(nb), dim3(256), 0, n->st, (const uint16_t*)w.gout,
                       w.wb + 3 * PACK, nullptr, g, nullptr, w.gz[0], nullptr, (const float*)w.z[2]);
    // layer 3: dW3 = sum y2 (x) dZ3 ; dZ2 = convT(dZ3, W3) * GELU'(z2)
    hipLaunchKernelGGL((wgrad_partial<16, 16>), dim3(kPartBlocks16), dim3(256), 0, n->st, (const uint16_t*)w.y[1],
                       (const uint16_t*)w.gz[0], g, w.part);
    hipLaunchKernelGGL(wgrad_reduce, dim3((16 * 16 * 27 + 16 + 63) / 64), dim3(1024), 0, n->st,
                       (const float*)w.part, kPartBlocks16, 16 * 16 * 27 + 16, w.grad + woff(2), acc);
    hipLaunchKernelGGL((conv_mfma<16, 16, EPI_BWD>), dim3(nb), dim3(256), 0, n->st, (const uint16_t*)w.gz[0],
                       w.wb + 2 * PACK, nullptr, g, nullptr, w.gz[1], nullptr, (const float*)w.z[1]);
    // layer 2: dW2 = sum y1 (x) dZ2 ; dZ1 = convT(dZ2, W2) * GELU'(z1)
    hipLaunchKernelGGL((wgrad_partial<16, 16>), dim3(kPartBlocks16), dim3(256), 0, n->st, (const uint16_t*)w.y[0],
                       (const uint16_t*)w.gz[1], g, w.part);
    hipLaunchKernelGGL(wgrad_reduce, dim3((16 * 16 * 27 + 16 + 63) / 64), dim3(1024), 0, n->st,
                       (const float*)w.part, kPartBlocks16, 16 * 16 * 27 + 16, w.grad + woff(1), acc);
    hipLaunchKernelGGL((conv_mfma<16, 16, EPI_BWD>), dim3(nb), dim3(256), 0, n->st, (const uint16_t*)w.gz[1],
                       w.wb + PACK, nullptr, g, nullptr, w.gz[0], nullptr, (const float*)w.z[0]);
    // layer 1: dW1 = sum x0 (x) dZ1
    hipLaunchKernelGGL((wgrad_partial<2, 16>), dim3(wblocks), dim3(256), 0, n->st, (const uint16_t*)w.x0,
                       (const uint16_t*)w.gz[0], g, w.part);
    hipLaunchKernelGGL(wgrad_reduce, dim3((2 * 16 * 27 + 16 + 63) / 64), dim3(1024), 0, n->st,
                       (const float*)w.part, wblocks, 2 * 16 * 27 + 16, w.grad + woff(0), acc);
    NCHK(hipGetLastError());
  }
  n->step += 1;
  hipLaunchKernelGGL(adam, dim3((TBS_NET_PARAMS + 255) / 256), dim3(256), 0, n->st, w.master, w.m, w.v,
                     (const float*)w.grad, TBS_NET_PARAMS, n->step, (float)n->lr, 0.9f, 0.999f, 1e-8f);
  rc = repack(n);
  if (rc) return rc;
  if (loss_out) {
    double l = 0;
    NCHK(hipMemcpyAsync(&l, w.sc + 4, 8, hipMemcpyDeviceToHost, n->st));
    NCHK(hipStreamSynchronize(n->st));
    *loss_out = (float)l;
  }
  return TBS_OK;
}

// ------------------------------------------------------------------------------------------
// kernel-level probes for parity tests (use the bound workspace's grid)

extern "C" int tbs_net_conv_layer(tbs_net* n, int layer, int mode, const uint16_t* x, const uint16_t* gin,
                                  int periodic, float* out) {
  if (!n || layer < 0 || layer >= NL || mode < 0 || mode > 2 || !aligned256(out)) return TBS_E_INVAL;
  int rc = check_grid(n, n->grid);
  if (rc) return rc;
  Grid3 g{(int)n->grid[0], (int)n->grid[1], (int)n->grid[2], periodic ? 1 : 0};
  const int nb = conv_blocks(n->grid);
  NetWs& w = n->w;
  const int ci = CIN[layer], co = COUT[layer];
  if (mode == 0) {  // forward pre-activation z = conv(x, W) + b, out [voxel][co]
    if (!aligned256(x)) return TBS_E_INVAL;
#define FWD(CI, CO) hipLaunchKernelGGL((conv_mfma<CI, CO, EPI_RAW>), dim3(nb), dim3(256), 0, n->st, x, \
                                       w.wf + layer * PACK, w.bias + layer * 16, g, nullptr, nullptr, out, nullptr)
    if (ci == 2) FWD(2, 16);
    else if (co == 16) FWD(16, 16);
    else
      hipLaunchKernelGGL(conv_last, dim3(conv_blocks(n->grid, kLastWgs)), dim3(256), 0, n->st, x,
                         w.wf + layer * PACK, w.bias + layer * 16, g, out, (const double*)nullptr);
#undef FWD
  } else if (mode == 1) {  // data gradient dx = convT(g, W), out [voxel][ci]
    if (!aligned256(gin)) return TBS_E_INVAL;
#define BWD(CI, CO) hipLaunchKernelGGL((conv_mfma<CI, CO, EPI_RAW>), dim3(nb), dim3(256), 0, n->st, gin, \
                                       w.wb + layer * PACK, nullptr, g, nullptr, nullptr, out, nullptr)
    if (co == 1) BWD(1, 16);
    else if (ci == 2) BWD(16, 2);
    else BWD(16, 16);
#undef BWD
  } else {  // weight gradient: out [co][ci][27] then [co] biases
    if (!n->training) return err(TBS_E_STATE, "weight gradients need a training workspace");
    if (!aligned256(x) || !aligned256(gin)) return TBS_E_INVAL;
    if (ci == 2) hipLaunchKernelGGL((wgrad_partial<2, 16>), dim3(kPartBlocks), dim3(256), 0, n->st, x, gin, g, w.part);
    else if (co == 16) hipLaunchKernelGGL((wgrad_partial<16, 16>), dim3(kPartBlocks16), dim3(256), 0, n->st, x, gin, g, w.part);
    else hipLaunchKernelGGL((wgrad_partial<16, 1>), dim3(kPartBlocks), dim3(256), 0, n->st, x, gin, g, w.part);
    const int cnt = ci * co * 27 + co;
    hipLaunchKernelGGL(wgrad_reduce, dim3((cnt + 63) / 64), dim3(1024), 0, n->st, (const float*)w.part,
                       ci * co == 256 ? kPartBlocks16 : kPartBlocks, cnt, out, 0);
  }
  NCHK(hipGetLastError());
  return TBS_OK;
}

// gradient of the last train step (flat parameter order) for parity tests
extern "C" int tbs_net_get_grad(const tbs_net* n, float* host, size_t count) {
  if (!n || !host || count != TBS_NET_PARAMS) return TBS_E_INVAL;
  if (!n->ws || !n->training) return TBS_E_STATE;
  NCHK(hipMemcpyAsync(host, n->w.grad, count * 4, hipMemcpyDeviceToHost, n->st));
  NCHK(hipStreamSynchronize(n->st));
  return TBS_OK;
}

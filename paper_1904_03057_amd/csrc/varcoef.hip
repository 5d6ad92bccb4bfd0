// Variable-coefficient system operator on gfx950 (Sec. 2.3: D and mu_a expanded in the solution's
// B-spline basis; Sec. 2.4: the domain kernels c_k d_m w^{klm} + c_k m_m f^{klm} of the tensor
// form; Sec. 2.5 strategy (c): computed on the fly):
//
//   F(c)_l = sum_k sum_m c_k (m_m f^{klm} + d_m w^{klm})
//          = int [ mu phi b_l + D (phi_x b_l,x / hx^2 + phi_y b_l,y / hy^2 + phi_z b_l,z / hz^2) ],
//
// phi = sum c_k b_k, mu = sum m_m b_m, D = sum d_m b_m, integrated cell by cell (grid units, the
// operator divided by hx hy hz) with Q = ceil((3n + 1) / 2) Gauss points per cell and axis, which is
// exact for the degree-3n products.  The integrals are evaluated by sum factorisation: the fields
// are interpolated to the Gauss points one axis at a time (z, then y, then x), multiplied there,
// and projected back onto the test functions in the reverse order (x, y, z).  Per cell (= per
// coefficient) this is about 6.7 k multiply-adds for cubic splines, against the (2n+1)^3 products
// of three-index kernels per output.
//
// Execution: a workgroup owns a strip of 64 coefficient columns (64 - 2n output columns and an
// n-column halo on each side) and vc_tile_y output rows, and marches through a z-chunk cell by cell.
// Its waves take the (z-cell, z-point) pairs in turn.  For its z-point a wave marches along y: a ring of
// n+1 rows of the z-interpolated fields (per lane: its column), the y-interpolation, the
// x-interpolation from the n neighbouring lanes (cross-lane shuffles), the point products, the
// x-projection (partial sums handed back to the output lanes by shuffles), and the y-projection into a
// ring of n+1 output rows that it leaves in LDS.  The waves then project the finished z-points, in
// order, onto an LDS accumulator of n+1 output planes (each wave its own rows); a plane is written to
// memory once the z-march has passed it.  Every output sums its terms in one fixed order, so results
// are bitwise reproducible and do not depend on the z-chunks.
//
// What bounds it is the vector ALU (225 instructions per 64 columns, row, y- and z-point for cubic FP32)
// and the halo cells.  The x-axis works on the even and odd parts of the basis under the cell's
// mirror symmetry and takes both points of a mirrored pair from one evaluation (104 + 68 multiply-adds
// and additions per point row instead of 120 + 80), and the point weights and h_d^-2 are folded into
// the projection tables (4 multiplications per point instead of 10).  Splitting a cell's z-points over the
// waves gives four times the waves without more halo cells, and the wave-uniform z-point keeps the
// tables in scalar registers (cubic: 109 vector registers in FP32 and 156 in FP64; 191 and 314 in the
// form it replaces, which gave each wave its own strip of all z-points).  Measured, against that form:
// cubic 192^3 FP32 2.14 against 6.70 ms, FP64 3.66 against 8.35; 400^3 FP32 14.8 against 24.7, FP64 28.6
// against 42.4; quartic 128^3 FP32 3.7 against 21.7; quintic 100^3 FP32 5.1 against 42.0.
#include "common.h"
#include "varcoef.h"

namespace tbs {

template <typename T> __device__ __forceinline__ T vfma(T a, T b, T c);
template <> __device__ __forceinline__ float vfma<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <> __device__ __forceinline__ double vfma<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }

// What a kernel needs of VarcoefArgs.
struct VarcoefGeo {
  int nx, ny, nz, zc;
  int tiles_x, tiles_y, nblocks;
  const void* c;
  const void* d;
  const void* m;
  void* y;
};

template <int N, typename T, int BC>
__global__ __launch_bounds__(64 * kVcWaves) void varcoef_kernel(VarcoefGeo a, VarcoefTab<T> tab) {
  constexpr int Q = (3 * N + 2) / 2;
  constexpr int NB = N + 1;
  constexpr int NP = NB / 2, NE = (NB + 1) / 2;  // pairs (t, n - t); even parts (with the middle B-spline)
  constexpr int QP = Q / 2;                      // pairs (q, Q - 1 - q) of points
  constexpr int H = N / 2;
  constexpr int TXO = 64 - 2 * N;
  constexpr int TY = vc_tile_y(sizeof(T) == 8 ? 0 : 1);
  __shared__ T acc[TY * NB * 64];            // [output row][plane slot][lane]; wave r % kVcWaves owns row r
  __shared__ T rows[kVcWaves][TY][2][64];    // y-projected rows of the waves' current z-points

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bid = xcd_remap(blockIdx.x, a.nblocks);
  const int txi = bid % a.tiles_x;
  const int rest = bid / a.tiles_x;
  const int tyi = rest % a.tiles_y;
  const int czi = rest / a.tiles_y;
  const int x0 = txi * TXO, y0 = tyi * TY, z0 = czi * a.zc;
  const int zc_eff = min(a.zc, a.nz - z0);
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int64_t plane = (int64_t)nx * ny;
  const T* __restrict__ Cc = (const T*)a.c;
  const T* __restrict__ Dc = (const T*)a.d;
  const T* __restrict__ Mc = (const T*)a.m;
  T* __restrict__ Y = (T*)a.y;

  // this lane's coefficient column: c is read there (zero outside a Dirichlet box), mu and D at
  // the nearest column inside (their expansions continue by the edge coefficients)
  const int xp = x0 - N + lane;
  int xcc, xcm;
  bool xok;
  if (BC == BC_PERIODIC) {
    xcc = ((xp % nx) + nx) % nx;
    xcm = xcc;
    xok = true;
  } else {
    xok = xp >= 0 && xp < nx;
    xcc = xok ? xp : 0;
    xcm = min(max(xp, 0), nx - 1);
  }

  for (int r = wave; r < TY; r += kVcWaves)
#pragma unroll
    for (int t = 0; t < NB; ++t) acc[(r * NB + t) * 64 + lane] = (T)0;

  const int jz0 = z0 + H - N, jz1 = z0 + zc_eff + H;  // z-cells whose support meets the chunk
  const int jy0 = y0 + H - N;                        // first y-cell of the strip's rows
  // tasks in the order (z-cell, z-point), kVcWaves at a time
  const int ntask = (jz1 - jz0) * Q;
  for (int task0 = 0; task0 < ntask; task0 += kVcWaves) {
    const int task = task0 + wave;
    if (task < ntask) {
      const int jz = jz0 + task / Q, zq = task % Q;
      // the n+1 coefficient planes of this z-cell
      int64_t pcz[NB], pmz[NB];
      bool zok[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int kz = jz - H + t;
        int kc, km;
        if (BC == BC_PERIODIC) {
          kc = ((kz % nz) + nz) % nz;
          km = kc;
          zok[t] = true;
        } else {
          zok[t] = kz >= 0 && kz < nz;
          kc = zok[t] ? kz : 0;
          km = min(max(kz, 0), nz - 1);
        }
        pcz[t] = (int64_t)kc * plane;
        pmz[t] = (int64_t)km * plane;
      }
      T bzv[NB], bzd[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        bzv[t] = tab.v[zq][t];
        bzd[t] = tab.d[zq][t];
      }
      // fields at (z-point zq, coefficient row ky, this column): c value, c z-derivative, mu, D
      auto load_row = [&](int ky, T* out) {
        int kc, km;
        bool yok;
        if (BC == BC_PERIODIC) {
          kc = ((ky % ny) + ny) % ny;
          km = kc;
          yok = true;
        } else {
          yok = ky >= 0 && ky < ny;
          kc = yok ? ky : 0;
          km = min(max(ky, 0), ny - 1);
        }
        const int64_t oc = (int64_t)kc * nx + xcc, om = (int64_t)km * nx + xcm;
        T cv = (T)0, cd = (T)0, mu = (T)0, dd = (T)0;
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const T c = (yok && xok && zok[t]) ? Cc[pcz[t] + oc] : (T)0;
          cv = vfma(bzv[t], c, cv);
          cd = vfma(bzd[t], c, cd);
          mu = vfma(bzv[t], Mc[pmz[t] + om], mu);
          dd = vfma(bzv[t], Dc[pmz[t] + om], dd);
        }
        out[0] = cv;
        out[1] = cd;
        out[2] = mu;
        out[3] = dd;
      };
      T zr[NB][4];   // ring of coefficient rows jy - H + t
      T ya[NB], yc[NB];  // y-projection ring of output rows jy - H + t (z-value and z-derivative parts)
#pragma unroll
      for (int t = 0; t < N; ++t) load_row(jy0 - H + t, zr[t]);
#pragma unroll
      for (int t = 0; t < NB; ++t) ya[t] = yc[t] = (T)0;
      for (int s = 0; s < TY + N; ++s) {
        const int jy = jy0 + s;
        load_row(jy - H + N, zr[N]);
#pragma unroll 1
        for (int yq = 0; yq < Q; ++yq) {
          // y-interpolation: c (value, y-derivative), c_z, mu, D at (yq, zq) in this column
          T f[5] = {(T)0, (T)0, (T)0, (T)0, (T)0};
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const T bv = tab.v[yq][t], bd = tab.d[yq][t];
            f[0] = vfma(bv, zr[t][0], f[0]);
            f[1] = vfma(bd, zr[t][0], f[1]);
            f[2] = vfma(bv, zr[t][1], f[2]);
            f[3] = vfma(bv, zr[t][2], f[3]);
            f[4] = vfma(bv, zr[t][3], f[4]);
          }
          // the cell of this lane uses columns lane .. lane + n: sums and differences of the pairs
          T fe[NE][5], fo[NP][5];
#pragma unroll
          for (int i = 0; i < 5; ++i) {
            T nb[NB];
            nb[0] = f[i];
#pragma unroll
            for (int t = 1; t < NB; ++t) nb[t] = __shfl_down(f[i], t, 64);
#pragma unroll
            for (int t = 0; t < NP; ++t) {
              fe[t][i] = nb[t] + nb[N - t];
              fo[t][i] = nb[t] - nb[N - t];
            }
            if (NB % 2) fe[NE - 1][i] = nb[NB / 2];
          }
          // even and odd sums of the projections: pa (value and x-derivative tests), pb, pc (value tests)
          T ae[NE], ao[NP], be[NE], bo[NP], ce[NE], co[NP];
#pragma unroll
          for (int t = 0; t < NE; ++t) ae[t] = be[t] = ce[t] = (T)0;
#pragma unroll
          for (int t = 0; t < NP; ++t) ao[t] = bo[t] = co[t] = (T)0;
#pragma unroll
          for (int q = 0; q < QP + Q % 2; ++q) {
            // even (E) and odd (O) parts of phi, phi_y, phi_z, mu, D and (XE, XO) of phi_x
            T E[5], O[5], XE = (T)0, XO = (T)0;
#pragma unroll
            for (int i = 0; i < 5; ++i) {
              E[i] = tab.xve[q][0] * fe[0][i];
#pragma unroll
              for (int t = 1; t < NE; ++t) E[i] = vfma(tab.xve[q][t], fe[t][i], E[i]);
              O[i] = (T)0;
              if (q < QP) {
                O[i] = tab.xvo[q][0] * fo[0][i];
#pragma unroll
                for (int t = 1; t < NP; ++t) O[i] = vfma(tab.xvo[q][t], fo[t][i], O[i]);
              }
            }
#pragma unroll
            for (int t = 0; t < NP; ++t) XO = vfma(tab.xdo[q][t], fo[t][0], XO);
            if (q < QP) {
#pragma unroll
              for (int t = 0; t < NE; ++t) XE = vfma(tab.xde[q][t], fe[t][0], XE);
              // points q and Q - 1 - q
              const T mu0 = E[3] + O[3], mu1 = E[3] - O[3], d0 = E[4] + O[4], d1 = E[4] - O[4];
              const T a0 = mu0 * (E[0] + O[0]), a1 = mu1 * (E[0] - O[0]);
              const T x0 = d0 * (XO + XE), x1 = d1 * (XO - XE);
              const T b0 = d0 * (E[1] + O[1]), b1 = d1 * (E[1] - O[1]);
              const T c0 = d0 * (E[2] + O[2]), c1 = d1 * (E[2] - O[2]);
              const T as = a0 + a1, ad = a0 - a1, xs = x0 + x1, xd = x0 - x1;
              const T bs = b0 + b1, bd = b0 - b1, cs = c0 + c1, cd = c0 - c1;
#pragma unroll
              for (int t = 0; t < NE; ++t) {
                ae[t] = vfma(tab.pve[q][t], as, vfma(tab.pde[q][t], xd, ae[t]));
                be[t] = vfma(tab.pve[q][t], bs, be[t]);
                ce[t] = vfma(tab.pve[q][t], cs, ce[t]);
              }
#pragma unroll
              for (int t = 0; t < NP; ++t) {
                ao[t] = vfma(tab.pvo[q][t], ad, vfma(tab.pdo[q][t], xs, ao[t]));
                bo[t] = vfma(tab.pvo[q][t], bd, bo[t]);
                co[t] = vfma(tab.pvo[q][t], cd, co[t]);
              }
            } else {
              // the middle point: even value parts and odd derivative parts only
              const T a0 = E[3] * E[0], x0 = E[4] * XO, b0 = E[4] * E[1], c0 = E[4] * E[2];
#pragma unroll
              for (int t = 0; t < NE; ++t) {
                ae[t] = vfma(tab.pve[q][t], a0, ae[t]);
                be[t] = vfma(tab.pve[q][t], b0, be[t]);
                ce[t] = vfma(tab.pve[q][t], c0, ce[t]);
              }
#pragma unroll
              for (int t = 0; t < NP; ++t) ao[t] = vfma(tab.pdo[q][t], x0, ao[t]);
            }
          }
          // x-projection: output column o collects partial t of the cell in lane o - t
          auto part = [&](const T* e, const T* o, int t) -> T {
            return t < NP ? e[t] + o[t] : (NB % 2 && t == NB / 2 ? e[NE - 1] : e[N - t] - o[N - t]);
          };
          T ax = part(ae, ao, 0), bx = part(be, bo, 0), cx = part(ce, co, 0);
#pragma unroll
          for (int t = 1; t < NB; ++t) {
            ax += __shfl_up(part(ae, ao, t), t, 64);
            bx += __shfl_up(part(be, bo, t), t, 64);
            cx += __shfl_up(part(ce, co, t), t, 64);
          }
          // y-projection onto the cell's n+1 output rows
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const T bv = tab.pv[yq][t], bd = tab.pdy[yq][t];
            ya[t] = vfma(bv, ax, vfma(bd, bx, ya[t]));
            yc[t] = vfma(bv, cx, yc[t]);
          }
        }
        // output row jy - H has all its y-cells for this z-point
        const int r = jy - H - y0;
        if (r >= 0 && r < TY) {
          rows[wave][r][0][lane] = ya[0];
          rows[wave][r][1][lane] = yc[0];
        }
#pragma unroll
        for (int t = 0; t < N; ++t) {
#pragma unroll
          for (int f = 0; f < 4; ++f) zr[t][f] = zr[t + 1][f];
          ya[t] = ya[t + 1];
          yc[t] = yc[t + 1];
        }
        ya[N] = yc[N] = (T)0;
      }
    }
    __syncthreads();
    // z-projection of the finished z-points, in order; each wave its own rows
    for (int w = 0; w < kVcWaves && task0 + w < ntask; ++w) {
      const int jz = jz0 + (task0 + w) / Q, zq = (task0 + w) % Q;
      for (int r = wave; r < TY; r += kVcWaves) {
        const T va = rows[w][r][0][lane], vc = rows[w][r][1][lane];
#pragma unroll
        for (int t = 0; t < NB; ++t) {
          const int slot = (((jz - H + t) % NB) + NB) % NB;
          T* p = &acc[(r * NB + slot) * 64 + lane];
          *p = vfma(tab.pv[zq][t], va, vfma(tab.pdz[zq][t], vc, *p));
        }
      }
      if (zq == Q - 1) {
        // output plane jz - H has all its z-cells: write it and clear its slot
        const int kz = jz - H;
        const int slot = ((kz % NB) + NB) % NB;
        const bool wcol = lane >= N && lane < N + TXO && xp < nx && kz >= z0 && kz < z0 + zc_eff;
        for (int r = wave; r < TY; r += kVcWaves) {
          T* p = &acc[(r * NB + slot) * 64 + lane];
          if (wcol && y0 + r < ny) Y[(int64_t)kz * plane + (int64_t)(y0 + r) * nx + xp] = *p;
          *p = (T)0;
        }
      }
    }
    __syncthreads();  // the rows are read before the next points overwrite them
  }
}

template <int N, typename T>
static hipError_t launch_nt(const VarcoefArgs& a, int bc, hipStream_t st) {
  constexpr int Q = (3 * N + 2) / 2, NB = N + 1, NP = NB / 2;
  const VarcoefGeo g{a.nx, a.ny, a.nz, a.zc, a.tiles_x, a.tiles_y, a.nblocks, a.c, a.d, a.m, a.y};
  VarcoefTab<T> tab{};
  auto bv = [&](int q, int t) { return a.bv[q * kVcMaxB + t]; };
  auto bd = [&](int q, int t) { return a.bd[q * kVcMaxB + t]; };
  // The kernel sums pairs of coefficients and of point products: the two interpolations before the x-axis
  // carry a factor 1/2 each, so that neither overflows where the result does not, and the x-axis
  // projection of the products of two fields a factor 16 (powers of two: no rounding changes).
  for (int q = 0; q < Q; ++q)
    for (int t = 0; t < NB; ++t) {
      tab.v[q][t] = (T)(0.5 * bv(q, t));
      tab.d[q][t] = (T)(0.5 * bd(q, t));
      tab.pv[q][t] = (T)(a.w[q] * bv(q, t));
      tab.pdy[q][t] = (T)(a.w[q] * bd(q, t) * a.ihy2);
      tab.pdz[q][t] = (T)(a.w[q] * bd(q, t) * a.ihz2);
    }
  for (int q = 0; q < (Q + 1) / 2; ++q) {
    for (int t = 0; t < NP; ++t) {
      const double ve = 0.5 * (bv(q, t) + bv(q, N - t)), vo = 0.5 * (bv(q, t) - bv(q, N - t));
      const double de = 0.5 * (bd(q, t) + bd(q, N - t)), dv = 0.5 * (bd(q, t) - bd(q, N - t));
      tab.xve[q][t] = (T)ve;
      tab.xvo[q][t] = (T)vo;
      tab.xde[q][t] = (T)de;
      tab.xdo[q][t] = (T)dv;
      tab.pve[q][t] = (T)(16.0 * a.w[q] * ve);
      tab.pvo[q][t] = (T)(16.0 * a.w[q] * vo);
      tab.pde[q][t] = (T)(16.0 * a.w[q] * de * a.ihx2);
      tab.pdo[q][t] = (T)(16.0 * a.w[q] * dv * a.ihx2);
    }
    if (NB % 2) {
      tab.xve[q][NP] = (T)bv(q, NP);
      tab.xde[q][NP] = (T)bd(q, NP);
      tab.pve[q][NP] = (T)(16.0 * a.w[q] * bv(q, NP));
      tab.pde[q][NP] = (T)(16.0 * a.w[q] * bd(q, NP) * a.ihx2);
    }
  }
  if (bc == BC_PERIODIC)
    hipLaunchKernelGGL((varcoef_kernel<N, T, BC_PERIODIC>), dim3(a.nblocks), dim3(64 * kVcWaves), 0, st, g, tab);
  else
    hipLaunchKernelGGL((varcoef_kernel<N, T, BC_DIRICHLET>), dim3(a.nblocks), dim3(64 * kVcWaves), 0, st, g, tab);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_t(const VarcoefArgs& a, int n, int bc, hipStream_t st) {
  switch (n) {
    case 1: return launch_nt<1, T>(a, bc, st);
    case 2: return launch_nt<2, T>(a, bc, st);
    case 3: return launch_nt<3, T>(a, bc, st);
    case 4: return launch_nt<4, T>(a, bc, st);
    case 5: return launch_nt<5, T>(a, bc, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_varcoef(const VarcoefArgs& a, int n, int bc, int dt, hipStream_t st) {
  if (dt == 0) return launch_t<double>(a, n, bc, st);
  if (dt == 1) return launch_t<float>(a, n, bc, st);
  return hipErrorInvalidValue;
}

}  // namespace tbs

#pragma once
// End of a one-kernel CG iteration: the FP64 sums p.q, r.q, q.q and r.r over all workgroups and the scalars
// that follow from them.
#include "common.h"

namespace tbs {

// part0..3: the thread's sums; red, last: LDS of the workgroup of NW waves.
template <int NW>
__device__ __forceinline__ void cg_finish(const StencilArgs& a, double part0, double part1, double part2, double part3,
                                          double (*red)[NW], bool* last) {
  static_assert(NW >= 4, "one wave per sum");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  part0 = wave_sum(part0);
  part1 = wave_sum(part1);
  part2 = wave_sum(part2);
  part3 = wave_sum(part3);
  if (lane == 0) { red[0][wv] = part0; red[1][wv] = part1; red[2][wv] = part2; red[3][wv] = part3; }
  __syncthreads();
  if (tid == 0) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) { s0 += red[0][q]; s1 += red[1][q]; s2 += red[2][q]; s3 += red[3][q]; }
    // written through to memory, where the last workgroup reads them whatever XCD it runs on; the
    // ticket is taken once they have arrived
    const double v[4] = {s0, s1, s2, s3};
    double* const p[4] = {a.part0, a.part1, a.part2, a.part3};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      __hip_atomic_store(p[q] + blockIdx.x, v[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    *last = __hip_atomic_fetch_add(&a.scal->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x;
  }
  // The last workgroup to finish reduces the partial sums (wave q the q-th of p.q, r.q, q.q, r.r: 1024
  // strided chains, then a binary tree, the order of the finalize kernel) and forms the scalars, which
  // saves a launch per iteration: 22.4 against 23.6 us per iteration at 32^3 (FP64), where the
  // wait for its stores, the ticket and the loads take 4 us against 5 for the launch.
  __syncthreads();
  if (!*last) return;
  if (wv < 4) {
    const double* p = wv == 0 ? a.part0 : (wv == 1 ? a.part1 : (wv == 2 ? a.part2 : a.part3));
    const int count = gridDim.x;
    double c[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) c[j] = 0.0;
    for (int base = 0; base < count; base += 1024) {
      double t[16];  // all in flight at once
#pragma unroll
      for (int j = 0; j < 16; ++j)
        t[j] = __hip_atomic_load(p + min(base + 64 * j + lane, count - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int j = 0; j < 16; ++j) c[j] += base + 64 * j + lane < count ? t[j] : 0.0;
    }
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
      for (int j = 0; j < h; ++j) c[j] += c[j + h];
    double v = c[0];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (lane == 0) red[wv][0] = v;
  }
  __syncthreads();
  if (tid == 0) {
    cg_fused_update(a.scal, red[0][0], red[1][0], red[2][0], red[3][0]);
    __hip_atomic_store(&a.scal->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.status) cg_publish(a.status, a.gen, a.scal);
  }
}

}  // namespace tbs

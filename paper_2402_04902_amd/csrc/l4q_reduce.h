// Sums of two arrays of partial results (dA and dB), by workgroups of a kernel of their own or of one that does more.
#pragma once

#include "l4q_kernels.h"

namespace l4q {

// workgroups of 256 threads that reduce_two_block wants
__host__ __device__ __forceinline__ int partials_blocks(int64_t n) { return (int)((n / 4 + 63) / 64); }
inline int two_partials_blocks(const TwoPartials& p) { return partials_blocks(p.na) + partials_blocks(p.nb); }

// 4 consecutive elements per thread (n % 4 == 0).
// A block is 64 element quads x 4 slices of the partial index: slice q sums partials [q*per, (q+1)*per) in
// ascending order and the four slice sums are added in ascending q, so the summation order is fixed.
__device__ __forceinline__ void reduce_two_block(const TwoPartials& p, int block, float4 (*slice_sum)[64]) {
  const int blocks_a = partials_blocks(p.na);
  const bool second = block >= blocks_a;
  const float* __restrict__ part = second ? p.pb : p.pa;
  float* __restrict__ out = second ? p.outb : p.outa;
  const int nblocks = second ? p.nbb : p.nba;
  const int64_t n = second ? p.nb : p.na;
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int64_t e = ((int64_t)(second ? block - blocks_a : block) * 64 + lane) * 4;
  const int per = (nblocks + 3) / 4;
  const int b0 = q * per, b1 = min(nblocks, b0 + per);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (e < n) {
#pragma unroll 4
    for (int b = b0; b < b1; ++b) {
      const float4 v = *reinterpret_cast<const float4*>(part + (int64_t)b * n + e);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
  }
  if (q > 0) slice_sum[q - 1][lane] = acc;
  __syncthreads();
  if (q > 0 || e >= n) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float4 v = slice_sum[k][lane];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  float4 r = make_float4(p.scale * acc.x, p.scale * acc.y, p.scale * acc.z, p.scale * acc.w);
  if (p.accumulate) {
    const float4 old = *reinterpret_cast<const float4*>(out + e);
    r = make_float4(old.x + r.x, old.y + r.y, old.z + r.z, old.w + r.w);
  }
  *reinterpret_cast<float4*>(out + e) = r;
}

}  // namespace l4q

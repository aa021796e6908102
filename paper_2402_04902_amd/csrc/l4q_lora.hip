// Rank-r side products of the QAT-LoRA layer (Sec. 3.1; Eq. lora_forward / lora_backward): the LoRA path kept
// next to the quantized weight instead of being merged into it.
//
//   down   U[T,r]   = Xs[T,n] . M            M = A^T (U = X A^T)  or  M = B (U = dY B)
//   up     Out[T,n] = Out + gamma U[T,r] . M  M = B^T (Y += gamma (X A^T) B^T)  or  M = A (dX += gamma (dY B) A)
//   tn     G[r,n]   = sum_t U[t,:]^T Xs[t,:]  per block of 128 tokens, summed in fixed order by reduce_partials_kernel
//                                             (dA = gamma (dY B)^T X,  dB^T = gamma (X A^T)^T dY)
// All three stream their large operand once per chunk of 16 ranks and are bound by HBM; U is binary32 and
// accumulation is binary32.  The small matrix is read either as [r, n] (rank-major, A) or as [n, r] (B).
#include "l4q_device.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

constexpr int LR_KC = 16;  // ranks per pass

// element (k, j) of the small matrix: rank-major [r, n] or [n, r]
template <class S, bool NR>
__device__ __forceinline__ float small_at(const S* __restrict__ M, int64_t n, int r, int k, int64_t j) {
  return load1(NR ? M + j * r + k : M + (int64_t)k * n + j);
}

// A wave (one per workgroup) takes LR_RB token rows, so that what it reads of the small matrix is used LR_RB times:
// U[t, k0 .. k0 + 15] = sum_j Xs[t, j] M(k, j).  Rank-major M (A, n % 4 == 0): a lane walks 4 consecutive columns
// with vector loads.  M as [n, r] (B): a lane walks single columns and reads that column's ranks contiguously.
constexpr int LR_RB = 4;

template <class S, bool NR>
__global__ __launch_bounds__(64) void lora_down_kernel(const S* __restrict__ Xs, int64_t T, int64_t n,
                                                         const S* __restrict__ M, int r, float* __restrict__ U) {
  const int lane = threadIdx.x & 63;
  const int64_t t0 = (int64_t)blockIdx.x * LR_RB;  // one wave per block
  if (t0 >= T) return;
  const S* xrow[LR_RB];
#pragma unroll
  for (int q = 0; q < LR_RB; ++q) xrow[q] = Xs + (t0 + q < T ? t0 + q : T - 1) * n;
  for (int k0 = 0; k0 < r; k0 += LR_KC) {
    float acc[LR_RB][LR_KC];
#pragma unroll
    for (int q = 0; q < LR_RB; ++q)
#pragma unroll
      for (int k = 0; k < LR_KC; ++k) acc[q][k] = 0.f;
    if (!NR) {
      for (int64_t j = (int64_t)lane * 4; j < n; j += 256) {
        float x[LR_RB][4];
#pragma unroll
        for (int q = 0; q < LR_RB; ++q) load4(xrow[q] + j, x[q]);
#pragma unroll
        for (int k = 0; k < LR_KC; ++k) {
          float a[4];
          load4(M + (int64_t)(k0 + k < r ? k0 + k : r - 1) * n + j, a);
          if (k0 + k >= r) a[0] = a[1] = a[2] = a[3] = 0.f;
#pragma unroll
          for (int q = 0; q < LR_RB; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[q][k] = fmaf(x[q][c], a[c], acc[q][k]);
        }
      }
    } else {
      for (int64_t j = lane; j < n; j += 64) {
        float m[LR_KC];
#pragma unroll
        for (int k = 0; k < LR_KC; ++k) m[k] = k0 + k < r ? load1(M + j * r + k0 + k) : 0.f;
#pragma unroll
        for (int q = 0; q < LR_RB; ++q) {
          const float x = load1(xrow[q] + j);
#pragma unroll
          for (int k = 0; k < LR_KC; ++k) acc[q][k] = fmaf(x, m[k], acc[q][k]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < LR_RB; ++q)
#pragma unroll
      for (int k = 0; k < LR_KC; ++k) {
        const float v = wave_sum_width(acc[q][k], 64);
        if (lane == 0 && k0 + k < r && t0 + q < T) U[(t0 + q) * r + k0 + k] = v;
      }
  }
}

template <class S> __device__ __forceinline__ float to_f32(S v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf16_to_f32(v); }
__device__ __forceinline__ void store1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store1(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// Out[t, j] += gamma * sum_k U[t, k] M(k, j).  A thread owns one column and LR_UT consecutive tokens: its column
// of the small matrix is read once per rank chunk and stays in registers; U[t, :] is uniform over the block.
constexpr int LR_UT = 16;

template <class S, bool NR>
__global__ __launch_bounds__(256) void lora_up_kernel(S* __restrict__ Out, int64_t T, int64_t n,
                                                       const float* __restrict__ U, const S* __restrict__ M, int r,
                                                       float gamma) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t t0 = (int64_t)blockIdx.y * LR_UT;
  if (j >= n) return;
  float acc[LR_UT];
#pragma unroll
  for (int q = 0; q < LR_UT; ++q) acc[q] = 0.f;
  for (int k0 = 0; k0 < r; k0 += LR_KC) {
    float m[LR_KC];
#pragma unroll
    for (int k = 0; k < LR_KC; ++k) m[k] = k0 + k < r ? small_at<S, NR>(M, n, r, k0 + k, j) : 0.f;
#pragma unroll
    for (int q = 0; q < LR_UT; ++q) {
      const float* u = U + (t0 + q < T ? t0 + q : T - 1) * r + k0;  // uniform over the block
#pragma unroll
      for (int k = 0; k < LR_KC; ++k)
        if (k0 + k < r) acc[q] = fmaf(u[k], m[k], acc[q]);
    }
  }
#pragma unroll
  for (int q = 0; q < LR_UT; ++q)
    if (t0 + q < T) {
      S* dst = Out + (t0 + q) * n + j;
      store1(dst, to_f32<S>(*dst) + gamma * acc[q]);
    }
}

// part[tb][k][j] (or [tb][j][k] when NR) = sum over the 128 rows of block tb of U[t, k] Xs[t, j].
// Bound: Xs read once.  v_mfma_f32_16x16x4_f32 takes 16 ranks x 4 rows x 16 columns in binary32: lane (h = lane / 16,
// c = lane % 16) holds row h of four and 4 consecutive columns, one per op, so its loads are 8 or 16 consecutive bytes, 16
// lanes a run of 128 or 256, and no operand passes through LDS but U.  A workgroup takes 64 columns; each of its 4 waves
// 32 of the rows, all requested at once and kept in registers for every 16 ranks; the waves' sums meet in LDS and are
// added in wave order.  2048 x 4096 bf16 at 16 ranks: 122 .. 129 us with one column per thread and a row's U fetched by
// scalar loads ahead of every 16 multiply-adds, 15.5 us as vector multiply-adds on U broadcast from LDS (the vector rate
// itself is half the matrix rate), 9.1 us in
// this form (10.0 written as [n, r]); 2048 x 2048 binary32 99, 15.0, 7.0 us; 256 x 256 binary32 65, 12.3, 5.1 us.
constexpr int LR_TB = 128;

// 4 consecutive elements as they lie in memory
template <class S> struct Row4;
template <> struct Row4<float> {
  typedef float vec_t __attribute__((ext_vector_type(4), aligned(4)));  // (rows of an odd number of floats)
  typedef float raw_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ raw_t load(const float* p) { return *reinterpret_cast<const vec_t*>(p); }
  static __device__ __forceinline__ float get(const raw_t& v, int c) { return v[c]; }
  static __device__ __forceinline__ void set(raw_t& v, int c, const float* p) { v[c] = *p; }
};
template <> struct Row4<bf16_t> {  // (rows are whole 16-byte pieces)
  typedef uint32_t raw_t __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ raw_t load(const bf16_t* p) { return *reinterpret_cast<const raw_t*>(p); }
  static __device__ __forceinline__ float get(const raw_t& v, int c) {
    return __uint_as_float(c & 1 ? v[c >> 1] & 0xFFFF0000u : v[c >> 1] << 16);
  }
  static __device__ __forceinline__ void set(raw_t& v, int c, const bf16_t* p) {
    v[c >> 1] |= (uint32_t)*p << (c & 1 ? 16 : 0);
  }
};

template <class S, class UT, bool NR>
__global__ __launch_bounds__(256) void tn_partial_kernel(const UT* __restrict__ U, const S* __restrict__ Xs, int64_t T,
                                                          int64_t n, int r, float* __restrict__ part) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  typedef Row4<float>::vec_t vec_t;
  constexpr int STEPS = LR_TB / 4 / 4;  // groups of 4 rows per wave
  __shared__ __align__(16) float sums[4][LR_KC][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 4, c16 = lane & 15;
  // the last workgroup of a row takes the last 64 columns, some of them its neighbour's (same sums, written twice);
  // rows of 4 to 63 columns end in lanes that repeat the last 4
  const int64_t j0 = n < 64 ? 0 : (int64_t)blockIdx.x * 64 < n - 64 ? (int64_t)blockIdx.x * 64 : n - 64;
  const int jl = n < 4 ? 0 : j0 + c16 * 4 < n - 4 ? c16 * 4 : (int)(n - 4 - j0);  // this lane's first column, from j0
  const int64_t tb = blockIdx.y, t0 = tb * LR_TB + wave * (LR_TB / 4) + h;
  typename Row4<S>::raw_t x[STEPS];
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int64_t t = t0 + 4 * q;
    const S* p = Xs + (t < T ? t : T - 1) * n + j0;
    if (n >= 4) x[q] = Row4<S>::load(p + jl);
    else {
      x[q] = typename Row4<S>::raw_t(0);
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c < n) Row4<S>::set(x[q], c, p + c);
    }
    if (t >= T) x[q] = typename Row4<S>::raw_t(0);
  }
  float* dst = part + tb * (int64_t)r * n;
  for (int k0 = 0; k0 < r; k0 += LR_KC) {
    float u[STEPS];
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
      const int64_t t = t0 + 4 * q;
      const bool live = t < T && k0 + c16 < r;
      const float v = load1(U + (live ? t * r + k0 + c16 : 0));
      u[q] = live ? v : 0.f;
    }
    f32x4_t acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(u[q], Row4<S>::get(x[q], c), acc[c], 0, 0, 0);
    if (k0 > 0) __syncthreads();  // the previous ranks' sums have been read
#pragma unroll
    for (int e = 0; e < 4; ++e)  // accumulator: rank 4 h + e, column c16 of op c
      *reinterpret_cast<vec_t*>(&sums[wave][4 * h + e][jl]) = vec_t{acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
    __syncthreads();
    auto total = [&](int k, int j) { return ((sums[0][k][j] + sums[1][k][j]) + sums[2][k][j]) + sums[3][k][j]; };
    if constexpr (NR) {
      const int j = tid >> 2, k = (tid & 3) * 4;
      if (j0 + j < n) {
        float* q = dst + (j0 + j) * r + k0 + k;
        if (k0 + k + 3 < r) *reinterpret_cast<vec_t*>(q) = vec_t{total(k, j), total(k + 1, j), total(k + 2, j), total(k + 3, j)};
        else
          for (int c = 0; c < 3; ++c)
            if (k0 + k + c < r) q[c] = total(k + c, j);
      }
    } else {
      if (j0 + lane < n) {
#pragma unroll
        for (int k = wave; k < LR_KC; k += 4)
          if (k0 + k < r) dst[(int64_t)(k0 + k) * n + j0 + lane] = total(k, lane);
      }
    }
  }
#endif
}

}  // namespace

template <class S>
void launch_lora_down(const S* Xs, int64_t T, int64_t n, const S* M, int r, bool m_is_n_by_r, float* U,
                      hipStream_t stream) {
  dim3 grid((unsigned)((T + LR_RB - 1) / LR_RB));
  if (m_is_n_by_r) hipLaunchKernelGGL((lora_down_kernel<S, true>), grid, dim3(64), 0, stream, Xs, T, n, M, r, U);
  else hipLaunchKernelGGL((lora_down_kernel<S, false>), grid, dim3(64), 0, stream, Xs, T, n, M, r, U);
}

template <class S>
void launch_lora_up(S* Out, int64_t T, int64_t n, const float* U, const S* M, int r, bool m_is_n_by_r, float gamma,
                    hipStream_t stream) {
  dim3 grid((unsigned)((n + 255) / 256), (unsigned)((T + LR_UT - 1) / LR_UT));
  if (m_is_n_by_r) hipLaunchKernelGGL((lora_up_kernel<S, true>), grid, dim3(256), 0, stream, Out, T, n, U, M, r, gamma);
  else hipLaunchKernelGGL((lora_up_kernel<S, false>), grid, dim3(256), 0, stream, Out, T, n, U, M, r, gamma);
}

int64_t lora_tn_blocks(int64_t T) { return (T + LR_TB - 1) / LR_TB; }

template <class S, class UT>
void launch_tn(const UT* U, const S* Xs, int64_t T, int64_t n, int r, bool out_n_by_r, float* partial, float gamma,
               float* out, bool accumulate, hipStream_t stream) {
  const int64_t nb = lora_tn_blocks(T);
  dim3 grid((unsigned)((n + 63) / 64), (unsigned)nb);
  if (out_n_by_r) hipLaunchKernelGGL((tn_partial_kernel<S, UT, true>), grid, dim3(256), 0, stream, U, Xs, T, n, r, partial);
  else hipLaunchKernelGGL((tn_partial_kernel<S, UT, false>), grid, dim3(256), 0, stream, U, Xs, T, n, r, partial);
  launch_reduce_partials(partial, nb, (int64_t)r * n, gamma, out, accumulate, stream);
}

template void launch_lora_down<float>(const float*, int64_t, int64_t, const float*, int, bool, float*, hipStream_t);
template void launch_lora_down<bf16_t>(const bf16_t*, int64_t, int64_t, const bf16_t*, int, bool, float*, hipStream_t);
template void launch_lora_up<float>(float*, int64_t, int64_t, const float*, const float*, int, bool, float, hipStream_t);
template void launch_lora_up<bf16_t>(bf16_t*, int64_t, int64_t, const float*, const bf16_t*, int, bool, float, hipStream_t);
template void launch_tn<float, float>(const float*, const float*, int64_t, int64_t, int, bool, float*, float, float*, bool,
                                      hipStream_t);
template void launch_tn<bf16_t, float>(const float*, const bf16_t*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);
template void launch_tn<float, bf16_t>(const bf16_t*, const float*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);

}  // namespace l4q

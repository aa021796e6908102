// Rank-r side products of the QAT-LoRA layer (Sec. 3.1; Eq. lora_forward / lora_backward): the LoRA path kept
// next to the quantized weight instead of being merged into it.
//
//   down   U[T,r]   = Xs[T,n] . M^T           U = X A^T, or U = dY B with B transposed first (bfloat16 operands; the
//                                             binary32 layer uses the binary32 GEMM)
//   up     Out[T,n] += gamma U[T,r] . M       inside the main product (RankTerm, l4q_gemm.hip), or the binary32 GEMM
//   tn     G[r,n]   = sum_t U[t,:]^T Xs[t,:]  per block of 128 tokens, summed in fixed order by reduce_partials_kernel
//                                             (dA = gamma (dY B)^T X,  dB^T = gamma (X A^T)^T dY)
// U is binary32 and accumulation is binary32.
#include "l4q_device.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

constexpr int LR_KC = 16;  // ranks per matrix op

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// U[t, k] = sum_j Xs[t, j] M[k, j].  Bound: Xs read once.  A workgroup takes 16 rows of Xs and NC x 16 ranks; its 16 waves
// deal the 32-wide k-steps of v_mfma_f32_16x16x32_bf16 out among themselves (8 rows' worth of waves is all a few thousand
// tokens give a chip of 256 compute units), four steps of loads in flight each, and their sums meet in LDS, added in wave
// order.  2048 x 4096 at 16 ranks: 9.1 us; a wave per 4 rows with vector multiply-adds, which this replaces, 81 us
// (127 us with B read as [n, r]).
constexpr int LD_WAVES = 16;
constexpr int LD_AHEAD = 4;

template <int NC>
__global__ __launch_bounds__(64 * LD_WAVES) void lora_down_kernel(const bf16_t* __restrict__ Xs, int64_t T, int64_t n,
                                                                  const bf16_t* __restrict__ M, int r,
                                                                  float* __restrict__ U) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ float sums[LD_WAVES][16][16 * NC + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, h = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * 16;
  const int k0 = blockIdx.y * (16 * NC);
  // rows past T and ranks past r repeat the last one; they are not stored
  const bf16_t* xp = Xs + (t0 + c16 < T ? t0 + c16 : T - 1) * n;
  const bf16_t* mp[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) mp[c] = M + (int64_t)(k0 + c * 16 + c16 < r ? k0 + c * 16 + c16 : r - 1) * n;
  f32x4_t acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int64_t j0 = wave * 32; j0 < n; j0 += LD_WAVES * LD_AHEAD * 32) {
    bf16x8_t fx[LD_AHEAD], fm[LD_AHEAD][NC];
    const bf16x8_t zero = {};
#pragma unroll
    for (int u = 0; u < LD_AHEAD; ++u) {
      const int64_t j = j0 + u * (LD_WAVES * 32) + h * 8;
      const bool live = j < n;  // (n % 8 == 0: a lane's 8 values are all inside or all outside)
      const bf16x8_t x = *reinterpret_cast<const bf16x8_t*>(xp + (live ? j : 0));
      fx[u] = live ? x : zero;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const bf16x8_t m = *reinterpret_cast<const bf16x8_t*>(mp[c] + (live ? j : 0));
        fm[u][c] = live ? m : zero;
      }
    }
#pragma unroll
    for (int u = 0; u < LD_AHEAD; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[u], fm[u][c], acc[c], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) sums[wave][4 * h + e][c * 16 + c16] = acc[c][e];
  __syncthreads();
  for (int q = tid; q < 256 * NC; q += 64 * LD_WAVES) {
    const int row = q / (16 * NC), k = q % (16 * NC);
    float v = sums[0][row][k];
#pragma unroll
    for (int w = 1; w < LD_WAVES; ++w) v += sums[w][row][k];
    if (t0 + row < T && k0 + k < r) U[(t0 + row) * r + k0 + k] = v;
  }
#endif
}

// out[k][j] = in[j][k]: 64 rows of `in` per workgroup through LDS
__global__ __launch_bounds__(256) void transpose_small_kernel(const bf16_t* __restrict__ in, int64_t n, int r,
                                                               bf16_t* __restrict__ out) {
  __shared__ bf16_t tile[64][256 + 2];  // (rank <= 256)
  const int64_t j0 = (int64_t)blockIdx.x * 64;
  const int rows = n - j0 < 64 ? (int)(n - j0) : 64;
  for (int q = threadIdx.x; q < rows * r; q += 256) tile[q / r][q % r] = in[j0 * r + q];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  if (lane < rows)
    for (int k = threadIdx.x >> 6; k < r; k += 4) out[(int64_t)k * n + j0 + lane] = tile[lane][k];
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

//
// WHOLE (up to 4 row blocks): a workgroup has 4 waves for each row block, and the blocks' sums, formed as above, are added in
// block order as the second pass would add them, scaled and stored: one launch instead of two, the same bits.
template <class S, class UT, bool NR, bool WHOLE>
__global__ __launch_bounds__(WHOLE ? 1024 : 256) void tn_partial_kernel(const UT* __restrict__ U, const S* __restrict__ Xs, int64_t T,
                                                          int64_t n, int r, float* __restrict__ part, float gamma, bool accumulate) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef Row4<float>::vec_t vec_t;
  constexpr int STEPS = LR_TB / 4 / 4;  // groups of 4 rows per wave
  __shared__ __align__(16) float sums[WHOLE ? 16 : 4][LR_KC][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 4, c16 = lane & 15, waves = WHOLE ? (int)blockDim.x >> 6 : 4;
  // the last workgroup of a row takes the last 64 columns, some of them its neighbour's (same sums, written twice);
  // rows of 4 to 63 columns end in lanes that repeat the last 4
  const int64_t j0 = n < 64 ? 0 : (int64_t)blockIdx.x * 64 < n - 64 ? (int64_t)blockIdx.x * 64 : n - 64;
  const int jl = n < 4 ? 0 : j0 + c16 * 4 < n - 4 ? c16 * 4 : (int)(n - 4 - j0);  // this lane's first column, from j0
  const int64_t tb = WHOLE ? 0 : blockIdx.y, t0 = tb * LR_TB + wave * (LR_TB / 4) + h;
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
    auto total = [&](int k, int j) {
      auto block = [&](int w) { return ((sums[w][k][j] + sums[w + 1][k][j]) + sums[w + 2][k][j]) + sums[w + 3][k][j]; };
      float v = 0.f + block(0);  // (as the second pass starts: no negative zero)
      if constexpr (WHOLE) {
        for (int w = 4; w < waves; w += 4) v += block(w);
      }
      return v;
    };
    if constexpr (WHOLE) {  // one output per thread and turn
      for (int q = tid; q < LR_KC * 64; q += waves * 64) {
        const int k = NR ? q % LR_KC : q / 64, j = NR ? q / LR_KC : q % 64;
        if (j0 + j < n && k0 + k < r && j0 + j >= (int64_t)blockIdx.x * 64) {  // (columns below are the neighbour's: added to once)
          float* p = part + (NR ? (j0 + j) * r + k0 + k : (int64_t)(k0 + k) * n + j0 + j);
          const float v = gamma * total(k, j);
          *p = accumulate ? *p + v : v;
        }
      }
    } else if constexpr (NR) {
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

void launch_lora_down(const bf16_t* Xs, int64_t T, int64_t n, const bf16_t* M, int r, float* U, hipStream_t stream) {
  const unsigned tiles = (unsigned)((T + 15) / 16);
  if (r <= 16)
    hipLaunchKernelGGL(lora_down_kernel<1>, dim3(tiles), dim3(64 * LD_WAVES), 0, stream, Xs, T, n, M, r, U);
  else if (r <= 32)
    hipLaunchKernelGGL(lora_down_kernel<2>, dim3(tiles), dim3(64 * LD_WAVES), 0, stream, Xs, T, n, M, r, U);
  else
    hipLaunchKernelGGL(lora_down_kernel<4>, dim3(tiles, (unsigned)((r + 63) / 64)), dim3(64 * LD_WAVES), 0, stream, Xs, T, n,
                       M, r, U);
}

void launch_transpose_small(const bf16_t* in, int64_t n, int r, bf16_t* out, hipStream_t stream) {
  hipLaunchKernelGGL(transpose_small_kernel, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, stream, in, n, r, out);
}

int64_t lora_tn_blocks(int64_t T) { return (T + LR_TB - 1) / LR_TB; }

template <class S, class UT>
void launch_tn(const UT* U, const S* Xs, int64_t T, int64_t n, int r, bool out_n_by_r, float* partial, float gamma,
               float* out, bool accumulate, hipStream_t stream) {
  const int64_t nb = lora_tn_blocks(T);
#define L4Q_TN(NR, WHOLE, GRID, THREADS, OUT) \
  hipLaunchKernelGGL((tn_partial_kernel<S, UT, NR, WHOLE>), GRID, dim3(THREADS), 0, stream, U, Xs, T, n, r, OUT, gamma, accumulate)
  const unsigned cols = (unsigned)((n + 63) / 64);
  if (nb <= 4) {
    if (out_n_by_r) L4Q_TN(true, true, dim3(cols), (unsigned)(256 * nb), out);
    else L4Q_TN(false, true, dim3(cols), (unsigned)(256 * nb), out);
    return;
  }
  if (out_n_by_r) L4Q_TN(true, false, dim3(cols, (unsigned)nb), 256u, partial);
  else L4Q_TN(false, false, dim3(cols, (unsigned)nb), 256u, partial);
#undef L4Q_TN
  launch_reduce_partials(partial, nb, (int64_t)r * n, gamma, out, accumulate, stream);
}

template void launch_tn<float, float>(const float*, const float*, int64_t, int64_t, int, bool, float*, float, float*, bool,
                                      hipStream_t);
template void launch_tn<bf16_t, float>(const float*, const bf16_t*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);
template void launch_tn<float, bf16_t>(const bf16_t*, const float*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);

}  // namespace l4q

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

// Two products of the same T and r (the backward pass's) share a launch: 2048 tokens are 128 workgroups each, half of the
// compute units (2 x 9.2 us apart, 10.9 together).
template <int NC>
__global__ __launch_bounds__(64 * LD_WAVES) void lora_down_kernel(LoraDown job0, LoraDown job1, int64_t T, int r) {
#if defined(__HIP_DEVICE_COMPILE__)
  const LoraDown& job = blockIdx.z == 0 ? job0 : job1;
  const bf16_t* __restrict__ Xs = job.Xs;
  const bf16_t* __restrict__ M = job.M;
  float* __restrict__ U = job.U;
  const int64_t n = job.n;
  __shared__ float sums[LD_WAVES][16][16 * NC + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, h = lane >> 4;
  const int64_t t0 = (int64_t)blockIdx.x * 16;
  const int k0 = blockIdx.y * (16 * NC);
  // rows past T and ranks past r repeat the last one; they are not stored
  const bf16_t* xp = Xs + (t0 + c16 < T ? t0 + c16 : T - 1) * n;
  const bf16_t* mp[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) mp[c] = M + (int64_t)(k0 + c * 16 + c16 < r ? k0 + c * 16 + c16 : r - 1) * job.ldm;
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

// WHOLE (see tn_whole): a workgroup has 4 waves for each row block, and the blocks' sums, formed as above, are added in
// block order as the second pass would add them, scaled and stored: one launch instead of two, the same bits.
typedef float TnSums[LR_KC][64];

template <class S, class UT, bool NR, bool WHOLE>
__device__ __forceinline__ void tn_columns(int block, TnSums* sums, const UT* __restrict__ U, const S* __restrict__ Xs, int64_t T,
                                           int64_t n, int r, float* __restrict__ part, float gamma, bool accumulate) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef Row4<float>::vec_t vec_t;
  constexpr int STEPS = LR_TB / 4 / 4;  // groups of 4 rows per wave
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 4, c16 = lane & 15, waves = WHOLE ? (int)blockDim.x >> 6 : 4;
  // the last workgroup of a row takes the last 64 columns, some of them its neighbour's (same sums, written twice);
  // rows of 4 to 63 columns end in lanes that repeat the last 4
  const int64_t j0 = n < 64 ? 0 : (int64_t)block * 64 < n - 64 ? (int64_t)block * 64 : n - 64;
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
    if constexpr (WHOLE) {
      auto mine = [&](int j) { return j0 + j < n && j0 + j >= (int64_t)block * 64; };  // (columns below are the neighbour's: added to once)
      if constexpr (NR) {  // 4 consecutive ranks per thread: 16 lanes read 16 columns (a rank per lane: one bank for all of them)
        const int j = tid >> 2, k = (tid & 3) * 4;
        if (tid < 256 && mine(j)) {
          float* q = part + (j0 + j) * r + k0 + k;
          if (k0 + k + 3 < r) {
            vec_t v = {gamma * total(k, j), gamma * total(k + 1, j), gamma * total(k + 2, j), gamma * total(k + 3, j)};
            if (accumulate) v = *reinterpret_cast<const vec_t*>(q) + v;
            *reinterpret_cast<vec_t*>(q) = v;
          } else {
            for (int c = 0; c < 3; ++c)
              if (k0 + k + c < r) {
                const float v = gamma * total(k + c, j);
                q[c] = accumulate ? q[c] + v : v;
              }
          }
        }
      } else if (mine(lane)) {
        for (int k = wave; k < LR_KC; k += waves)
          if (k0 + k < r) {
            float* p = part + (int64_t)(k0 + k) * n + j0 + lane;
            const float v = gamma * total(k, lane);
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

template <class S, class UT, bool NR, bool WHOLE>
__global__ __launch_bounds__(WHOLE ? 512 : 256) void tn_partial_kernel(const UT* __restrict__ U, const S* __restrict__ Xs, int64_t T,
                                                          int64_t n, int r, float* __restrict__ part, float gamma, bool accumulate) {
  __shared__ __align__(16) TnSums sums[WHOLE ? 8 : 4];
  tn_columns<S, UT, NR, WHOLE>((int)blockIdx.x, sums, U, Xs, T, n, r, part, gamma, accumulate);
}

// dA and dB of the QAT-LoRA layer in one launch (2048 tokens, 4096 x 4096, rank 16: 9.7 + 10.6 us apart, 17.5 together, and one
// second pass instead of two): the first `cols` workgroups of a row take a as [r, n], the others b as [n, r].
struct TnJob {
  const float* U;
  const bf16_t* Xs;
  int64_t n;
  float* out;  // partial sums, or the result (WHOLE)
};
template <bool WHOLE>
__global__ __launch_bounds__(WHOLE ? 512 : 256) void tn_pair_kernel(TnJob a, TnJob b, int cols, int64_t T, int r, float gamma,
                                                                     bool accumulate) {
  __shared__ __align__(16) TnSums sums[WHOLE ? 8 : 4];
  if ((int)blockIdx.x < cols)
    tn_columns<bf16_t, float, false, WHOLE>((int)blockIdx.x, sums, a.U, a.Xs, T, a.n, r, a.out, gamma, accumulate);
  else
    tn_columns<bf16_t, float, true, WHOLE>((int)blockIdx.x - cols, sums, b.U, b.Xs, T, b.n, r, b.out, gamma, accumulate);
}

}  // namespace

void launch_lora_down(const LoraDown* jobs, int njobs, int64_t T, int r, hipStream_t stream) {
  const unsigned tiles = (unsigned)((T + 15) / 16), z = (unsigned)njobs;
  const LoraDown &a = jobs[0], &b = jobs[njobs - 1];
  if (r <= 16) hipLaunchKernelGGL(lora_down_kernel<1>, dim3(tiles, 1, z), dim3(64 * LD_WAVES), 0, stream, a, b, T, r);
  else if (r <= 32) hipLaunchKernelGGL(lora_down_kernel<2>, dim3(tiles, 1, z), dim3(64 * LD_WAVES), 0, stream, a, b, T, r);
  else
    hipLaunchKernelGGL(lora_down_kernel<4>, dim3(tiles, (unsigned)((r + 63) / 64), z), dim3(64 * LD_WAVES), 0, stream, a, b, T, r);
}

// One pass or two (WHOLE): a workgroup of one pass takes all row blocks, so with two of them and high ranks, whose steps of 16 it
// goes through one after the other, its waves meet at barriers twice as often for the launch it saves.  Binary32, us in two passes /
// one, [r, n], n = 1024: 128 rows 10.2 / 7.8 at ranks up to 16, 10.7 / 7.8 at 64, 28 / 23 at 256; 200 rows 10.5 / 7.9 at 16, 10.8 /
// 10.4 at 64 (as [n, r] 10.3 / 11.2), 29 / 34 at 256.  Four blocks (1024 threads), 495 columns: 67.3 / 68.2 for a whole step.
static bool tn_whole(int64_t row_blocks, int r) { return row_blocks == 1 || (row_blocks == 2 && r <= 32); }

int64_t lora_tn_blocks(int64_t T) { return (T + LR_TB - 1) / LR_TB; }

template <class S, class UT>
void launch_tn(const UT* U, const S* Xs, int64_t T, int64_t n, int r, bool out_n_by_r, float* partial, float gamma,
               float* out, bool accumulate, hipStream_t stream) {
  const int64_t nb = lora_tn_blocks(T);
#define L4Q_TN(NR, WHOLE, GRID, THREADS, OUT) \
  hipLaunchKernelGGL((tn_partial_kernel<S, UT, NR, WHOLE>), GRID, dim3(THREADS), 0, stream, U, Xs, T, n, r, OUT, gamma, accumulate)
  const unsigned cols = (unsigned)((n + 63) / 64);
  if (tn_whole(nb, r)) {
    if (out_n_by_r) L4Q_TN(true, true, dim3(cols), (unsigned)(256 * nb), out);
    else L4Q_TN(false, true, dim3(cols), (unsigned)(256 * nb), out);
    return;
  }
  if (out_n_by_r) L4Q_TN(true, false, dim3(cols, (unsigned)nb), 256u, partial);
  else L4Q_TN(false, false, dim3(cols, (unsigned)nb), 256u, partial);
#undef L4Q_TN
  launch_reduce_partials(partial, nb, (int64_t)r * n, gamma, out, accumulate, stream);
}

void launch_tn_pair(const float* Ua, const bf16_t* Xa, int64_t na, float* outa, float* parta, const float* Ub, const bf16_t* Xb,
                    int64_t nb, float* outb, float* partb, int64_t T, int r, float gamma, bool accumulate, hipStream_t stream) {
  const int64_t blocks = lora_tn_blocks(T);
  const int cols = (int)((na + 63) / 64), all = cols + (int)((nb + 63) / 64);
  if (tn_whole(blocks, r)) {
    hipLaunchKernelGGL(tn_pair_kernel<true>, dim3((unsigned)all), dim3((unsigned)(256 * blocks)), 0, stream, TnJob{Ua, Xa, na, outa},
                       TnJob{Ub, Xb, nb, outb}, cols, T, r, gamma, accumulate);
    return;
  }
  hipLaunchKernelGGL(tn_pair_kernel<false>, dim3((unsigned)all, (unsigned)blocks), dim3(256), 0, stream, TnJob{Ua, Xa, na, parta},
                     TnJob{Ub, Xb, nb, partb}, cols, T, r, gamma, accumulate);
  launch_reduce_two_partials({parta, (int)blocks, (int64_t)r * na, outa, partb, (int)blocks, (int64_t)r * nb, outb, gamma, accumulate},
                             stream);
}

template void launch_tn<float, float>(const float*, const float*, int64_t, int64_t, int, bool, float*, float, float*, bool,
                                      hipStream_t);
template void launch_tn<bf16_t, float>(const float*, const bf16_t*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);
template void launch_tn<float, bf16_t>(const bf16_t*, const float*, int64_t, int64_t, int, bool, float*, float, float*,
                                       bool, hipStream_t);

}  // namespace l4q

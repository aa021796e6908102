// bf16 MFMA GEMMs of the layer with a plain store epilogue (main loop: l4q_gemm_core.h).
//
//   forward   Y  [T,o] = X  [T,i] . Wq  [o,ipad]^T      both operands K-contiguous; Wq in blocks of 32 k-values
//   dX        dX [T,i] = dY [T,o] . WqT [i,opad]^T      both operands K-contiguous; WqT likewise
//   dWq       dWq[o,i] = dY [T,o]^T . X [T,i]           both operands K-major (unfused backward only;
//                                                       the fused form lives in l4q_bwd_fused.hip)
// The workspace operand (Wq, WqT) is zero-padded along k to the 32-wide k-step; the caller's operand is
// not: its 16-byte chunks past the row end are masked (read as zeros) in the last unit of 64 k-values.
#include "l4q_device.h"
#include "l4q_gemm_core.h"
#include "l4q_kernels.h"
#include "l4q_reduce.h"

namespace l4q {

namespace {

// ---------------------------------------------------------------------------------------------
// Direct-to-LDS ring pipeline (l4q_gemm_core.h) + plain store epilogue.  Operands below 1 GiB.
// ---------------------------------------------------------------------------------------------
// Store epilogue of a macro tile; `LDS_BYTES` of LDS at `lds` are free.
template <class T, bool OUT_BF16, int LDS_BYTES>
__device__ __forceinline__ void store_tile(gemm::Accum<T>& acc, int M, int N, void* __restrict__ Cout, int64_t ldc,
                                           int m0, int n0, unsigned char* lds) {
  // bf16 output through LDS (free after the main loop): a lane holds 4 consecutive columns of 64 different
  // rows, which as direct stores are 16-byte pieces of 32 cache lines per instruction.  Each wave instead
  // parks its 128 x 128 block in its own LDS region (rows padded to 272 bytes) and writes it out as 16 bytes
  // per lane, 16 lanes per 256-byte row segment.  Needs 16-byte aligned rows: ldc % 8 == 0 and N % 8 == 0.
  constexpr int EP_ROW = T::WTN * 2 + 16;
  constexpr int EP_LPR = T::WTN / 8;  // lanes that cover a row of the wave's block with 16 bytes each
  constexpr bool EP_FITS = OUT_BF16 && (T::WTN == 128 || T::WTN == 64) && T::NW * T::WTM * EP_ROW <= LDS_BYTES;
  if (EP_FITS && (ldc & 7) == 0 && (N & 7) == 0) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* region = lds + wave * (T::WTM * EP_ROW);
#pragma unroll
    for (int a = 0; a < T::TM; ++a)
#pragma unroll
      for (int b = 0; b < T::TN; ++b)
#pragma unroll
        for (int eg = 0; eg < 4; ++eg) {
          uint2 v;
          v.x = pack_bf16x2(acc.v[a][b][4 * eg], acc.v[a][b][4 * eg + 1]);
          v.y = pack_bf16x2(acc.v[a][b][4 * eg + 2], acc.v[a][b][4 * eg + 3]);
          *reinterpret_cast<uint2*>(region + (a * 32 + (lane & 31)) * EP_ROW + (b * 32 + 8 * eg + 4 * (lane >> 5)) * 2) = v;
        }
    bf16_t* C = reinterpret_cast<bf16_t*>(Cout);
    const int mw = m0 + (wave / T::WAVES_N) * T::WTM;
    const int nw = n0 + (wave % T::WAVES_N) * T::WTN + (lane % EP_LPR) * 8;
#pragma unroll 8
    for (int it = 0; it < T::WTM * EP_LPR / 64; ++it) {
      const int row = it * (64 / EP_LPR) + lane / EP_LPR;
      const uint4 v = *reinterpret_cast<const uint4*>(region + row * EP_ROW + (lane % EP_LPR) * 16);
      if (mw + row < M && nw < N) *reinterpret_cast<uint4*>(C + (int64_t)(mw + row) * ldc + nw) = v;
    }
    return;
  }
#pragma unroll
  for (int a = 0; a < T::TM; ++a) {
#pragma unroll
    for (int b = 0; b < T::TN; ++b) {
#pragma unroll
      for (int eg = 0; eg < 4; ++eg) {
        int m, n;
        gemm::acc_coords<T>(a, b, eg, m, n);
        m += m0;
        n += n0;
        if (m < M && n < N) {  // N % 4 == 0: the 4 consecutive columns are all inside
          const float v[4] = {acc.v[a][b][4 * eg], acc.v[a][b][4 * eg + 1], acc.v[a][b][4 * eg + 2],
                              acc.v[a][b][4 * eg + 3]};
          if (OUT_BF16) store4(reinterpret_cast<bf16_t*>(Cout) + (int64_t)m * ldc + n, v);
          else store4(reinterpret_cast<float*>(Cout) + (int64_t)m * ldc + n, v);
        }
      }
    }
  }
}

// Leaves gamma U . M^T (see RankTerm) in the tile's accumulators, zero on entry, operands straight from memory: U is
// binary32 and goes through the bfloat16 matrix op as the exact sum of three bfloat16 parts (8 significand bits each, cut
// off rather than rounded, so that no part of a finite value is infinite), so the product is what binary32 operands would
// give.  A non-finite M meets the first part alone: the others may be zero or of either sign, and would make NaN of an
// infinite sum.  gamma scales the sum, as in gamma (U . M^T): gamma U by itself may overflow.
// At most 3 r / 16 matrix ops per accumulator tile against K / 16 of the main loop.
template <class T>
__device__ __forceinline__ void add_rank_term(gemm::Accum<T>& acc, const RankTerm& t, int M, int N, int m0, int n0) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef gemm::bf16x8_t bf16x8_t;
  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mw = m0 + (wave / T::WAVES_N) * T::WTM + l32, nw = n0 + (wave % T::WAVES_N) * T::WTN + l32;
#pragma unroll 1
  for (int k0 = 0; k0 < t.r; k0 += 16) {
    const int kb = k0 + half * 8;
    bf16x8_t fb[T::TN];
#pragma unroll
    for (int b = 0; b < T::TN; ++b) {
      const int n = nw + b * 32 < N ? nw + b * 32 : N - 1;  // (columns and rows past the matrix are not stored)
      if (t.n_by_r && (t.r & 7) == 0) {
        const uint4 v = *reinterpret_cast<const uint4*>(t.M + (int64_t)n * t.r + (kb < t.r ? kb : 0));
        fb[b] = __builtin_bit_cast(bf16x8_t, kb < t.r ? v : make_uint4(0, 0, 0, 0));
      } else {
        union { bf16_t h[8]; bf16x8_t v; } f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = kb + e < t.r ? kb + e : 0;
          const bf16_t v = t.n_by_r ? t.M[(int64_t)n * t.r + k] : t.M[(int64_t)k * N + n];
          f.h[e] = kb + e < t.r ? v : (bf16_t)0;
        }
        fb[b] = f.v;
      }
    }
    bf16x8_t fin[T::TN];  // fb with its infinities and NaN taken out
#pragma unroll
    for (int b = 0; b < T::TN; ++b) {
      union { uint32_t w[4]; bf16x8_t v; } f;
      f.v = fb[b];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        f.w[e] = ((f.w[e] & 0x7F80u) == 0x7F80u ? 0u : f.w[e] & 0xFFFFu) |
                 ((f.w[e] & 0x7F800000u) == 0x7F800000u ? 0u : f.w[e] & 0xFFFF0000u);
      fin[b] = f.v;
    }
    float u[T::TM][8];  // all rows requested before the first is used
#pragma unroll
    for (int a = 0; a < T::TM; ++a) {
      const int m = mw + a * 32 < M ? mw + a * 32 : M - 1;
      const float* up = t.U + (int64_t)m * t.r;
      if ((t.r & 7) == 0) {  // 16-byte rows, and a lane's 8 ranks are all inside or all outside
        load4(up + (kb < t.r ? kb : 0), *reinterpret_cast<float(*)[4]>(&u[a][0]));
        load4(up + (kb < t.r ? kb + 4 : 0), *reinterpret_cast<float(*)[4]>(&u[a][4]));
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) u[a][e] = up[kb + e < t.r ? kb + e : 0];
      }
    }
#pragma unroll
    for (int a = 0; a < T::TM; ++a) {
      union { bf16_t h[8]; bf16x8_t v; } part[3];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = kb + e < t.r ? u[a][e] : 0.f;
        const bool finite = fabsf(x) <= 3.4028235e38f;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          part[q].h[e] = finite ? (bf16_t)(__float_as_uint(x) >> 16) : f32_to_bf16(x);
          x = finite ? x - bf16_to_f32(part[q].h[e]) : 0.f;  // exact; an infinity has no remainder
        }
      }
#pragma unroll
      for (int q = 2; q >= 0; --q)
#pragma unroll
        for (int b = 0; b < T::TN; ++b)
          acc.v[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q == 0 ? fb[b] : fin[b], part[q].v, acc.v[a][b], 0, 0, 0);
    }
  }
#pragma unroll
  for (int a = 0; a < T::TM; ++a)
#pragma unroll
    for (int b = 0; b < T::TN; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc.v[a][b][e] *= t.gamma;
#endif
}

// One macro tile: main loop, then the store epilogue.  `term` (TERM): added before the main loop, while nothing else
// of the tile is in registers.
// Wide tiles: K-contiguous operands, B row-major (ldb) or, B_BLK, in blocks of 32 k-values; others: K-major operands.
template <class T, bool OUT_BF16, bool MASK_A_K = false, bool B_BLK = false, bool TERM = false>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ B,
                                          int64_t ldb, int M, int N, int K, int K_a, void* __restrict__ Cout,
                                          int64_t ldc, int m0, int n0, unsigned char* lds,
                                          const RankTerm& term = RankTerm()) {
  gemm::Accum<T> acc;
#pragma unroll
  for (int a = 0; a < T::TM; ++a)
#pragma unroll
    for (int b = 0; b < T::TN; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc.v[a][b][e] = 0.f;
  if constexpr (TERM) add_rank_term<T>(acc, term, M, N, m0, n0);
  if constexpr (T::WIDE)
    gemm::mainloop_wide<T, MASK_A_K, B_BLK>(A, lda, B, ldb, M, N, K, m0, n0, lds, acc, K_a);
  else
    gemm::mainloop<T>(A, lda, B, ldb, M, N, K, m0, n0, lds, acc);
  store_tile<T, OUT_BF16, T::LDS_BYTES>(acc, M, N, Cout, ldc, m0, n0, lds);
}

template <class T, bool OUT_BF16, bool MASK_A_K = false, bool B_BLK = false>
__global__ __launch_bounds__(T::NT) void gemm_bf16_fast_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                const bf16_t* __restrict__ B, int64_t ldb, int M, int N,
                                                                int K, int K_a, void* __restrict__ Cout, int64_t ldc,
                                                                int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::LDS_BYTES];
  int tile_m, tile_n;
  gemm::tile_of_block(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  gemm_tile<T, OUT_BF16, MASK_A_K, B_BLK>(A, lda, B, ldb, M, N, K, K_a, Cout, ldc, tile_m * T::BM, tile_n * T::BN, lds);
}

// C = A . B^T + gamma U . M^T: the QAT-LoRA layer's product and its LoRA path in one pass over C.
template <class T, bool MASK_A_K>
__global__ __launch_bounds__(T::NT) void gemm_bf16_nt_rank_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                   const bf16_t* __restrict__ B, int M, int N, int K,
                                                                   int K_a, bf16_t* __restrict__ C, int64_t ldc,
                                                                   int tiles_m, int tiles_n, RankTerm term) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::LDS_BYTES];
  int tile_m, tile_n;
  gemm::tile_of_block(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  gemm_tile<T, true, MASK_A_K, true, true>(A, lda, B, 0, M, N, K, K_a, C, ldc, tile_m * T::BM,
                                                         tile_n * T::BN, lds, term);
}

// One (tile, k-slice) of a product with few tiles: slice blockIdx.y of gridDim.y takes a run of whole stage pairs of
// the k range and leaves its binary32 tile in part[slice][M][N].  K-contiguous operands; B row-major (ldb) or, B_BLK, in
// blocks of 32 k-values.
template <class T, bool MASK_A_K, bool B_BLK>
__global__ __launch_bounds__(T::NT) void gemm_bf16_nt_splitk_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                     const bf16_t* __restrict__ B, int64_t ldb, int M,
                                                                     int N, int K, int K_a, float* __restrict__ part,
                                                                     int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::LDS_BYTES];
  int tile_m, tile_n;
  gemm::tile_of_block(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int slices = gridDim.y, slice = blockIdx.y;
  const int pairs = ((K + T::BK - 1) / T::BK + 1) / 2;
  const int k0 = (int)((int64_t)pairs * slice / slices) * (2 * T::BK);
  int k1 = (int)((int64_t)pairs * (slice + 1) / slices) * (2 * T::BK);
  if (k1 > K) k1 = K;
  // rows of A end at K_a: inside the last slice, at or past the end of every other
  const int ka = (K_a < k1 ? K_a : k1) - k0;
  const bf16_t* Bs = B_BLK ? B + (int64_t)(k0 / T::BK) * N * T::BK : B + k0;
  gemm_tile<T, false, MASK_A_K, B_BLK>(A + k0, lda, Bs, ldb, M, N, k1 - k0, ka,
                                                     part + (int64_t)slice * M * N, N, tile_m * T::BM, tile_n * T::BN, lds);
}

// The same for K-major operands (rows = k): slice blockIdx.y takes a run of whole stages.
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_bf16_kmajor_splitk_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                         const bf16_t* __restrict__ B, int64_t ldb,
                                                                         int M, int N, int K, float* __restrict__ part,
                                                                         int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::LDS_BYTES];
  int tile_m, tile_n;
  gemm::tile_of_block(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int slices = gridDim.y, slice = blockIdx.y;
  const int nk = (K + T::BK - 1) / T::BK;
  const int k0 = (int)((int64_t)nk * slice / slices) * T::BK;
  int k1 = (int)((int64_t)nk * (slice + 1) / slices) * T::BK;
  if (k1 > K) k1 = K;
  gemm_tile<T, false>(A + (int64_t)k0 * lda, lda, B + (int64_t)k0 * ldb, ldb, M, N, k1 - k0,
                                                k1 - k0, part + (int64_t)slice * M * N, N, tile_m * T::BM,
                                                tile_n * T::BN, lds);
}

// C[m, n] = bf16(sum over the slices, in slice order, of part[slice][m][n]); N % 4 == 0, four columns per thread.
__device__ __forceinline__ void splitk_sum(int64_t block, const float* __restrict__ part, int slices, int64_t M, int64_t N,
                                           bf16_t* __restrict__ C, int64_t ldc) {
  const int64_t q = block * 256 + threadIdx.x;
  if (q >= M * N / 4) return;
  float4 v = reinterpret_cast<const float4*>(part)[q];
  for (int s = 1; s < slices; ++s) {
    const float4 w = reinterpret_cast<const float4*>(part + (int64_t)s * M * N)[q];
    v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
  }
  const int64_t m = q * 4 / N, n = q * 4 - m * N;
  const float f[4] = {v.x, v.y, v.z, v.w};
  store4(C + m * ldc + n, f);
}
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float* __restrict__ part, int slices, int64_t M, int64_t N,
                                                         bf16_t* __restrict__ C, int64_t ldc) {
  splitk_sum((int64_t)blockIdx.x, part, slices, M, N, C, ldc);
}

// The same with the partial sums of dA and dB, which the weight-gradient kernel has left, added by the workgroups after the
// first `own`: either launch alone is 5 us, most of it latency (301 tokens, 4096 x 4096, rank 16: a training step of 126.7 us
// takes 124.1 in one).
__global__ __launch_bounds__(256) void splitk_sum_and_partials_kernel(const float* __restrict__ part, int slices, int64_t M,
                                                                      int64_t N, bf16_t* __restrict__ C, int64_t ldc, int own,
                                                                      TwoPartials sums) {
  __shared__ float4 slice_sum[3][64];
  if ((int)blockIdx.x < own) splitk_sum((int64_t)blockIdx.x, part, slices, M, N, C, ldc);
  else reduce_two_block(sums, (int)blockIdx.x - own, slice_sum);
}

// Matrix-core-only loop with the GEMM's register shape (4 x 4 accumulator tiles, 8 fragments per wave) and
// no memory traffic inside the loop: what the matrix pipeline sustains on this chip for the given data.
__global__ __launch_bounds__(256) void mfma_probe_kernel(const bf16_t* __restrict__ data, int iterations,
                                                         float* __restrict__ sink) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef gemm::bf16x8_t bf16x8_t;
  typedef gemm::f32x16_t f32x16_t;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bf16x8_t fa[4], fb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // 8 fragments of 16 bytes per lane out of the first 64 KiB of data
    fa[q] = *reinterpret_cast<const bf16x8_t*>(data + ((wave * 8 + q) * 64 + lane) * 8);
    fb[q] = *reinterpret_cast<const bf16x8_t*>(data + ((wave * 8 + 4 + q) * 64 + lane) * 8);
  }
  f32x16_t acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
  for (int it = 0; it < iterations; ++it) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b], fa[a], acc[a][b], 0, 0, 0);
  }
  float t = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) t += acc[a][b][e];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = t;
#endif
}

}  // namespace

double launch_mfma_probe(const bf16_t* data, int iterations, int workgroups, float* sink, hipStream_t stream) {
  hipLaunchKernelGGL(mfma_probe_kernel, dim3((unsigned)workgroups), dim3(256), 0, stream, data, iterations, sink);
  return (double)workgroups * 4.0 * (double)iterations * 16.0 * (2.0 * 32 * 32 * 16);
}

int device_compute_units() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

namespace {

// Macro tiles of the K-contiguous products.
//   NtFull     256 x 256, 8 waves (2 x 4, two per SIMD, 128 x 64 each): a second wave on the SIMD keeps the matrix pipe busy
//              while the first waits for a barrier or for operands (1.5 % over 2 x 2)
//   NtHalf     128 x 256, 4 waves (64 x 128 each): 4/7 of a full tile's time for half its work
//   NtQuarter  128 x 128, 4 waves (64 x 64 each): 2/5 of a full tile's time for a quarter of it
// the smaller ones for products whose full tiles leave compute units idle.  X and dY come in rows of 128 bytes, the rings
// fill the LDS (mainloop_wide).  Against loads of 64-byte rows (us, kernel times in the step): 2048 x 4096 x 11008 in half
// tiles 173 -> 160, 2048 x 11008 x 4096 197 -> 172, 301 x 4096 x 4096 in quarter tiles and two slices 21.1 -> 19.0; steps of
// both directions: 4096 x 11008 x 4096 988 -> 967, 512 x 4096 x 4096 132 -> 122, 1000 x 2048 x 2048 83.7 -> 79.7.
typedef gemm::WideTile<256, 256, 3, 4, 4> NtFull;
typedef gemm::WideTile<128, 256, 4, 6, 2> NtHalf;
typedef gemm::WideTile<128, 128, 5, 8, 2> NtQuarter;
enum NtForm { kNtFull, kNtHalf, kNtQuarter };

template <class F> int64_t nt_tiles(int64_t M, int64_t N) {
  return ((M + F::BM - 1) / F::BM) * ((N + F::BN - 1) / F::BN);
}

// How far the layer's weight operand has left the memory-side cache (256 MB) by the time the product reads it, 0 .. 1.
// In a training step the merge pass reads W0 from memory and writes Wq right before the forward product (4 N K bytes):
// felt from 40 M weights on, complete at 107 M.  Between it and the dX product (`late`) lie the weight-gradient kernel and
// its factor array, another 4 N K bytes: from 30 M on, complete at 60 M.  A stage's loads then take about 2.6 us instead of
// 1.3, which a full tile's rings (operand B three stages of 0.52 us ahead, A two units of two stages) nearly cover and the
// smaller tiles' (0.28, 0.19 us a stage) do not: per 1024 k a full / half / quarter tile takes 16.6 / 9 / 6.2 us from the cache
// and 20.6 / 15 .. 17 / 12 from memory (late, quarter tiles come off better than that: 9).
double nt_uncached(int64_t N, int64_t K, bool late) {
  const double weights = (double)N * (double)K;
  const double c = late ? (weights - 30e6) / 30e6 : (weights - 40e6) / 67e6;
  return c < 0.0 ? 0.0 : c > 1.0 ? 1.0 : c;
}

// One pass over k: which tile.  In us (full / half / quarter; their numbers on 256 compute units; M x N x K), as is what follows
// up to nt_plan measured with X and dY in rows of 64 bytes; with whole cache lines all three forms are 4 to 10 % faster, and
// constants fitted to that would gain 0.4 % at most:
//    32,   64,  128   72 /  41 / 29    512 x  4096 x 4096      172,  344,  688    80 /  94 /  92   1024 x 11008 x 4096
//    32,   64,  128   39 /  23 / 15   1000 x  2048 x 2048      192,  384,  768    84 /  95 /   -   3000 x  4096 x 4096
//    64,  128,  256   73 /  42 / 33   1024 x  4096 x 4096      240,  440,  880   118 / 123 / 156   1328 x 10224 x 5120
//    86,  172,  344   73 /  45 / 60    512 x 11008 x 4096      256,  512, 1024   100 / 111 /   -   4096 x  4096 x 4096
//   128,  256,  512   74 /  57 / 64   2048 x  4096 x 4096      344,  688, 1376   169 / 152 /   -   2048 x 11008 x 4096
//    99,  198,  396  158 / 103 / 133  2179 x  2784 x 9216      688, 1376, 2752   271 / 309 /   -   4096 x 11008 x 4096
// i.e. rounds of tiles over the units, a round of full / half / quarter tiles counting 70 : 40 : 29; short products, where
// the fill of the ring and the store count for more, 22 : 16 : 13 (K = 1024, with the merge pass: 3000 x 8192 68 / 74,
// 2048 x 11008 71 / 75, 4096 x 5120 63 / 66); weights out of the cache up to 87 : 60 : 44 (with the merge pass, 768 x
// 28672 x 8192 574 / 628, 640 x 11008 x 11008 335 / 298, 1300 x 11008 x 11008 573 / 443, 2048 x 11008 x 11008 587 / 635).
NtForm nt_one_pass_form(int64_t M, int64_t N, int64_t K, bool late) {
  const int64_t cus = device_compute_units();
  auto rounds = [&](int64_t tiles) { return (double)((tiles + cus - 1) / cus); };
  const bool is_short = K < 1536;
  const double c = nt_uncached(N, K, late);
  const double full = ((is_short ? 22.0 : 70.0) + 17.0 * c) * rounds(nt_tiles<NtFull>(M, N));
  const double half = ((is_short ? 16.0 : 40.0) + 20.0 * c) * rounds(nt_tiles<NtHalf>(M, N));
  const double quarter = ((is_short ? 13.0 : 29.0) + 15.0 * c) * rounds(nt_tiles<NtQuarter>(M, N));
  if (quarter < half && quarter < full) return kNtQuarter;
  return half < full ? kNtHalf : kNtFull;
}

// Products of few tiles (full ones on at most half of the compute units): half or quarter tiles in k-slices, at most one
// (tile, slice) per compute unit, each slice at least four stage pairs (256 k) long, at most 8, no more than keep the
// partial tiles (slices x M x N x 4 bytes, written and read once) within the size of operand B (N x K x 2 bytes), nor more
// than fit the slices of full tiles; of those the form with the least estimated time: 9 us (half) or 6.2 us (quarter
// tiles) per 1024 k of a slice, and beyond one slice 6 us for the second launch and the partial tiles at 5 TB/s.
// Estimated, measured (us):
//   301 x 4096 x 4096    quarter x 2 22, 23   half x 4 23, 25     512 x 4096 x 11008  half x 4 44, 52   quarter x 2 46, 52
//   512 x 4096 x 4096    quarter x 2 25, 26   half x 3 28, 29     100 x 4096 x 4096   quarter x 5 14, 15   half x 6 16, 19
//   400 x 2048 x 2048    quarter x 1 12, 13   half x 3 19, 21    1024 x 4096 x 4096   quarter x 1 25, 33   half x 1 36, 42
// (256 x 256 tiles in as many slices as fill the chip took 35, 63, 38, 22, 25 and 54.)
// Weights out of the cache take full tiles into account, at the times of nt_uncached.  Measured in us, full tiles / the
// smaller ones as chosen from their cached times: merge pass and product 512 x 9600 x 9600 190 / 237, 256 x 11008 x 11008
// 191 / 234, 640 x 7168 x 11008 183 / 212, 1024 x 5120 x 13824 210 / 244, 512 x 8192 x 11008 182 / 200, but 64 x 4096 x 28672
// 183 / 161, 300 x 7168 x 11008 158 / 144; training steps with the dX product in either, 768 x 4096 x 11008 405 / 430,
// 768 x 7168 x 7168 452 / 480, 1500 x 3072 x 11008 465 / 493.
struct NtPlan {
  NtForm form;
  int slices;
};
NtPlan nt_plan(int64_t M, int64_t N, int64_t K, bool late) {
  const NtPlan one_pass = {nt_one_pass_form(M, N, K, late), 1};
  const int64_t full = nt_tiles<NtFull>(M, N), cus = device_compute_units();
  if (full <= 0 || 2 * full > cus) return one_pass;
  const int64_t pairs = ((K + 31) / 32 + 1) / 2;
  int64_t most = cus / full;
  if (most > pairs / 4) most = pairs / 4;
  if (most > 8) most = 8;
  if (most > K / (2 * M)) most = K / (2 * M);
  if (most < 1) most = 1;
  const double c = nt_uncached(N, K, late);
  NtPlan best = one_pass;
  double best_us = 1e30;
  auto consider = [&](NtForm form, int64_t tiles, double us_per_1024) {
    const double pass_us = us_per_1024 * (double)K / 1024.0 * (double)((tiles + cus - 1) / cus);
    for (int s = 1; s <= most && (s == 1 || tiles * s <= cus); ++s) {
      const double us = pass_us / s + (s > 1 ? 6.0 + (double)s * (double)M * (double)N * 8.0 / 5e6 : 0.0);
      if (us < best_us) {
        best = {form, s};
        best_us = us;
      }
    }
  };
  consider(kNtQuarter, nt_tiles<NtQuarter>(M, N), 6.2 + (late ? 2.5 : 5.8) * c);
  consider(kNtHalf, nt_tiles<NtHalf>(M, N), 9.0 + 6.5 * c);
  if (c > 0.0) consider(kNtFull, full, 16.6 + 4.0 * c);
  return best;
}

}  // namespace

int gemm_nt_splitk_slices(int64_t M, int64_t N, int64_t K, bool late) { return nt_plan(M, N, K, late).slices; }

namespace {

// `f` with the tile type and whether rows of A need masking past K_a, where that is no multiple of 64 (an instance of its
// own, so that the usual shapes do not pay for the selection)
template <class Fn> void nt_dispatch(NtForm form, bool mask, Fn&& f) {
  auto with_mask = [&](auto tile) {
    if (mask) f(tile, std::true_type());
    else f(tile, std::false_type());
  };
  if (form == kNtQuarter) with_mask(NtQuarter());
  else if (form == kNtHalf) with_mask(NtHalf());
  else with_mask(NtFull());
}

}  // namespace

void launch_gemm_bf16_nt(const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int64_t M, int64_t N,
                         int64_t K, int64_t K_a, bf16_t* C, int64_t ldc, hipStream_t stream, float* partial, bool late,
                         const TwoPartials* sums) {
  NtPlan plan = nt_plan(M, N, K, late);
  if (plan.slices > 1 && !partial) plan = {nt_one_pass_form(M, N, K, late), 1};
  const int slices = plan.slices;
  nt_dispatch(plan.form, K_a % 64 != 0, [&](auto tile, auto mask) {
    typedef decltype(tile) F;
    constexpr bool MASK = decltype(mask)::value;
    const int tiles_m = (int)((M + F::BM - 1) / F::BM), tiles_n = (int)((N + F::BN - 1) / F::BN);
    if (slices > 1) {
      hipLaunchKernelGGL((gemm_bf16_nt_splitk_kernel<F, MASK, true>), dim3((unsigned)(tiles_m * tiles_n), (unsigned)slices),
                         dim3(F::NT), 0, stream, A, lda, B, ldb, (int)M, (int)N, (int)K, (int)K_a, partial, tiles_m, tiles_n);
      const int own = (int)((M * N / 4 + 255) / 256);
      if (sums)
        hipLaunchKernelGGL(splitk_sum_and_partials_kernel, dim3((unsigned)(own + two_partials_blocks(*sums))), dim3(256), 0,
                           stream, partial, slices, M, N, C, ldc, own, *sums);
      else
        hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)own), dim3(256), 0, stream, partial, slices, M, N, C, ldc);
    } else {
      hipLaunchKernelGGL((gemm_bf16_fast_kernel<F, true, MASK, true>),
                         dim3((unsigned)(tiles_m * tiles_n)), dim3(F::NT), 0, stream, A, lda, B, ldb, (int)M, (int)N,
                         (int)K, (int)K_a, (void*)C, ldc, tiles_m, tiles_n);
    }
  });
}

void launch_gemm_bf16_nt_rank(const bf16_t* A, int64_t lda, const bf16_t* B, int64_t M, int64_t N, int64_t K, int64_t K_a,
                              bf16_t* C, int64_t ldc, const RankTerm& term, hipStream_t stream) {
  nt_dispatch(nt_one_pass_form(M, N, K, false), K_a % 64 != 0, [&](auto tile, auto mask) {
    typedef decltype(tile) F;
    const int tiles_m = (int)((M + F::BM - 1) / F::BM), tiles_n = (int)((N + F::BN - 1) / F::BN);
    hipLaunchKernelGGL((gemm_bf16_nt_rank_kernel<F, decltype(mask)::value>), dim3((unsigned)(tiles_m * tiles_n)),
                       dim3(F::NT), 0, stream, A, lda, B, (int)M, (int)N, (int)K, (int)K_a, C, ldc, tiles_m, tiles_n, term);
  });
}

void launch_gemm_bf16_kmajor_f32(const bf16_t* A, int64_t lda, const bf16_t* B, int64_t ldb, int64_t M, int64_t N,
                                 int64_t K, float* C, int64_t ldc, hipStream_t stream) {
  typedef gemm::Tile<256, 256, 32, 4> F;
  const int tiles_m = (int)((M + F::BM - 1) / F::BM), tiles_n = (int)((N + F::BN - 1) / F::BN);
  hipLaunchKernelGGL((gemm_bf16_fast_kernel<F, false>), dim3((unsigned)(tiles_m * tiles_n)),
                     dim3(F::NT), 0, stream, A, lda, B, ldb, (int)M, (int)N, (int)K, (int)K, (void*)C, ldc, tiles_m,
                     tiles_n);
}

// k-slices of the two thin products of the masked form (dB = dWm A^T: [o, r], k = i; dA = B^T dWm: [r, i], k = o): each
// has o / 256 or i / 256 tiles only, one tile row or column, and a long k range; as many slices as put a workgroup on
// every compute unit, each at least 8 stages long, at most 8 (and 32 MiB of partial results).
void dw_masked_product_slices(const LayerDims& d, int* slices_a, int* slices_b) {
  const int64_t cus = device_compute_units();
  auto pick = [&](int64_t tiles, int64_t stages, int64_t out_elems) {
    int64_t s = cus / (tiles > 0 ? tiles : 1);
    if (s > stages / 8) s = stages / 8;
    if (s > 8) s = 8;
    while (s > 1 && s * out_elems * 4 > (32ll << 20)) --s;
    return (int)(s < 1 ? 1 : s);
  };
  const int64_t tr = (d.r + 255) / 256;
  *slices_b = pick(((d.o + 255) / 256) * tr, (d.i + 31) / 32, d.o * d.r);
  *slices_a = pick(tr * ((d.i + 255) / 256), (d.o + 31) / 32, (int64_t)d.r * d.i);
}

void launch_dw_masked_products(const LayerDims& d, const bf16_t* dWm, const bf16_t* A, const bf16_t* B, float* rawA,
                               float* rawB, hipStream_t stream) {
  int sa = 1, sb = 1;
  dw_masked_product_slices(d, &sa, &sb);
  // rawB [sb][o, r] = dWm [o, i] . A [r, i]^T: both K-contiguous, k = i (a multiple of 32).  Bound
  // by reading dWm once.  Ranks up to 128 in 128 x 128 tiles: twice the workgroups, and half of a tile's columns at rank 64
  // instead of a quarter (rank 64 on 4096 x 11008: 22 us against 35 in 256 x 256 tiles).
  auto thin_b = [&](auto tile, auto mask) {
    typedef decltype(tile) F;
    const int tiles_m = (int)((d.o + F::BM - 1) / F::BM), tiles_n = (d.r + F::BN - 1) / F::BN;
    hipLaunchKernelGGL((gemm_bf16_nt_splitk_kernel<F, decltype(mask)::value, false>), dim3((unsigned)(tiles_m * tiles_n), (unsigned)sb),
                       dim3(F::NT), 0, stream, dWm, d.i, A, d.i, (int)d.o, d.r, (int)d.i, (int)d.i, rawB, tiles_m, tiles_n);
  };
  nt_dispatch(d.r <= 128 ? kNtQuarter : kNtFull, d.i % 64 != 0, thin_b);
  // rawA [sa][r, i] = B [o, r]^T . dWm [o, i]: both K-major, k = o.  Bound by reading dWm once; with all 256 columns of a tile
  // multiplied, whatever the rank, the matrix ops of a slice took 11 us at full rate, so up to 128 ranks the waves share out 64
  // or 128 of them (rank 64 on 4096 x 11008: 27.1 us -> 20.8, steps of drawn layers at ranks 40 .. 128 1.02 times as fast,
  // the sums the same).
  auto thin_a = [&](auto tile) {
    typedef decltype(tile) F;
    const int tiles_m = (d.r + F::BM - 1) / F::BM, tiles_n = (int)((d.i + F::BN - 1) / F::BN);
    hipLaunchKernelGGL((gemm_bf16_kmajor_splitk_kernel<F>), dim3((unsigned)(tiles_m * tiles_n), (unsigned)sa), dim3(F::NT),
                       0, stream, B, (int64_t)d.r, dWm, d.i, d.r, (int)d.i, (int)d.o, rawA, tiles_m, tiles_n);
  };
  if (d.r <= 64) thin_a(gemm::Tile<256, 256, 32, 4, 64>());
  else if (d.r <= 128) thin_a(gemm::Tile<256, 256, 32, 4, 128>());
  else thin_a(gemm::Tile<256, 256, 32, 4>());
}

}  // namespace l4q

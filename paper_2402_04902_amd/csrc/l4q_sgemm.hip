// Binary32 products on the matrix cores:  C[m,n] = scale * sum_k A[m,k] B[k,n]  (+ C[m,n] with accumulate), each operand
// with one unit-stride axis.  Serves the binary32 mode end to end (forward, dX, dWq, dB) and the LoRA products of the
// binary32 QAT-LoRA layer.
//
// v_mfma_f32_32x32x2_f32 multiplies and adds in binary32 like the vector unit, at the vector unit's peak rate, but one
// instruction is 64 cycles of work on two registers of operands, so neither instruction issue nor LDS reads are in the
// way.  (The vector kernel this replaces, 64 x 64 tiles with 4 x 4 outputs per thread, reached 26 TFLOP/s: two LDS
// reads per four multiply-adds, element-wise loads, one tile per compute unit and nothing in flight across its barriers.)
//
// Operand fragments.  A matrix op takes two k-values, one per half-wave, and the order of k in a sum is free as long as
// both operands agree: op j of four contracts k = j (lanes 0..31) and k = 4 + j (lanes 32..63) of a run of 8.  A lane of
// a K-contiguous operand therefore reads 4 consecutive k of its row (one 16-byte read); a K-major operand is read one
// float per op, 32 consecutive columns per half-wave.  No transposition in either form.
#include "l4q_device.h"
#include "l4q_gemm_core.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));  // 16-byte global access at 4-byte alignment: rows
                                                                         // of an odd number of floats
typedef gemm::f32x16_t f32x16_t;

struct SgemmArgs {
  const float* A;
  const float* B;
  float* C;
  int64_t lda, ldb, ldc;  // stride of the axis that is not unit-stride
  int64_t M, N, K;
  float scale;
  bool accumulate;
};

__device__ __forceinline__ void store_out(const SgemmArgs& a, int64_t m, int64_t n, float v) {
  float* dst = a.C + m * a.ldc + n;
  *dst = a.accumulate ? *dst + a.scale * v : a.scale * v;
}

// ------------------------------------------------------------------ tiled form
// KG groups of 4 waves (2 x 2) on the same tile, group q taking the k-steps q, q + KG, ..., their sums added at the end; k in
// steps of 32, the next two steps' operands travelling to registers while the current one is
// multiplied out of LDS; two LDS buffers, one barrier per step.  For operands that are not whole 16-byte pieces, and for
// products of few steps.  K-contiguous operands lie in LDS as rows
// of 32 k + 4 floats of padding (16-byte reads of 16 consecutive rows meet all banks once), K-major ones as they come.
constexpr int SG_BK = 32;
constexpr int SG_KPITCH = SG_BK + 4;

// One operand tile of ROWS rows (its M or N axis) x 32 k-values, ROWS / 8 floats per thread.
template <int ROWS, bool KMAJOR>
struct SgemmOperand {
  static constexpr int NV = ROWS * SG_BK / 4 / 256;  // 16-byte pieces per thread
  static constexpr int PITCH = KMAJOR ? ROWS + 4 : SG_KPITCH;
  static constexpr int FLOATS = KMAJOR ? SG_BK * PITCH : ROWS * PITCH;
  f32x4u_t v[NV];

  // piece e of thread tid: row and first column of 4 consecutive elements along the unit-stride axis
  __device__ static void place(int tid, int e, int& row, int& col) {
    constexpr int PER_ROW = (KMAJOR ? ROWS : SG_BK) / 4;
    const int q = tid + e * 256;
    row = q / PER_ROW;
    col = (q % PER_ROW) * 4;
  }
  // P: the operand; r0 .. extent: its M / N axis; k0 .. K
  __device__ void load(const float* __restrict__ P, int64_t ld, int64_t r0, int64_t extent, int64_t k0, int64_t K, int tid) {
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      int row, col;
      place(tid, e, row, col);
      const int64_t outer = (KMAJOR ? k0 : r0) + row, outer_end = KMAJOR ? K : extent;
      const int64_t inner = (KMAJOR ? r0 : k0) + col, inner_end = KMAJOR ? extent : K;
      f32x4u_t t = {0.f, 0.f, 0.f, 0.f};
      if (outer < outer_end) {
        const float* p = P + outer * ld + inner;
        if (inner + 3 < inner_end) t = *reinterpret_cast<const f32x4u_t*>(p);
        else {
          if (inner < inner_end) t[0] = p[0];
          if (inner + 1 < inner_end) t[1] = p[1];
          if (inner + 2 < inner_end) t[2] = p[2];
        }
      }
      v[e] = t;
    }
  }
  __device__ void store(float* lds, int tid) const {
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      int row, col;
      place(tid, e, row, col);
      *reinterpret_cast<float4*>(lds + row * PITCH + col) = make_float4(v[e][0], v[e][1], v[e][2], v[e][3]);
    }
  }
  // the 4 k-values of run kk (8 k-values) this lane feeds to the 4 matrix ops, for row `row` of the tile
  __device__ static void fragment(const float* lds, int row, int kk, int half, float (&f)[4]) {
    if constexpr (KMAJOR) {
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = lds[(kk * 8 + half * 4 + j) * PITCH + row];
    } else {
      const float4 t = *reinterpret_cast<const float4*>(lds + row * PITCH + kk * 8 + half * 4);
      f[0] = t.x; f[1] = t.y; f[2] = t.z; f[3] = t.w;
    }
  }
};

// The waves' accumulators to C: with two groups, group 1's sums through LDS to group 0 first.
template <int TM, int TN, int KG>
__device__ __forceinline__ void store_tile(const SgemmArgs& a, f32x16_t (&acc)[TM][TN], float* lds, int64_t mw, int64_t nw, int group,
                                           int tid, int l32, int half) {
  if constexpr (KG == 2) {
    __syncthreads();
    float* sums = lds + tid * 17;  // (odd pitch: no bank conflicts)
    if (group == 1) {
#pragma unroll
      for (int e = 0; e < 16; ++e) sums[e] = acc[0][0][e];
    }
    __syncthreads();
    if (group == 1) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][0][e] += sums[e];
  }
  // accumulator: lane = column n, register e = row 8 (e / 4) + 4 half + e % 4
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) {
      const int64_t n = nw + y * 32 + l32;
      if (n >= a.N) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int64_t m = mw + x * 32 + 8 * (e / 4) + 4 * half + (e % 4);
        if (m < a.M) store_out(a, m, n, acc[x][y][e]);
      }
    }
}

template <int BM, int BN, int KG, bool A_KM, bool B_KM>
__global__ __launch_bounds__(256 * KG, KG == 2 ? 4 : 1) void sgemm_tile_kernel(SgemmArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef SgemmOperand<BM, A_KM> OpA;
  typedef SgemmOperand<BN, B_KM> OpB;
  constexpr int STAGE = OpA::FLOATS + OpB::FLOATS;
  constexpr int TM = BM / 64, TN = BN / 64;  // 32 x 32 accumulator tiles per wave
  static_assert(KG == 1 || (KG == 2 && BM == 64 && BN == 64), "the second group's sums fit its buffers");
  __shared__ __align__(16) float lds[2 * KG * STAGE];
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
  int tm, tn;
  gemm::tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;

  OpA oa[2];
  OpB ob[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    oa[p].load(a.A, a.lda, m0, a.M, (p * KG + group) * SG_BK, a.K, tid);
    ob[p].load(a.B, a.ldb, n0, a.N, (p * KG + group) * SG_BK, a.K, tid);
  }
  for (int64_t k0 = 0; k0 < a.K; k0 += 2 * KG * SG_BK) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {  // steps of one buffer and register set each
      if (p == 1 && k0 + KG * SG_BK >= a.K) break;  // (the same for all groups: a step past K multiplies zeros)
      float* la = lds + (group * 2 + p) * STAGE;
      float* lb = la + OpA::FLOATS;
      oa[p].store(la, tid);
      ob[p].store(lb, tid);
      __syncthreads();  // (the buffer's previous readers passed the barrier of the step between)
      const int64_t next = k0 + ((p + 2) * KG + group) * SG_BK;
      if (k0 + (p + 2) * KG * SG_BK < a.K) {
        oa[p].load(a.A, a.lda, m0, a.M, next, a.K, tid);
        ob[p].load(a.B, a.ldb, n0, a.N, next, a.K, tid);
      }
#pragma unroll
      for (int kk = 0; kk < SG_BK / 8; ++kk) {
        float fa[TM][4], fb[TN][4];
#pragma unroll
        for (int x = 0; x < TM; ++x) OpA::fragment(la, wm + x * 32 + l32, kk, half, fa[x]);
#pragma unroll
        for (int y = 0; y < TN; ++y) OpB::fragment(lb, wn + y * 32 + l32, kk, half, fb[y]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[x][j], fb[y][j], acc[x][y], 0, 0, 0);
      }
    }
  }
  store_tile<TM, TN, KG>(a, acc, lds, m0 + wm, n0 + wn, group, tid, l32, half);
#endif
}

// ------------------------------------------------------------------ tiled form, operands straight to LDS
// The tiled form for operands of whole 16-byte pieces.  Binary32 matrix ops take the vector unit's time (a loop of each runs
// in the sum of their times), so what the form above spends on bounds, addresses and copies through registers, about 50
// vector ops and 8 branches per step beside 16 matrix ops, comes off its rate.  Here a step's operands travel memory -> LDS
// (buffer_load ... lds) at offsets that a lane computes once, into the buffer that the previous step has left, one barrier
// per step; the loop has no vector ops but the matrix ops.  1000 x 2048 x 2048 inside a training step, the three
// orientations: 103 / 102 / 102 us -> 85 / 81 / 89; 512 x 2048 x 1024 28.4 -> 24.4; 2048 x 4096 x 2048 in 128-wide tiles 307 -> 288,
// 4096 x 2048 x 2048 with both K-major 322 -> 277, 2048 x 2048 x 4096 in 64-wide ones 348 -> 287.  The sums and their order are the
// same.  (The line to the sliced form stays where it is: 96 tiles, K = 1024 23.0 / 22.1 here / sliced, 128 tiles, K = 2048 41.8 / 41.6,
// 64 tiles, K = 1024 22.4 / 13.9.)  K-contiguous rows: 8 pieces, piece p of row m at
// position p ^ (m % 8) (8 consecutive lanes meet all banks); K-major rows: pieces of rows with bit 2 of k set are moved by 32
// columns, so that the two half-waves of a read, 4 rows apart, meet different banks.
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int ROWS, bool KMAJOR>
struct SgemmPieces {
  static constexpr int NV = ROWS / 32;           // loads per wave and step: 1 KiB each
  static constexpr int BYTES = ROWS * SG_BK * 4;
  __amdgpu_buffer_rsrc_t rs;
  unsigned voff[NV];
  int kpos[NV];      // this lane's k within the step
  unsigned step_bytes;

  __device__ void init(const float* P, int64_t ld, int64_t r0, int64_t extent, int wave, int lane) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P + (KMAJOR ? r0 : r0 * ld)), 0, 0x7FFFFFFF, 0x00020000);
    step_bytes = (unsigned)(KMAJOR ? SG_BK * ld * 4 : SG_BK * 4);
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const int idx = (wave * NV + e) * 64 + lane;
      constexpr int PER = KMAJOR ? ROWS / 4 : SG_BK / 4;
      const int outer = idx / PER;
      const int piece = (idx % PER) ^ (KMAJOR ? 8 * ((outer >> 2) & 1) : outer & 7);
      const int64_t row = r0 + (KMAJOR ? 4 * piece : outer);  // (K-major: extents are whole pieces)
      kpos[e] = KMAJOR ? outer : 4 * piece;
      voff[e] = row < extent ? (unsigned)(((int64_t)outer * ld + 4 * piece) * 4) : gemm::OOB_OFFSET;
    }
  }
  // step `step` of the operand's K values into lds; what lies from K on comes as zeros
  __device__ __forceinline__ void load(unsigned char* lds, int step, int64_t K, int wave) const {
    const int left = (int)(K - (int64_t)step * SG_BK);
    if (left >= SG_BK) {
#pragma unroll
      for (int e = 0; e < NV; ++e)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (gemm::lds_ptr_t)(lds + (wave * NV + e) * 1024), 16, voff[e],
                                                 (int)(step * step_bytes), 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < NV; ++e)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (gemm::lds_ptr_t)(lds + (wave * NV + e) * 1024), 16,
                                                 kpos[e] < left ? voff[e] + step * step_bytes : gemm::OOB_OFFSET, 0, 0, 0);
    }
  }
  // the 4 k-values of run kk (8 k-values) this lane feeds to the 4 matrix ops, for row `row` of the tile
  __device__ static __forceinline__ f32x4_t fragment(const unsigned char* lds, int row, int kk, int half) {
    f32x4_t f;
    if constexpr (KMAJOR) {
      const float* p = reinterpret_cast<const float*>(lds) + (kk * 8 + half * 4) * ROWS + (row ^ (32 * half));
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = p[j * ROWS];
    } else {
      f = *reinterpret_cast<const f32x4_t*>(lds + row * 128 + (((2 * kk + half) ^ (row & 7)) << 4));
    }
    return f;
  }
};

template <int BM, int BN, int KG, bool A_KM, bool B_KM>
__global__ __launch_bounds__(256 * KG, KG == 2 ? 4 : 2) void sgemm_dma_kernel(SgemmArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef SgemmPieces<BM, A_KM> OpA;
  typedef SgemmPieces<BN, B_KM> OpB;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES;
  constexpr int TM = BM / 64, TN = BN / 64;  // 32 x 32 accumulator tiles per wave
  static_assert(KG == 1 || (KG == 2 && BM == 64 && BN == 64), "the second group's sums fit its buffers");
  __shared__ __align__(1024) unsigned char lds[2 * KG * STAGE];
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
  int tm, tn;
  gemm::tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;

  OpA oa;
  OpB ob;
  oa.init(a.A, a.lda, m0, a.M, wave, lane);
  ob.init(a.B, a.ldb, n0, a.N, wave, lane);
  const int steps = (int)((a.K + SG_BK - 1) / SG_BK), turns = (steps + KG - 1) / KG;
  auto buffer = [&](int t) { return lds + (group * 2 + (t & 1)) * STAGE; };
  oa.load(buffer(0), group, a.K, wave);
  ob.load(buffer(0) + OpA::BYTES, group, a.K, wave);
  for (int t = 0; t < turns; ++t) {
    __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm(0));  // this wave's share of the step has landed
    __builtin_amdgcn_s_waitcnt(gemm::waitcnt_lgkm0());
    __builtin_amdgcn_s_barrier();                     // everyone's has, and everyone has read the other buffer
    __builtin_amdgcn_sched_barrier(0);
    if (t + 1 < turns) {
      oa.load(buffer(t + 1), (t + 1) * KG + group, a.K, wave);
      ob.load(buffer(t + 1) + OpA::BYTES, (t + 1) * KG + group, a.K, wave);
    }
    const unsigned char* la = buffer(t);
    const unsigned char* lb = la + OpA::BYTES;
#pragma unroll
    for (int kk = 0; kk < SG_BK / 8; ++kk) {
      f32x4_t fa[TM], fb[TN];
#pragma unroll
      for (int x = 0; x < TM; ++x) fa[x] = OpA::fragment(la, wm + x * 32 + l32, kk, half);
#pragma unroll
      for (int y = 0; y < TN; ++y) fb[y] = OpB::fragment(lb, wn + y * 32 + l32, kk, half);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
          for (int y = 0; y < TN; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[x][j], fb[y][j], acc[x][y], 0, 0, 0);
    }
  }
  store_tile<TM, TN, KG>(a, acc, reinterpret_cast<float*>(lds), m0 + wm, n0 + wn, group, tid, l32, half);
#endif
}

// ------------------------------------------------------------------ sliced form
// Few output tiles: a workgroup of NWV waves owns 32 x 32 outputs, each wave takes every NWV-th run of 8 k-values
// straight from memory into registers, and the waves' sums meet in LDS, added in wave order.
template <bool KMAJOR>
__device__ __forceinline__ void sliced_fragment(const float* __restrict__ P, int64_t ld, int64_t row, bool row_ok, int64_t k,
                                                int64_t K, float (&f)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) f[j] = 0.f;
  if (!row_ok) return;
  if constexpr (KMAJOR) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (k + j < K) f[j] = P[(k + j) * ld + row];
  } else {
    const float* p = P + row * ld + k;
    if (k + 3 < K) {
      const f32x4u_t t = *reinterpret_cast<const f32x4u_t*>(p);
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = t[j];
    } else {
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (k + j < K) f[j] = p[j];
    }
  }
}

constexpr int SL_WAVES = 8;
constexpr int SL_UNROLL = 4;  // runs of 8 k-values in flight per wave

typedef float SlicedSums[SL_WAVES][32][33];

template <bool A_KM, bool B_KM>
__device__ __forceinline__ void sliced_tile(const SgemmArgs& a, int tile, SlicedSums& part) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int tiles_n = (int)((a.N + 31) / 32);
  const int64_t m0 = (int64_t)(tile / tiles_n) * 32, n0 = (int64_t)(tile % tiles_n) * 32;
  const bool m_ok = m0 + l32 < a.M, n_ok = n0 + l32 < a.N;
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  for (int64_t k0 = (int64_t)wave * 8; k0 < a.K; k0 += SL_WAVES * 8 * SL_UNROLL) {
    float fa[SL_UNROLL][4], fb[SL_UNROLL][4];
#pragma unroll
    for (int u = 0; u < SL_UNROLL; ++u) {
      const int64_t k = k0 + u * (SL_WAVES * 8) + half * 4;
      sliced_fragment<A_KM>(a.A, a.lda, m0 + l32, m_ok, k, a.K, fa[u]);
      sliced_fragment<B_KM>(a.B, a.ldb, n0 + l32, n_ok, k, a.K, fb[u]);
    }
#pragma unroll
    for (int u = 0; u < SL_UNROLL; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u][j], fb[u][j], acc, 0, 0, 0);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) part[wave][8 * (e / 4) + 4 * half + (e % 4)][l32] = acc[e];
  __syncthreads();
  for (int q = tid; q < 32 * 32; q += 64 * SL_WAVES) {
    const int r = q >> 5, c = q & 31;
    float v = part[0][r][c];
#pragma unroll
    for (int w = 1; w < SL_WAVES; ++w) v += part[w][r][c];
    if (m0 + r < a.M && n0 + c < a.N) store_out(a, m0 + r, n0 + c, v);
  }
#endif
}

template <bool A_KM, bool B_KM>
__global__ __launch_bounds__(64 * SL_WAVES) void sgemm_sliced_kernel(SgemmArgs a) {
  __shared__ SlicedSums part;
  sliced_tile<A_KM, B_KM>(a, (int)blockIdx.x, part);
}

// Two products that do not need each other in one launch (dX and dWq of a small layer): the first `tiles` workgroups take
// a, the others b.  Each is a single chain of loads, matrix ops and stores of about 5 us.
template <bool A1, bool B1, bool A2, bool B2>
__global__ __launch_bounds__(64 * SL_WAVES) void sgemm_sliced_pair_kernel(SgemmArgs a, SgemmArgs b, int tiles) {
  __shared__ SlicedSums part;
  if ((int)blockIdx.x < tiles) sliced_tile<A1, B1>(a, (int)blockIdx.x, part);
  else sliced_tile<A2, B2>(b, (int)blockIdx.x - tiles, part);
}

// operand of whole 16-byte pieces, every offset from a tile's first row within 31 bits
template <bool KMAJOR>
bool whole_pieces(const float* P, int64_t ld, int64_t extent, int64_t K) {
  if ((reinterpret_cast<uintptr_t>(P) & 15) != 0 || ld % 4 != 0) return false;
  if (KMAJOR) return extent % 4 == 0 && (K + SG_BK) * ld < (1ll << 29);
  return K % 4 == 0 && 128 * ld + K + SG_BK < (1ll << 29);
}

// Which form, in us (K-contiguous operands; sliced / 64 x 64 tiles by one, by two groups of waves / 128 x 128 tiles):
//   64-wide tiles   16 (100 x 512 x 1024)   11 / 30 / 25 / 82     the vector kernel took 36 .. 44 us on a 4-tile product
//                   80 (300 x 1024 x 1024)  21 / 31 / 26 / 83     of K = 256 (sliced form: 4.8) and 318 .. 363 us on
//                  128 (512 x 1024 x 2048)  41 / 59 / 49 / 161    1000 x 2048 x 2048
//                  160 (1000 x 600 x 2048)  63 / 60 / 49 / 161
//                  256 (1000 x 1024 x 1024) 42 / 32 / 28 / 84
//                  512 (1000 x 2048 x 2048) 155 / 96 / 91 / 160   (93 TFLOP/s; matrix peak 157)
//                  512 (1000 x 2048 x 16)   11 / 6.3 / 8.2 / 11
//                 1024 (2048 x 2048 x 1000) 147 / 96 / 92 / 87
//                 2048 (2048 x 4096 x 2048) 606 / 342 / 330 / 290 (118 TFLOP/s)
// A 64-wide tile of one group occupies a compute unit for its whole k range with one wave per SIMD; a second group on the
// other k-steps halves the steps a wave waits through.  Below 5/8 of the units' number the sliced form, eight times as many
// waves on a quarter of the tile, is ahead.  128-wide tiles halve the operand traffic; the line at two of them per compute
// unit leaves them out at one per unit, where they are 5 % ahead at K = 1000 (92 / 87) but add up k in one chain instead of
// two of half the length (a layer of 1000 x 2048 x 2048 is 5.8e-7 off its value in 64 bits with two groups, 8.1e-7 with one).
template <bool A_KM, bool B_KM>
void launch_sgemm_form(const SgemmArgs& a, hipStream_t stream) {
  auto tiles = [&](int64_t bm, int64_t bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
  const int64_t cus = device_compute_units();
  const bool whole = whole_pieces<A_KM>(a.A, a.lda, a.M, a.K) && whole_pieces<B_KM>(a.B, a.ldb, a.N, a.K);
  if (tiles(64, 64) * 8 < cus * 5)
    hipLaunchKernelGGL((sgemm_sliced_kernel<A_KM, B_KM>), dim3((unsigned)tiles(32, 32)), dim3(64 * SL_WAVES), 0, stream, a);
  else if (tiles(128, 128) < 2 * cus && a.K <= 4 * SG_BK)  // (fewer than two steps for each group)
    hipLaunchKernelGGL((sgemm_tile_kernel<64, 64, 1, A_KM, B_KM>), dim3((unsigned)tiles(64, 64)), dim3(256), 0, stream, a);
  else if (tiles(128, 128) < 2 * cus && whole)
    hipLaunchKernelGGL((sgemm_dma_kernel<64, 64, 2, A_KM, B_KM>), dim3((unsigned)tiles(64, 64)), dim3(512), 0, stream, a);
  else if (tiles(128, 128) < 2 * cus)
    hipLaunchKernelGGL((sgemm_tile_kernel<64, 64, 2, A_KM, B_KM>), dim3((unsigned)tiles(64, 64)), dim3(512), 0, stream, a);
  else if (whole)
    hipLaunchKernelGGL((sgemm_dma_kernel<128, 128, 1, A_KM, B_KM>), dim3((unsigned)tiles(128, 128)), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((sgemm_tile_kernel<128, 128, 1, A_KM, B_KM>), dim3((unsigned)tiles(128, 128)), dim3(256), 0, stream, a);
}

}  // namespace

namespace {
SgemmArgs sgemm_args(const float* A, int64_t a_rs, int64_t a_cs, const float* B, int64_t b_rs, int64_t b_cs, float* C,
                     int64_t ldc, int64_t M, int64_t N, int64_t K, float scale, bool accumulate) {
  SgemmArgs a;
  a.A = A; a.B = B; a.C = C;
  a.M = M; a.N = N; a.K = K;
  a.ldc = ldc;
  a.scale = scale;
  a.accumulate = accumulate;
  a.lda = a_cs != 1 ? a_cs : a_rs;  // (one of an operand's strides is 1)
  a.ldb = b_rs != 1 ? b_rs : b_cs;
  return a;
}
}  // namespace

void launch_sgemm(const float* A, int64_t a_rs, int64_t a_cs, const float* B, int64_t b_rs, int64_t b_cs, float* C,
                  int64_t ldc, int64_t M, int64_t N, int64_t K, float scale, hipStream_t stream, bool accumulate) {
  const SgemmArgs a = sgemm_args(A, a_rs, a_cs, B, b_rs, b_cs, C, ldc, M, N, K, scale, accumulate);
  const bool a_km = a_cs != 1, b_km = b_rs != 1;
  if (a_km && b_km) launch_sgemm_form<true, true>(a, stream);
  else if (a_km) launch_sgemm_form<true, false>(a, stream);
  else if (b_km) launch_sgemm_form<false, true>(a, stream);
  else launch_sgemm_form<false, false>(a, stream);
}

void launch_sgemm_dx_dw(const float* dY, const float* X, const float* Wq, int64_t T, int64_t i, int64_t o, float* dX, float* dWq,
                        hipStream_t stream) {
  // dX[t,j] = sum_p dY[t,p] Wq[p,j];  dWq[p,j] = sum_t dY[t,p] X[t,j]
  auto tiles = [](int64_t m, int64_t n, int64_t b) { return ((m + b - 1) / b) * ((n + b - 1) / b); };
  const int64_t few = device_compute_units() * 5;
  // both of few tiles (the line of launch_sgemm_form), and in forms whose operands' unit strides are where they are expected
  if (tiles(T, i, 64) * 8 < few && tiles(o, i, 64) * 8 < few && i != 1 && o != 1) {
    const SgemmArgs a = sgemm_args(dY, o, 1, Wq, i, 1, dX, i, T, i, o, 1.f, false);
    const SgemmArgs b = sgemm_args(dY, 1, o, X, i, 1, dWq, i, o, i, T, 1.f, false);
    const int first = (int)tiles(T, i, 32);
    hipLaunchKernelGGL((sgemm_sliced_pair_kernel<false, true, true, true>), dim3((unsigned)(first + tiles(o, i, 32))),
                       dim3(64 * SL_WAVES), 0, stream, a, b, first);
    return;
  }
  launch_sgemm(dY, o, 1, Wq, i, 1, dX, i, T, i, o, 1.f, stream);
  launch_sgemm(dY, 1, o, X, i, 1, dWq, i, o, i, T, 1.f, stream);
}

}  // namespace l4q

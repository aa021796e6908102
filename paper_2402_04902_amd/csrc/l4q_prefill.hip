// Fully quantized layer at prompt sizes: Y[T,o] = X[T,i] . (w~ scale + zero)^T from the packed codes, more than 64 tokens.
//
// Bound: the matrix cores, with the vector unit close behind (the codes are turned into operands where they are used, and
// the affine part of every section of k is applied to its sums): per section of a 128 x 256 tile a wave has 1152 cycles of
// matrix ops and 950 of vector ops.  The decode kernels read and convert the whole weight once per 64 tokens: 8 passes of
// 27 us at 512 tokens on [11008 x 4096]; this kernel takes 58 us (calls one after the other; 64 under a kernel trace).  A workgroup of 8 waves (2 x 4, two per SIMD; for 192 rows
// 2 x 6, three) owns a tile of 64 TM tokens x 32 WN TN weight rows, so a converted code is used for 32 TM tokens of a wave and the weight is read once per
// tile row.  Arithmetic as in the decode kernels: the matrix cores multiply X with the exact integers w~ + K0, and
//   sum_k X (w~ s + b) = s sum_k X (w~ + K0) + (b - K0 s) sum_k X   per section of SEC k-values (128, or groups of 64),
// in binary32.
//  * X and the packed codes of a section travel memory -> LDS (buffer_load ... lds) into a ring of three sections, two
//    ahead; 16-byte pieces are swizzled so that fragment reads (lane = row) meet all banks.  The half-waves take 32
//    consecutive codes each: section sub-stage jj, matrix op d contracts k = 64 jj + 32 half + 8 d + 0 .. 7.
//  * scale and zero: every lane loads its own rows' values for four sections at a time into registers.
//  * within a section everything is one matrix-op step ahead: reads, conversions, sums of X and the next loads are dealt
//    out between the matrix ops (ahead of them in a lump they cost a third more, 93 us against 69 before the codes were taken in
//    X's order: both waves of a SIMD come out of the barrier together and do the same thing at the same time).
//  * sums of X per (token, section): dot products with ones by the four waves that hold the token, a quarter of the
//    section each; the partial sums meet in LDS, and the zero term of two sections is one K = 2 binary32 matrix op.
//  * 4 bits: a byte's two codes by one multiplication with the byte picked by the op, one mask-or per pair, in the order in
//    which X lies.  (Pairs (j, j + 4) take a shift less but X fragments permuted to match, by each of the four waves that
//    hold the tokens: 7 % more time in 128 x 256 tiles, 14 % in 128 x 128.)
#include <type_traits>
#include <utility>

#include "l4q_codes.h"
#include "l4q_device.h"
#include "l4q_gemm_core.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

typedef gemm::f32x16_t f32x16_t;
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int N, class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl<N>(static_cast<F&&>(f), std::make_integer_sequence<int, N>());
}

template <int BITS, int TM_, int TN_, int SEC_, bool WIDE_ = false, int WN_ = 4>
struct Prefill {
  static constexpr int TM = TM_, TN = TN_, SEC = SEC_;
  static constexpr bool WIDE = WIDE_;                  // groups of more than a section
  static constexpr int WN = WN_, NT = 128 * WN;        // 2 x 4 waves, two per SIMD; or 2 x 6, three
  static constexpr int BM = 64 * TM, BN = 32 * WN * TN;
  static constexpr int NJ = SEC / 64;                  // 64-k sub-stages: 128-byte rows of X
  static constexpr int PPR = SEC * BITS / 128;         // 16-byte pieces of a weight row's section
  static constexpr int X_TOTAL = BM * SEC * 2 / 1024;  // loads of X per section, and per wave (the last ones of nothing)
  static constexpr int X_INSTR = (X_TOTAL + 2 * WN - 1) / (2 * WN);
  static constexpr bool X_EVEN = X_INSTR * 2 * WN == X_TOTAL;
  static constexpr int W_INSTR = (BN * PPR + NT - 1) / NT;
  static constexpr int LOADS = X_INSTR + W_INSTR;
  static constexpr int X_BYTES = BM * SEC * 2;
  static constexpr int SLOT = X_BYTES + W_INSTR * 16 * NT;
  static constexpr int RING = 3;
  static constexpr int SX = RING * SLOT;               // [4 sections][BM tokens][8 partial sums]
  static constexpr int EP_ROW = 32 * TN * 2 + 16;      // bytes of a token's row in a wave's output block
  static constexpr int IDLE = SX + 4 * BM * 32;        // where loads of nothing go
  static constexpr int LDS = IDLE + (X_EVEN ? 0 : 1024);
  static_assert(SEC * BITS % 128 == 0, "a row's section is whole 16-byte pieces");
  static_assert(2 * WN * 32 * TM * EP_ROW <= SX, "the output blocks take the ring's place");
  static_assert(LDS <= 160 * 1024, "LDS");
  // piece `pos` of row `row` lies at position pos ^ swz(row)
  static __device__ __forceinline__ int swz(int row) {
    return PPR == 8 ? (row >> 1) & 7 : PPR == 4 ? (row >> 2) & 3 : PPR == 2 ? (row >> 3) & 1 : 0;
  }
};

template <int BITS, class P>
__global__ __launch_bounds__(P::NT) void qgemm_prefill_kernel(const bf16_t* __restrict__ X,
                                                            const uint32_t* __restrict__ packed,
                                                            const float* __restrict__ scale,
                                                            const float* __restrict__ zero, bf16_t* __restrict__ Y,
                                                            int T, int o, int i, int g, int tiles_m, int tiles_n) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char plds[];
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int TM = P::TM, TN = P::TN, SEC = P::SEC, NJ = P::NJ;
  constexpr float K0 = BITS == 8 ? 0.f : 128.f + (float)(1 << (BITS - 1));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / P::WN, wn = wave % P::WN;
  int tile_m, tile_n;
  gemm::tile_of_block(blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
  const int t0 = tile_m * P::BM, p0 = tile_n * P::BN;
  const int rb = i / 8 * BITS, G = i / g, nsec = i / SEC;
  const int gsh = P::WIDE ? 31 - __builtin_clz((unsigned)(g / SEC)) : 0;  // group of section q: q >> gsh

  const __amdgpu_buffer_rsrc_t rsX = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(X), 0, T * i * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsW =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(packed), 0, o * rb, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(scale), 0, o * G * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsZ = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(zero), 0, o * G * 4, 0x00020000);

  // source offsets of the ring's loads
  unsigned voffX[P::X_INSTR], voffW[P::W_INSTR];
#pragma unroll
  for (int c = 0; c < P::X_INSTR; ++c) {  // instruction q of the slot: 8 token rows of sub-stage q / (BM / 8)
    const int q = wave * P::X_INSTR + c, jj = q / (P::BM / 8), row = (q % (P::BM / 8)) * 8 + (lane >> 3);
    const int ch = (lane & 7) ^ ((row >> 1) & 7);
    voffX[c] = t0 + row < T && (P::X_EVEN || q < P::X_TOTAL) ? (unsigned)(((t0 + row) * i + jj * 64 + ch * 8) * 2) : gemm::OOB_OFFSET;
  }
#pragma unroll
  for (int c = 0; c < P::W_INSTR; ++c) {
    const int idx = (wave * P::W_INSTR + c) * 64 + lane, row = idx / P::PPR, pos = idx % P::PPR;
    voffW[c] = row < P::BN && p0 + row < o ? (unsigned)((p0 + row) * rb + (pos ^ P::swz(row)) * 16) : gemm::OOB_OFFSET;
  }
  // load c of section sec (X first, then the codes); past the last section: the same number of loads, of nothing
  auto issue_one = [&](int sec, int slot, auto ctag) {
    constexpr int c = decltype(ctag)::value;
    unsigned char* base = plds + slot * P::SLOT;
    if constexpr (c < P::X_INSTR) {
      const unsigned kx = sec < nsec ? (unsigned)sec * (SEC * 2) : gemm::PAST_END_OFFSET;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsX, (gemm::lds_ptr_t)(P::X_EVEN || wave * P::X_INSTR + c < P::X_TOTAL ? base + (wave * P::X_INSTR + c) * 1024
                                                                                              : plds + P::IDLE), 16,
                                               voffX[c] + kx, 0, 0, 0);
    } else {
      constexpr int cw = c - P::X_INSTR;
      const unsigned kw = sec < nsec ? (unsigned)sec * (SEC * BITS / 8) : gemm::PAST_END_OFFSET;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (gemm::lds_ptr_t)(base + P::X_BYTES + (wave * P::W_INSTR + cw) * 1024), 16,
                                               voffW[cw] + kw, 0, 0, 0);
    }
  };
  // scale and zero of this lane's rows, sections quad .. quad + 3
  u32x4_t ts[TN], tz[TN];
  auto request_table = [&](int quad) {
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int row = p0 + (wn * TN + b) * 32 + l32;
      const unsigned off = row < o && quad < nsec ? (unsigned)((row * G + (quad >> gsh)) * 4) : gemm::OOB_OFFSET;
      ts[b] = __builtin_amdgcn_raw_buffer_load_b128(rsS, off, 0, 0);
      tz[b] = __builtin_amdgcn_raw_buffer_load_b128(rsZ, off, 0, 0);
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
  float* sx = reinterpret_cast<float*>(plds + P::SX);
  for (int q = threadIdx.x; q < 4 * P::BM * 8; q += P::NT) sx[q] = 0.f;

  uint32_t pair_mask = 0x000F000Fu, pair_bias = 0x43004300u;  // (opaque: one v_and_or_b32 needs them in registers)
  asm volatile("" : "+s"(pair_mask));
  asm volatile("" : "+v"(pair_bias));

  float zpair[TN] = {};  // zero - K0 scale of section 2 m + half, for the pair whose zero term is due
  request_table(0);
  static_for<P::LOADS>([&](auto c) { issue_one(0, 0, c); });
  static_for<P::LOADS>([&](auto c) { issue_one(1, 1, c); });

  // zero term of the two sections whose sums of X lie in slots slot0, slot0 + 1
  auto zero_term = [&](int slot0, const float (&z)[TN]) {
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const unsigned char* q = plds + P::SX + ((slot0 + h) * P::BM + (wm * TM + a) * 32 + l32) * 32;
      const f32x4_t u = *reinterpret_cast<const f32x4_t*>(q), v = *reinterpret_cast<const f32x4_t*>(q + 16);
      const float sum = ((u[0] + u[1]) + (u[2] + u[3])) + ((v[0] + v[1]) + (v[2] + v[3]));
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(sum, z[b], acc[a][b], 0, 0, 0);
    }
  };

  // One section: K matrix-op steps of 16 k-values.  While step ks multiplies, step ks + 1 is converted and the X fragments of
  // step ks + 2 are read; the loads of section sec + 2 go out one per step, so that neither bunches up in front of the
  // matrix ops.
  auto section = [&](int sec, int j, int slot, int slot_fill, const float (&s)[TN]) {
    constexpr int K = NJ * 4;
    const unsigned char* base = plds + slot * P::SLOT;
    const unsigned char* xrow[TM];
    int xsw[TM];
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const int row = (wm * TM + a) * 32 + l32;
      xrow[a] = base + row * 128;
      xsw[a] = (row >> 1) & 7;
    }
    auto read_x = [&](int a, int ks) {
      return *reinterpret_cast<const bf16x8_t*>(xrow[a] + (ks >> 2) * (P::BM * 128) + (((4 * h + (ks & 3)) ^ xsw[a]) << 4));
    };
    code_chunk_t w[TN][NJ][BITS == 8 ? 2 : 1];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int row = (wn * TN + b) * 32 + l32;
      const unsigned char* wrow = base + P::X_BYTES + row * (P::PPR * 16);
      const int sw = P::swz(row);
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) {
        if constexpr (BITS == 4) {
          w[b][jj][0] = *reinterpret_cast<const code_chunk_t*>(wrow + (((2 * jj + h) ^ sw) << 4));
        } else if constexpr (BITS == 8) {
          w[b][jj][0] = *reinterpret_cast<const code_chunk_t*>(wrow + (((4 * jj + 2 * h) ^ sw) << 4));
          w[b][jj][1] = *reinterpret_cast<const code_chunk_t*>(wrow + (((4 * jj + 2 * h + 1) ^ sw) << 4));
        } else if constexpr (BITS == 2) {
          const uint2 v = *reinterpret_cast<const uint2*>(wrow + ((jj ^ sw) << 4) + 8 * h);
          w[b][jj][0] = code_chunk_t{v.x, v.y, 0u, 0u};
        } else {
          const uint32_t* v = reinterpret_cast<const uint32_t*>(wrow) + 6 * jj + 3 * h;
          w[b][jj][0] = code_chunk_t{v[0], v[1], v[2], 0u};
        }
      }
    }
    auto convert = [&](int b, int ks) {
      const int jj = ks >> 2, d = ks & 3;
      if constexpr (BITS == 4) {
        u32x4_t f;  // (a byte's two codes by one multiplication, see code_fragment; the byte is picked by the op itself)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = ((((w[b][jj][0][d] >> (8 * e)) & 0xFFu) * 0x1001u) & pair_mask) | pair_bias;
        return __builtin_bit_cast(bf16x8_t, f);
      } else if constexpr (BITS == 8) {
        return code_fragment<8>(w[b][jj][d >> 1], d & 1);
      } else {
        return code_fragment<BITS>(w[b][jj][0], d);
      }
    };
    const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3F803F80u);
    // vector ops dealt to a matrix op: 4 bits 8 TN conversions a step and sums of X (128 x 256 tiles 6: 70 us, 4: 73); the other
    // widths convert in 12 to 16
    constexpr int VALU_PER = BITS == 4 ? (TN == 1 ? 8 / TM : 6) : P::WN == 6 ? 4 : (TM * 4 + TN * 8 + TM * TN - 1) / (TM * TN);
    bf16x8_t xr[3][TM], wf[2][TN], xq[TM];
    float part[TM];
    f32x16_t tw[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      part[a] = 0.f;
      xr[0][a] = read_x(a, 0);
      xr[1][a] = read_x(a, 1);
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) tw[a][b][e] = 0.f;
    }
#pragma unroll
    for (int b = 0; b < TN; ++b) wf[0][b] = convert(b, 0);
    static_for<K>([&](auto kt) {
      constexpr int ks = decltype(kt)::value;
      if constexpr (ks + 2 < K) {
#pragma unroll
        for (int a = 0; a < TM; ++a) xr[(ks + 2) % 3][a] = read_x(a, ks + 2);
      }
      // the loads of this step (LOADS over K steps, the first steps first)
      constexpr int PER = (P::LOADS + K - 1) / K;
      static_for<PER>([&](auto q) {
        constexpr int c = ks * PER + decltype(q)::value;
        if constexpr (c < P::LOADS) issue_one(sec + 2, slot_fill, std::integral_constant<int, c>());
      });
      if constexpr (ks + 1 < K) {
#pragma unroll
        for (int b = 0; b < TN; ++b) wf[(ks + 1) & 1][b] = convert(b, ks + 1);
      }
      // sums of X: the steps of this wave's quarter, read a step ahead
      if constexpr (ks > 0 && ks <= NJ) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          const u32x4_t x = __builtin_bit_cast(u32x4_t, xq[a]);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const uint32_t pair = x[c];  // (a copy: the bit cast of a vector's element itself takes element 0)
            part[a] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair), ones, part[a], false);
          }
        }
      }
      if constexpr (ks < NJ) {
        const int kq = (P::WN == 4 ? wn : wn & 3) * NJ + ks;  // (waves past the fourth: as the first ones, and not stored)
#pragma unroll
        for (int a = 0; a < TM; ++a)
          xq[a] = *reinterpret_cast<const bf16x8_t*>(xrow[a] + (kq >> 2) * (P::BM * 128) + (((4 * h + (kq & 3)) ^ xsw[a]) << 4));
      }
#pragma unroll
      for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
          tw[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xr[ks % 3][a], wf[ks & 1][b], tw[a][b], 0, 0, 0);
      // matrix ops one by one, the vector ops, reads and loads of the step between them: issued back to back they would
      // hold up the wave's vector ops until the last has started
#pragma unroll
      for (int q = 0; q < TM * TN; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (q == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    });
    if (P::WN == 4 || wn < 4) {
#pragma unroll
      for (int a = 0; a < TM; ++a) sx[(j * P::BM + (wm * TM + a) * 32 + l32) * 8 + 2 * wn + h] = part[a];
    }
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[a][b][e] = fmaf(s[b], tw[a][b][e], acc[a][b][e]);
  };

  int slot = 0;
  for (int quad = 0; quad < nsec; quad += 4) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int sec = quad + j;
      if (sec >= nsec) break;  // (uniform)
      // this section's loads have landed; the LOADS issued last, the next section's, may not have (the table's pieces, asked
      // for ahead of them, count among the older ones: they are needed here)
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm(P::LOADS));
      __builtin_amdgcn_s_waitcnt(gemm::waitcnt_lgkm0());  // (this wave's sums of X are in LDS, its reads of the slot refilled below done)
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      float s[TN], zdue[TN];
#pragma unroll
      for (int b = 0; b < TN; ++b) zdue[b] = zpair[b];
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        auto pick = [&](const u32x4_t& t, int q) {  // section quad + q of the four
          const uint32_t v = !P::WIDE ? t[q] : gsh == 1 ? t[q >> 1] : t[0];
          return __uint_as_float(v);
        };
        s[b] = pick(ts[b], j);
        if (j == 0 || j == 2) {  // the pair that starts here is due at the next pair's start
          const float z0 = pick(tz[b], j) - K0 * pick(ts[b], j);
          const float z1 = pick(tz[b], j + 1) - K0 * pick(ts[b], j + 1);
          zpair[b] = h == 0 ? z0 : sec + 1 < nsec ? z1 : 0.f;
        }
      }
      if (j == 3) request_table(quad + 4);  // this quad's values have all been picked
      const int fill = slot == 0 ? P::RING - 1 : slot - 1;  // (sec + 2) % RING: section sec - 1's, free now
      section(sec, j, slot, fill, s);
      slot = slot + 1 == P::RING ? 0 : slot + 1;
      if (j == 0 && quad > 0) zero_term(2, zdue);
      if (j == 2) zero_term(0, zdue);
    }
  }
  __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm(0));
  // the last section of an odd count has no partner: the sums an earlier section has left in the partner's place are taken
  // out (its zero factor would make NaN of an infinite one).  No wave is behind the last barrier's section, and that reads
  // the other two places.  (Sections of 64, and of 128 with several to a group, come in even numbers.)
  if constexpr (SEC == 128 && !P::WIDE) if (nsec & 1)
    for (int q = threadIdx.x; q < P::BM * 8; q += P::NT) sx[(nsec & 3) * P::BM * 8 + q] = 0.f;
  __syncthreads();  // the last pair's sums of X; every wave is done with the ring
  zero_term((nsec - 1) & 2, zpair);

  // accumulator: lane = weight row, register e = token 8 (e / 4) + 4 h + e % 4.  Through LDS (each wave its own block of the
  // ring) to 16 bytes per lane along a token's outputs.
  unsigned char* region = plds + wave * (32 * TM * P::EP_ROW);
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int t = a * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
        *reinterpret_cast<bf16_t*>(region + t * P::EP_ROW + (b * 32 + l32) * 2) = f32_to_bf16(acc[a][b][e]);
      }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int PIECES = 4 * TN;  // 16-byte pieces of a token's row
#pragma unroll
  for (int it = 0; it < 32 * TM * PIECES / 64; ++it) {
    const int q = it * 64 + lane, t = q / PIECES, c = q % PIECES;
    const int tok = t0 + wm * 32 * TM + t, p = p0 + wn * 32 * TN + c * 8;
    const uint4 v = *reinterpret_cast<const uint4*>(region + t * P::EP_ROW + c * 16);
    if (tok < T && p < o) *reinterpret_cast<uint4*>(Y + (int64_t)tok * o + p) = v;  // (o % 8 == 0)
  }
#endif
}

template <int BITS, class P>
void launch_form(const LayerDims& d, const bf16_t* X, const uint32_t* packed, const float* scale, const float* zero,
                 bf16_t* Y, hipStream_t stream) {
  const int tiles_m = (int)((d.T + P::BM - 1) / P::BM), tiles_n = (int)((d.o + P::BN - 1) / P::BN);
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&qgemm_prefill_kernel<BITS, P>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, P::LDS);  // (above 64 KiB: per function and device)
  hipLaunchKernelGGL((qgemm_prefill_kernel<BITS, P>), dim3((unsigned)(tiles_m * tiles_n)), dim3(P::NT), P::LDS, stream, X,
                     packed, scale, zero, Y, (int)d.T, (int)d.o, (int)d.i, d.g, tiles_m, tiles_n);
}

// 128-token tiles of 256 weight rows (8 waves of 64 x 64) or of 192 (12 waves of 64 x 32): a section of a round is put at 1.95 and
// 1.72 us, and the smaller sum of rounds is taken, so 192 wherever it needs no more rounds (it leaves fewer units idle in the
// last one), or 9 for 8.  us at 4, 3, 2 bits, 256 / 192: 512, 11008 x 4096 62 / 59, 77 / 63, 73 / 62;  1000, 11008 x 4096 126 / 114,
// 154 / 127, 147 / 122;  700, 6144 x 5120 73 / 65, 92 / 74, 88 / 71;  512, 4096 x 4096 59 / 52, 74 / 59, 71 / 57.
struct WideTiles {
  int rows;
  double section_us;  // of all rounds
};
WideTiles wide_tiles(const LayerDims& d) {
  const int64_t cus = device_compute_units(), tiles_m = (d.T + 127) / 128;
  const double r256 = (double)((tiles_m * ((d.o + 255) / 256) + cus - 1) / cus) * 1.95;
  const double r192 = (double)((tiles_m * ((d.o + 191) / 192) + cus - 1) / cus) * 1.72;
  return r192 < r256 ? WideTiles{192, r192} : WideTiles{256, r256};
}

// Forms: 0 = 64 x 128 tiles (two workgroups per compute unit), 1 = 128 x 128, 2 = wide tiles (groups of 128, not 8 bits).
template <int BITS, int SEC, bool WIDE>
void launch_bits(int form, const LayerDims& d, const bf16_t* X, const uint32_t* packed, const float* scale,
                 const float* zero, bf16_t* Y, hipStream_t stream) {
  if (form == 0) launch_form<BITS, Prefill<BITS, 1, 1, SEC, WIDE>>(d, X, packed, scale, zero, Y, stream);
  else if (form == 1) launch_form<BITS, Prefill<BITS, 2, 1, SEC, WIDE>>(d, X, packed, scale, zero, Y, stream);
  else if constexpr (BITS != 8 && SEC == 128 && !WIDE) {
    if (wide_tiles(d).rows == 256) launch_form<BITS, Prefill<BITS, 2, 2, SEC, WIDE>>(d, X, packed, scale, zero, Y, stream);
    else launch_form<BITS, Prefill<BITS, 2, 1, SEC, WIDE, 6>>(d, X, packed, scale, zero, Y, stream);
  }
}

}  // namespace

int qgemm_prompt_wide_rows(const LayerDims& d) { return wide_tiles(d).rows; }

// Time of the three forms in us: rounds of tiles over the compute units, times sections of 128 k-values, times what a section
// of a round takes, plus 5 for the launch, the first loads and the store.  Measured at 4 bits (64 x 128 / 128 x 128 / wide
// tiles, here all of 192 rows; T, o x i): 200, 4096 x 4096 29 / 38 / 50;  512, 4096 x 4096 31 / 41 / 52;  1024, 4096 x 4096
// 51 / 47 / 56;  256, 11008 x 4096 46 / 41 / 52;  512, 11008 x 4096 75 / 84 / 58;  1000, 11008 x 4096 143 / 132 / 115;
// 200, 4096 x 11008 75 / 102 / 134.  2 and 3 bits take 2 .. 20 % more, 8 bits 10 .. 40 %, groups of
// 64 20 .. 35 % (twice the barriers and scalings).
// (One pass of the decode kernels per 64 tokens: 512 tokens on 11008 x 4096 214, 256 on 4096 x 11008 103.)
// The choice against those passes falls where 64 x 128 tiles are the best form, and needs their time closer than that: one
// workgroup on a unit is put at 0.885 us per section at 4 bits, two together at 1.46 (2, 3, 8 bits: 0.97 and 1.6, 1.02 and 1.65,
// 1.13 and 2.37; groups of 64 28 % more, 23 % at 8 bits).  On 470 drawn calls of 65 to 1024 tokens that is 2 to 3 % off on
// average, but 10 % above the time at 4 bits in groups of 128, whose conversion has become faster since: of 260 such calls
// 8, of 84 to 290 tokens, go through the passes and would be 5 to 19 % faster here; the mean loss of all is 0.4 %.
PrefillPlan qgemm_prefill_plan(const LayerDims& d) {
  PrefillPlan plan = {-1, 0.0};
  const bool g_ok = d.g >= 128 || (d.g == 64 && d.bits != 3);
  if (!g_ok || d.i % 128 != 0 || d.o % 8 != 0 || d.o * (d.i / 8 * d.bits) >= (1ll << 30) || d.T * d.i >= (1ll << 29) ||
      d.o * (d.i / d.g) >= (1ll << 28))
    return plan;
  const int64_t cus = device_compute_units();
  const int64_t bm[2] = {64, 128}, bn[2] = {128, 128};
  const double per_section[2] = {0.8, 1.35};
  const double bits_factor = (d.bits == 4 ? 1.0 : d.bits == 8 ? 1.25 : 1.12) * (d.g == 64 ? 1.25 : 1.0);
  for (int f = 0; f < (d.g == 128 && d.bits != 8 ? 3 : 2); ++f) {
    double section_us;  // of all rounds
    if (f == 2) section_us = wide_tiles(d).section_us;
    else {
      const int64_t tiles = ((d.T + bm[f] - 1) / bm[f]) * ((d.o + bn[f] - 1) / bn[f]);
      double rounds = (double)((tiles + cus - 1) / cus);
      if (f == 0 && rounds < 1.1) rounds = 1.1;  // (two workgroups share a unit: one alone is not twice as fast)
      section_us = rounds * per_section[f];
    }
    const double us = 5.0 + (double)d.i / 128.0 * section_us * bits_factor;
    if (plan.form < 0 || us < plan.us) {
      plan.form = f;
      plan.us = us;
    }
  }
  if (plan.form == 0) {
    const double one[4] = {0.97, 1.02, 0.885, 1.13}, two[4] = {1.6, 1.65, 1.46, 2.37};
    const int b = d.bits == 8 ? 3 : d.bits - 2;
    const int64_t tiles = ((d.T + 63) / 64) * ((d.o + 127) / 128), left = tiles % (2 * cus);
    const double rounds = (double)(tiles / (2 * cus)) * two[b] + (left > cus ? two[b] : left > 0 ? one[b] : 0.0);
    plan.us = 3.3 + (double)d.i / 128.0 * rounds * (d.g != 64 ? 1.0 : d.bits == 8 ? 1.23 : 1.28);
  }
  return plan;
}

void launch_qgemm_prefill(const PrefillPlan& plan, const LayerDims& d, const bf16_t* X, const uint32_t* packed,
                          const float* scale, const float* zero, bf16_t* Y, hipStream_t stream) {
#define L4Q_PF(B, S, W) launch_bits<B, S, W>(plan.form, d, X, packed, scale, zero, Y, stream)
#define L4Q_PF_BITS(S, W)                   \
  do {                                      \
    if (d.bits == 2) L4Q_PF(2, S, W);       \
    else if (d.bits == 4) L4Q_PF(4, S, W);  \
    else L4Q_PF(8, S, W);                   \
  } while (0)
  if (d.bits == 3 && d.g == 128) L4Q_PF(3, 128, false);
  else if (d.bits == 3) L4Q_PF(3, 128, true);
  else if (d.g == 64) L4Q_PF_BITS(64, false);
  else if (d.g == 128) L4Q_PF_BITS(128, false);
  else L4Q_PF_BITS(128, true);
#undef L4Q_PF_BITS
#undef L4Q_PF
}

}  // namespace l4q

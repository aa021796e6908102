// The fully quantized layer at one to four token blocks (up to 64 tokens; Sec. 3.2, Eq. l4q_forward on Eq. l4q_Wdequant):
// Y = X . dequant(codes)^T in one pass over the weights and one over the activations.
//
// A workgroup of 8 waves takes NT 16-row tiles and a k-slice (usually the whole of k); each wave takes a run of
// consecutive k of it and all TB token blocks, so that every byte of X and of the weights is loaded by exactly one
// wave of the workgroup and every code converted once.  Nothing is shared between the waves, and there is no barrier, until
// their partial sums meet in LDS at the end.
//
// What bounds it is the fetch of X: each compute unit reads the whole of it out of its L2 ([4096 x 4096], 64 tokens: 512 KB a
// unit, 10.5 of 20 us when the loads touch 64 bytes of a token at a time, as the matrix op's operands lie).  A load of 16 rows x
// 64 bytes takes the unit's cache three times as long as one of 8 rows x 128 bytes, whole lines (all units reading one 512 KB
// array: 15.4 against 5.8 us).  So X comes into LDS by loads of 8 tokens x 128 bytes (64 k), into a ring of the wave's own,
// and the codes come in loads of 8 rows x 128 bytes (4 and 8 bits) into registers, where halves of 16 lanes change places.
// [4096 x 4096], 4 bits, 43 tokens: 14.5 us with operand-shaped loads, 8.3 so (64-row tiles in k-slices: 13.5); 64 tokens:
// 19.7, 10.2 (13.8).  Requesting the second macro's codes with the first, ahead of the step that needs none of them: 0 - 10 % slower.
#include <type_traits>

#include "l4q_codes.h"
#include "l4q_device.h"
#include "l4q_gemm_core.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

constexpr int QB_WAVES = 8;
typedef float qb_acc_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The codes of 8 consecutive k-values: 8 BITS bits (8 bits: two dwords).
template <int BITS> struct CodeWindow { uint32_t v[BITS == 8 ? 2 : 1]; };

// A lane's load of a step is F consecutive windows of its row, lane group kq's at 8 F kq; the matrix ops want, as operand d,
// window kq of the d-th run of four (in some order).  Exchanged between the lane groups by swaps of half-waves (F = 4: also of
// rows of 16 lanes): register index and lane group change places.
template <int BITS, int F>
__device__ __forceinline__ void windows(const uint32_t (&w)[F * BITS / 4], CodeWindow<BITS> (&win)[F]) {
#pragma unroll
  for (int f = 0; f < F; ++f) {
    if constexpr (BITS == 8) { win[f].v[0] = w[2 * f]; win[f].v[1] = w[2 * f + 1]; }
    else if constexpr (BITS == 4) win[f].v[0] = w[f];
    else if constexpr (BITS == 2) win[f].v[0] = f % 2 ? w[f / 2] >> 16 : w[f / 2];
    else win[f].v[0] = f == 0 ? w[0] : f == 1 ? (w[0] >> 24) | (w[1] << 8) : f == 2 ? (w[1] >> 16) | (w[2] << 16) : w[2] >> 8;
  }
#pragma unroll
  for (int e = 0; e < (BITS == 8 ? 2 : 1); ++e) {
#pragma unroll
    for (int f = 0; f < F / 2; ++f) {
      const u32x2 s = __builtin_amdgcn_permlane32_swap(win[f].v[e], win[f + F / 2].v[e], false, false);
      win[f].v[e] = s[0];
      win[f + F / 2].v[e] = s[1];
    }
    if constexpr (F == 4) {
#pragma unroll
      for (int f = 0; f < F; f += 2) {
        const u32x2 s = __builtin_amdgcn_permlane16_swap(win[f].v[e], win[f + 1].v[e], false, false);
        win[f].v[e] = s[0];
        win[f + 1].v[e] = s[1];
      }
    }
  }
}

template <int BITS> __device__ __forceinline__ bf16x8_t codes_of_window(const CodeWindow<BITS>& win) {
  if constexpr (BITS == 8) return code_fragment<8>(code_chunk_t{win.v[0], win.v[1], 0u, 0u}, 0);
  else if constexpr (BITS == 3) return code_fragment<3>(code_chunk_t{win.v[0], 0u, 0u, 0u}, 0);
  else return code_fragment<BITS>(code_chunk_t{win.v[0], 0u, 0u, 0u}, 0);
}

struct QbArgs {
  const bf16_t* X;
  const uint32_t* packed;
  const float* scale;
  const float* zero;
  bf16_t* Y;
  float* part;       // null: one slice
  int T, o, i, gshift;
  int slice_macros;  // runs of 256 k-values of a slice
  int tab_groups;    // groups that a slice can meet
};

constexpr int qb_ring(int tb) { return tb <= 2 ? 4 : 2; }  // steps of 64 k-values of X per wave in LDS

template <int BITS, int KSTEP, int NT, int TB>
__global__ __launch_bounds__(QB_WAVES * 64) void qgemm_blocks_kernel(QbArgs p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char qb_lds[];
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int F = KSTEP / 32;              // matrix ops per code step, tile and token block
  constexpr int XS = KSTEP / 64;             // X steps (64 k) per code step
  constexpr int WD = KSTEP / 4 * BITS / 32;  // dwords of codes per lane and load
  constexpr int QW = 256 / (2 * KSTEP);      // loads per macro, tile and row half
  constexpr int R = qb_ring(TB);
  constexpr int XL = 2 * TB;                 // loads per X step
  constexpr int WL = NT * 2 * QW;            // loads of codes per macro
  constexpr float K0 = BITS == 8 ? 0.f : 128.f + (float)(1 << (BITS - 1));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 15, kq = lane >> 4;
  const int rb = p.i / 8 * BITS, G = p.i >> p.gshift;
  const u32x4 ones_bits = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
  const bf16x8_t ones = __builtin_bit_cast(bf16x8_t, ones_bits);

  // this wave's macros (256 k) of the slice
  const int total = (p.i + 255) / 256;
  const int sl0 = (int)blockIdx.y * p.slice_macros;
  const int sln = sl0 + p.slice_macros < total ? p.slice_macros : total - sl0;
  const int s0 = sl0 + sln * wave / QB_WAVES;
  const int nm = sl0 + sln * (wave + 1) / QB_WAVES - s0;
  const int k_first = s0 * 256;
  const int k_end = k_first + nm * 256 < p.i ? k_first + nm * 256 : p.i;

  const __amdgpu_buffer_rsrc_t rsrcW = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(p.packed), 0, (int)((int64_t)p.o * rb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcX = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.X), 0, (int)((int64_t)p.T * p.i * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcS = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.scale), 0, (int)((int64_t)p.o * G * 4), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcZ = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(p.zero), 0, (int)((int64_t)p.o * G * 4), 0x00020000);

  unsigned char* const ring = qb_lds + wave * (R * TB * 2048);
  const int pitch = ((p.tab_groups + 1) / 2) | 1;  // pairs of groups, 16 bytes each
  const int grp0 = (sl0 * 256) >> p.gshift;
  unsigned char* const tab = qb_lds + QB_WAVES * (R * TB * 2048);
  auto row_of = [&](int n) { return ((int)blockIdx.x * NT + n) * 16; };

  // X: load c of a step fetches 128 bytes of tokens 8 c .. 8 c + 7; chunk e of token row r at position e ^ (r / 2) % 8
  unsigned xoff[XL];
#pragma unroll
  for (int c = 0; c < XL; ++c) {
    const int row = 8 * c + (lane >> 3);
    xoff[c] = (unsigned)(row * p.i * 2 + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
  }
  auto load_x = [&](int slot, int x) {  // X step x of the wave
    const int k = k_first + x * 64;
    const bool live = k < k_end;
    const int so = live ? k * 2 : 0;
#pragma unroll
    for (int c = 0; c < XL; ++c)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcX, (gemm::lds_ptr_t)(ring + (slot * XL + c) * 1024), 16,
                                               (int)(live ? xoff[c] : gemm::OOB_OFFSET), so, 0, 0);
  };
  // codes: a load fetches 8 rows x two code steps; lane: row lane % 8 of the half, piece 4 (lane / 8 % 2) + kq
  const int wrow = lane & 7, whalf = (lane >> 3) & 1;
  unsigned woff[NT][2];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = row_of(n) + 8 * h + wrow;
      woff[n][h] = row < p.o ? (unsigned)(row * rb + (4 * whalf + kq) * (KSTEP / 32 * BITS)) : gemm::OOB_OFFSET;
    }
  uint32_t w[2][NT][QW][2][WD];
  auto load_w = [&](int buf, int m) {
#pragma unroll
    for (int q = 0; q < QW; ++q) {
      const int k = k_first + m * 256 + q * 2 * KSTEP;
      const int so = k < k_end ? k / 8 * BITS : 0;
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const unsigned v = k + whalf * KSTEP < k_end ? woff[n][h] : gemm::OOB_OFFSET;
          uint32_t* dst = w[buf][n][q][h];
          if constexpr (WD == 4) {
            const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(rsrcW, (int)v, so, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[e] = c[e];
          } else if constexpr (WD == 3) {
            const u32x3 c = __builtin_amdgcn_raw_buffer_load_b96(rsrcW, (int)v, so, 0);
#pragma unroll
            for (int e = 0; e < 3; ++e) dst[e] = c[e];
          } else if constexpr (WD == 2) {
            const u32x2 c = __builtin_amdgcn_raw_buffer_load_b64(rsrcW, (int)v, so, 0);
            dst[0] = c[0];
            dst[1] = c[1];
          } else {
            static_assert(WD == 1, "dwords per lane");
            dst[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrcW, (int)v, so, 0);
          }
        }
    }
  };

  // scale and zero - K0 scale of the workgroup's rows and the slice's groups, pairs of them, by way of LDS: a thread fetches
  // four groups of a row.  Requested first, so that nothing behind them is waited for.  (By each wave for itself, its own
  // groups of 16 rows a load, they took the unit's cache about 1 us.)
  {
    const int ppr = (p.tab_groups + 3) / 4, pieces = NT * 16 * ppr;
    float4 sv, zv;
    int row, c;
    auto fetch = [&](int piece) {
      row = piece / ppr;
      c = piece - row * ppr;
      const unsigned off = piece < pieces && row_of(0) + row < p.o ? (unsigned)(((row_of(0) + row) * G + grp0 + 4 * c) * 4) : gemm::OOB_OFFSET;
      sv = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrcS, (int)off, 0, 0));
      zv = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrcZ, (int)off, 0, 0));
    };
    auto put = [&](int piece) {
      if (piece < pieces) {
        unsigned char* dst = tab + (row * pitch + 2 * c) * 16;
        const float s4[4] = {sv.x, sv.y, sv.z, sv.w}, z4[4] = {zv.x, zv.y, zv.z, zv.w};
#pragma unroll
        for (int e = 0; e < 4; e += 2)
          if (2 * c + e / 2 < pitch)
            *reinterpret_cast<bf16x8_t*>(dst + 8 * e) = __builtin_bit_cast(
                bf16x8_t, make_float4(s4[e], z4[e] - K0 * s4[e], s4[e + 1], z4[e + 1] - K0 * s4[e + 1]));
      }
    };
#pragma unroll 1
    for (int piece = (int)threadIdx.x + QB_WAVES * 64; piece < pieces; piece += QB_WAVES * 64) {  // (small groups)
      fetch(piece);
      put(piece);
    }
    fetch((int)threadIdx.x);
    __builtin_amdgcn_sched_barrier(0);
    load_w(0, 0);
#pragma unroll
    for (int x = 0; x < R; ++x) load_x(x, x);
    __builtin_amdgcn_sched_barrier(0);
    put((int)threadIdx.x);
    __builtin_amdgcn_s_waitcnt(gemm::waitcnt_lgkm0());
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  const unsigned char* tab_row = tab + ln * pitch * 16;

  qb_acc_t acc[NT][TB], tw[NT][TB], xs[TB];
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[n][t][e] = 0.f;

  // operand chunk of matrix op d of a 64-k step, within the step's row of 8 chunks
  const int piece = KSTEP == 128 ? kq : ((kq & 1) << 1) | (kq >> 1);
  unsigned xfrag[2];
#pragma unroll
  for (int d = 0; d < 2; ++d) xfrag[d] = (unsigned)(ln * 128 + (((4 * d + piece) ^ ((ln >> 1) & 7)) << 4));

  auto macro = [&](auto bufc, int m) {
    constexpr int BUF = decltype(bufc)::value;
    CodeWindow<BITS> win[NT][F];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      // X step x has landed: the R - 1 steps after it may be in flight and, where they were requested since, the next codes
      __builtin_amdgcn_sched_barrier(0);
      if (x >= 1 && x <= R - 1) __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm((R - 1) * XL + WL));
      else __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm((R - 1) * XL));
      __builtin_amdgcn_sched_barrier(0);
      if (x == 0) {
        load_w(1 - BUF, m + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int cs = x / XS, xi = x % XS;  // code step of the macro, X step within it
      const int q = cs / 2, f = cs % 2;
      if (xi == 0) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          uint32_t c[WD];
#pragma unroll
          for (int e = 0; e < WD; ++e) {
            // rows of 16 lanes: half f of both loads, the other row half's from 8 lanes further on
            c[e] = f == 0 ? (uint32_t)__builtin_amdgcn_update_dpp((int)w[BUF][n][q][0][e], (int)w[BUF][n][q][1][e], 0x128, 0xF, 0xC, false)
                          : (uint32_t)__builtin_amdgcn_update_dpp((int)w[BUF][n][q][1][e], (int)w[BUF][n][q][0][e], 0x128, 0xF, 0x3, false);
          }
          windows<BITS, F>(c, win[n]);
        }
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            xs[t][e] = 0.f;
#pragma unroll
            for (int n = 0; n < NT; ++n) tw[n][t][e] = 0.f;
          }
      }
      bf16x8_t xf[TB][2];
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int d = 0; d < 2; ++d)
          xf[t][d] = *reinterpret_cast<const bf16x8_t*>(ring + (x % R) * (XL * 1024) + t * 2048 + xfrag[d]);
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int t = 0; t < TB; ++t) xs[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[t][d], ones, xs[t], 0, 0, 0);
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const bf16x8_t wf = codes_of_window<BITS>(win[n][xi * 2 + d]);
#pragma unroll
          for (int t = 0; t < TB; ++t) tw[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[t][d], wf, tw[n][t], 0, 0, 0);
        }
      if (xi == XS - 1 && k_first + m * 256 + cs * KSTEP < k_end) {
        const int gi = ((k_first + m * 256 + cs * KSTEP) >> p.gshift) - grp0;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          // (opaque, so that it stays one 16-byte read of the operands' type: before others the compiler would wait for every
          // load in flight into LDS)
          u32x4 v = __builtin_bit_cast(u32x4, *reinterpret_cast<const bf16x8_t*>(tab_row + (n * 16 * pitch + (gi >> 1)) * 16));
          asm volatile("" : "+v"(v));
          const float4 pair = __builtin_bit_cast(float4, v);
          const float2 sz = gi & 1 ? make_float2(pair.z, pair.w) : make_float2(pair.x, pair.y);
#pragma unroll
          for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[n][t][e] = fmaf(sz.x, tw[n][t][e], fmaf(sz.y, xs[t][e], acc[n][t][e]));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(gemm::waitcnt_lgkm0());  // the step's operands are in registers: its slot is free
      __builtin_amdgcn_sched_barrier(0);
      load_x(x % R, m * 4 + x + R);
    }
  };
  int m = 0;
  for (; m + 1 < nm; m += 2) {
    macro(std::integral_constant<int, 0>(), m);
    macro(std::integral_constant<int, 1>(), m + 1);
  }
  if (m < nm) macro(std::integral_constant<int, 0>(), m);
  // (the codes requested past the end are kept alive: the waits count every request)
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int q = 0; q < QW; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < WD; ++e) asm volatile("" ::"v"(w[0][n][q][h][e]), "v"(w[1][n][q][h][e]));
  __builtin_amdgcn_s_waitcnt(gemm::waitcnt_vm(0));
  __syncthreads();  // every wave is done with its ring and its tables

  // the waves' sums meet: red[tile, block][wave][lane][4]
  float* const red = reinterpret_cast<float*>(qb_lds);
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int t = 0; t < TB; ++t)
      *reinterpret_cast<float4*>(red + (((n * TB + t) * QB_WAVES + wave) * 64 + lane) * 4) =
          make_float4(acc[n][t][0], acc[n][t][1], acc[n][t][2], acc[n][t][3]);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < (NT * TB + 1) / 2; ++it) {
    // thread -> (tile and block u, token te of the block, row r): 16 consecutive threads = 16 consecutive rows of a token
    const int u = it * 2 + ((int)threadIdx.x >> 8), idx = (int)threadIdx.x & 255;
    const int r = idx & 15, te = idx >> 4;
    if (u < NT * TB) {
      const int n = u / TB, t = u - n * TB;
      const float* src = red + u * QB_WAVES * 256 + ((te >> 2) * 16 + r) * 4 + (te & 3);
      float v = src[0];
#pragma unroll
      for (int wv = 1; wv < QB_WAVES; ++wv) v += src[wv * 256];
      const int row = row_of(n) + r, tok = t * 16 + te;
      if (tok < p.T && row < p.o) {
        if (p.part == nullptr) p.Y[(int64_t)tok * p.o + row] = f32_to_bf16(v);
        else p.part[((int64_t)blockIdx.y * p.T + tok) * p.o + row] = v;
      }
    }
  }
#endif
}

// layers that this form covers
bool qb_layer(const LayerDims& d) {
  const int64_t rb = d.i / 8 * d.bits;
  if (d.i % d.g != 0 || d.o % 8 != 0 || (d.g & (d.g - 1)) != 0) return false;
  if (d.g < (d.bits == 3 ? 128 : 64) || (d.bits != 2 && d.bits != 3 && d.bits != 4 && d.bits != 8)) return false;
  return d.o * rb < (1ll << 31) && d.o * (d.i / d.g) * 4 < (1ll << 31);
}

constexpr int QB_SLICES_MAX = 4;
int qb_tiles_max(const LayerDims& d, int64_t cus) { return (d.o + 15) / 16 <= cus ? 2 : 3; }

// k-slices of at least four macros, none of them empty, whose workgroups all run at once
bool qb_slices_ok(const LayerDims& d, int64_t cus, int nt, int sl) {
  const int64_t tiles = (d.o + 15) / 16, macros = (d.i + 255) / 256;
  return sl <= macros / 4 && (tiles + nt - 1) / nt * sl <= cus && (sl - 1) * ((macros + sl - 1) / sl) < macros;
}

int qb_kstep(const LayerDims& d) { return d.bits == 8 || d.g == 64 ? 64 : 128; }

// groups that a slice can meet, wherever it starts
int qb_groups(const LayerDims& d, const BlocksPlan& plan) {
  if (plan.slices == 1) return (int)(d.i / d.g);
  const int64_t n = ((int64_t)plan.slice_macros * 256 - 1) / d.g + 2;
  return (int)(n < d.i / d.g ? n : d.i / d.g);
}

size_t qb_lds_bytes(const LayerDims& d, const BlocksPlan& plan) {
  const int tb = (int)((d.T + 15) / 16);
  const size_t ring = (size_t)QB_WAVES * qb_ring(tb) * tb * 2048;
  const size_t tab = (size_t)plan.nt * 16 * (((qb_groups(d, plan) + 1) / 2) | 1) * 16;
  const size_t red = (size_t)plan.nt * tb * QB_WAVES * 1024;
  return ring + tab > red ? ring + tab : red;
}

// Estimated time (us), fitted to 11600 calls of 260 layers; over 1275 drawn calls in graphs it is 10 / 7 / 4 / 3 % too high on average
// (one to four token blocks) and 4 to 7 % rms off beside that: workgroups that run one after the other on a unit (two share one
// where registers and LDS allow: `sets` counts the latencies), their bytes of X, their waves' matrix ops, conversions and
// scalings, their outputs; the matrix' bytes; with k-slices the second launch.
double qb_us(const LayerDims& d, int64_t cus, const BlocksPlan& plan) {
  static const double c[4][10] = {
      // fixed, set, 100 KB of X, tiles + 1, conversions, scalings, slices, 4 MB of partial sums, 4 MB of codes, output blocks
      {2.43, 1.09, 0.29, 0.000, 0.32, 0.17, 1.98, 1.33, 0.24, 0.14},
      {1.62, 1.61, 0.50, 0.043, 0.20, 0.11, 2.20, 0.00, 0.29, 0.32},
      {1.59, 1.10, 0.52, 0.071, 0.10, 0.07, 2.25, 0.20, 0.37, 0.29},
      {1.61, 1.39, 0.61, 0.012, 0.31, 0.06, 1.91, 0.85, 0.37, 0.25},
  };
  const int64_t tb = (d.T + 15) / 16;
  const double* k = c[tb - 1];
  const int64_t wgs = ((d.o + 15) / 16 + plan.nt - 1) / plan.nt * plan.slices;
  const bool two = tb == 1 && qb_lds_bytes(d, plan) <= 80 * 1024 && plan.nt * (d.bits == 8 ? 2 : 1) <= 2;
  const double rounds = (double)((wgs + cus - 1) / cus), sets = (double)((wgs + (two ? 2 : 1) * cus - 1) / ((two ? 2 : 1) * cus));
  const int64_t klen = plan.slice_macros * 256 < d.i ? plan.slice_macros * 256 : d.i;
  const double run = (double)((plan.slice_macros + QB_WAVES - 1) / QB_WAVES);  // macros of a wave
  const double conv = d.bits == 3 ? 1.1 : d.bits == 8 ? 1.5 : 1.0, nt = (double)plan.nt;
  double us = k[0] + k[1] * sets + rounds * (k[2] * (double)(klen * d.T) * 2e-5 + k[3] * run * (double)tb * (nt + 1.0) + k[4] * run * nt * conv +
                                             k[5] * run * nt * (double)tb * (qb_kstep(d) == 64 ? 4.0 : 2.0) + k[9] * nt * (double)tb) +
              k[8] * (double)d.o * (double)d.i * d.bits / 32e6;
  if (plan.slices > 1) us += k[6] + k[7] * (double)plan.slices * (double)(d.T * d.o) * 2e-6;
  return us;
}

}  // namespace

size_t qgemm_blocks_workspace_bytes(const LayerDims& d) {
  if (!qb_layer(d)) return 0;
  const int64_t cus = device_compute_units();
  for (int sl = QB_SLICES_MAX; sl > 1; --sl)
    if (qb_slices_ok(d, cus, qb_tiles_max(d, cus), sl)) return (size_t)sl * 64 * (size_t)d.o * sizeof(float);
  return 0;
}

// Which calls take this form, and how.  Measured (us, the other kernels' best / this one):
//   4 bits, groups of 128  [4096 x 4096]  16 / 32 / 43 / 64 tokens 6.4 / 5.6, 11.3 / 7.4, 13.5 / 8.3, 13.8 / 10.2;
//                          [11008 x 4096] 10.9 / 10.3, 15.0 / 13.1, 19.7 / 14.2, 23.2 / 16.8;  groups of 64 [4096 x 4096]
//                          1 / 16 / 43 / 64 tokens 9.7 / 6.2, 13.2 / 6.7, 23.7 / 9.6, 27.3 / 11.2
//   3 bits  [4096 x 11008] 16 / 43 / 64 tokens 14.6 / 10.8, 30.3 / 17.6 (two slices), 29.1 / 20.0
//   8 bits, groups of 64   [4096 x 4096]  16 / 32 / 43 / 64 tokens 8.9 / 8.5, 13.4 / 10.2, 16.0 / 11.2, 15.7 / 12.7
// At few tokens, where the matrix is all there is to load, the in-register form's sixteen waves with every request in the
// first instructions stay ahead on layers of more row tiles than units: 1.1 - 1.4 times up to 2 tokens (8 bits: 3), on rows of one chunk per
// wave (4096) up to 8 tokens with two tiles per unit (8 bits: 16), 12 with three and more (8 bits: 4; in groups of 64, 8); and its two-block form on
// short rows (up to 2048: 1.05 - 1.14 times up to 32 tokens; 2 and 3 bits with one tile per unit up to 512 and 1024, 1.05 times)
// and, up to 24 tokens, with four tiles per unit.  8 bits, short rows and four tiles per unit: 64-row tiles ([14336 x 1024], 20 / 64
// tokens 9.6 / 13.2, 11.2 / 16.5), and with three where these fill most units ([11184 x 512] 31 tokens 7.4 / 8.6, [11808 x 256] 50 6.1 /
// 10.1).  Rows of 128 or 384, whose last macro is half empty, 17 to 32 tokens: the streaming form ([8848 x 128], 8 bits, 5.2 / 6.6;
// 4 bits in groups of 64, rows up to 256 [12000 x 256] 6.0 / 6.9).  One tile per unit: one token
// 0.85 - 1.1 times either way, from two (8 bits: three) on this form; but 4 and 8 bits with the activations in LDS
// (qgemm_decode_kernel) where a wave has one macro of a short row or some waves have one macro more than others: in a graph, us,
// that kernel / this one, 4 bits [512 x 512] 4 tokens 3.7 / 4.0, [4096 x 1024] 2 3.7 / 4.2, [2048 x 3072] 2 4.7 / 5.1, [2048 x 5120]
// 2 5.4 / 5.8; 8 bits [2048 x 512] 3 3.6 / 4.4, 16 3.9 / 4.5, [512 x 1536] 4 4.0 / 4.3, groups of 64 [8192 x 384] 16 4.4 / 5.6.
// 2 and 3 bits, two tiles per unit, rows of two chunks per wave (6144 to 8192): in registers up to 7 tokens ([8192 x 8192], 3 bits,
// 3 tokens 11.3 / 11.9).
BlocksPlan qgemm_blocks_plan(const LayerDims& d, bool have_workspace) {
  const BlocksPlan none = {0, 1, 0, 0.0};
  if (d.T > 64 || !qb_layer(d) || d.T * d.i * 2 >= (1ll << 31)) return none;
  const int64_t tiles = (d.o + 15) / 16, cus = device_compute_units(), macros = (d.i + 255) / 256;
  const int64_t per_unit = (tiles + cus - 1) / cus;
  if (d.g >= 128 || d.bits == 8) {  // (2 and 4 bits in groups of 64 have no other fast form)
    int from = d.bits == 8 ? 3 : 2;
    if (per_unit > 1 && d.i > 4096) from = d.bits == 8 ? 4 : 3;
    else if (per_unit > 1) from = d.g < 128 ? 9 : per_unit == 2 ? (d.bits == 8 ? 17 : 9) : d.bits == 8 ? 5 : 13;
    if ((d.bits == 2 || d.bits == 3) && per_unit == 2 && d.i > 6144 && d.i <= 8192) from = 8;
    if (d.bits == 8 && d.g < 128 && per_unit > 1 && d.i <= 1024) from = 17;
    if (d.T < from) return none;
    // (calls that the in-register form does not take: qgemm_decode_kernel's)
    if (per_unit == 1 && d.T <= 16 && (d.bits == 4 || (d.bits == 8 && (2 * tiles < cus || d.g < 128)))) {
      if (d.i <= 1024 && d.T <= (d.bits == 8 || d.i <= 512 ? 16 : 12)) return none;
      if ((d.bits == 8 && d.i <= 1536) || (d.i > 2048 && d.i <= 3072)) {
        if (d.T <= (d.bits == 8 ? 6 : 4)) return none;
      }
      if (d.T == 2 && d.i > 4096 && d.i <= 5120) return none;
    }
    if (d.g >= 128 && d.bits != 8 && d.T > 16 &&
        ((per_unit > 1 && d.i <= 2048 && d.T <= 32) || (per_unit > 3 && d.i <= 4096 && d.T <= 24)))
      return none;
    if (d.g >= 128 && d.bits < 4 && d.T > 16 && d.T <= 32 && per_unit == 1 && d.i <= (d.bits == 3 ? 1024 : 512)) return none;
    if (d.bits == 8 && per_unit > 3 && d.i <= 2048) return none;
    if (d.bits == 8 && per_unit == 3 && d.i % 128 == 0 && (d.i <= 512 || (d.i <= 1024 && d.T > 48)) && d.T > 16) {
      const int64_t wide = (d.o + 63) / 64;
      if (8 * wide >= 5 * ((wide + cus - 1) / cus) * cus) return none;
    }
    if (d.bits == 8 && per_unit > 1 && d.T > 16 && d.T <= 32 && d.i < 512 && d.i % 256 == 128 && (d.g < 128 || (per_unit == 3 && d.i == 128)))
      return none;
  } else if (d.bits == 4 && per_unit > 2 && d.T > 16 && d.T <= 32 && d.i <= 256) {
    return none;
  }
  BlocksPlan best = none, best_split = none;
  auto fits = [&](const BlocksPlan& plan) { return qb_lds_bytes(d, plan) <= 160 * 1024; };
  // beyond a block, as many tiles per workgroup as give one round of them, where their tables fit; slices within a round
  const int whole = (int)(d.T > 16 && per_unit <= 3 ? per_unit : 1);
  const int nt_min = fits({whole, 1, (int)macros, 0.0}) ? whole : 1;
  for (int nt = nt_min; nt <= qb_tiles_max(d, cus); ++nt)
    for (int sl = 1; sl <= QB_SLICES_MAX; ++sl) {
      BlocksPlan plan = {nt, sl, (int)((macros + sl - 1) / sl), 0.0};
      if (!fits(plan) || (per_unit == 1 && nt > 1 && sl == 1)) continue;
      if (sl > 1 && (!have_workspace || !qb_slices_ok(d, cus, nt, sl))) continue;
      plan.us = qb_us(d, cus, plan);
      BlocksPlan& b = sl > 1 ? best_split : best;
      if (b.nt == 0 || plan.us < b.us) b = plan;
    }
  // (at four token blocks the estimate is 0.2 us too good for slices: of 4700 layers with both measured, the slices it takes are
  // more than 3 % slower than one slice on 31 and up to 2.2 times as fast on the others)
  const double off = d.T > 48 ? 0.2 : 0.0;
  // (a second launch is 2.7 us of the caller's time: in a loop of eager calls one launch takes 7.8 us, two 10.4, whatever the
  // kernels take; in a graph slices gain 0.7 us on layers of 7 to 8 us in one slice, 1.4 on those of 9 to 10.  At 8.5 what the
  // one loses is what the other gains)
  if (best.nt > 0 && (best_split.nt == 0 || best.us < 8.5 || best.us <= best_split.us + off)) return best;
  return best_split;
}

void launch_qgemm_blocks(const BlocksPlan& plan, const LayerDims& d, const bf16_t* X, const uint32_t* packed,
                         const float* scale, const float* zero, bf16_t* Y, float* partial, hipStream_t stream) {
  QbArgs a;
  a.X = X; a.packed = packed; a.scale = scale; a.zero = zero; a.Y = Y;
  a.part = plan.slices > 1 ? partial : nullptr;
  a.T = (int)d.T; a.o = (int)d.o; a.i = (int)d.i;
  a.gshift = __builtin_ctz((unsigned)d.g);
  a.slice_macros = plan.slice_macros;
  const int kstep = qb_kstep(d), tb = (int)((d.T + 15) / 16);
  a.tab_groups = qb_groups(d, plan);
  const size_t lds = qb_lds_bytes(d, plan);
  const dim3 grid((unsigned)(((d.o + 15) / 16 + plan.nt - 1) / plan.nt), (unsigned)plan.slices);
#define L4Q_QB(B, K, N, P)                                                                                    \
  do {                                                                                                        \
    if (lds > 64 * 1024)                                                                                      \
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&qgemm_blocks_kernel<B, K, N, P>),              \
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);                      \
    hipLaunchKernelGGL((qgemm_blocks_kernel<B, K, N, P>), grid, dim3(QB_WAVES * 64), lds, stream, a);         \
  } while (0)
#define L4Q_QB_T(B, K, N)                                                                     \
  do {                                                                                        \
    if (tb == 1) L4Q_QB(B, K, N, 1); else if (tb == 2) L4Q_QB(B, K, N, 2); else if (tb == 3) L4Q_QB(B, K, N, 3); else L4Q_QB(B, K, N, 4); \
  } while (0)
#define L4Q_QB_N(B, K)                                                                                     \
  do {                                                                                                     \
    if (plan.nt == 1) L4Q_QB_T(B, K, 1); else if (plan.nt == 2) L4Q_QB_T(B, K, 2); else L4Q_QB_T(B, K, 3); \
  } while (0)
  if (d.bits == 8) L4Q_QB_N(8, 64);
  else if (d.bits == 3) L4Q_QB_N(3, 128);
  else if (d.bits == 4 && kstep == 64) L4Q_QB_N(4, 64);
  else if (d.bits == 4) L4Q_QB_N(4, 128);
  else if (kstep == 64) L4Q_QB_N(2, 64);
  else L4Q_QB_N(2, 128);
#undef L4Q_QB_N
#undef L4Q_QB_T
#undef L4Q_QB
}

}  // namespace l4q

// Merge + quantize pass, streaming form for bfloat16 storage (Sec. 3.2, Eqs. l4q_Wcombine, l4q_Wquant,
// l4q_Wdequant; the backward form also leaves what the fused weight-gradient kernel needs: Wq^T, the
// d(Wq)/d(scale) factor of Eq. quant_lsq_s with the straight-through mask of Eq. appen_ste in its magnitude, B^T).
//
// Bound: memory for the forward, statistics and packing forms, vector arithmetic for the backward and initialisation forms:
// binary32 matrix ops and vector ops take turns (measured: a loop of each runs in the sum of their times, while bfloat16
// matrix ops run beside vector ops), and 45 M weights x one vector op are 1.15 us of the chip.  A wavefront owns 64 columns of
// the weight and walks a run of row blocks of 32 down them; it shares nothing with the others of its workgroup (but for the
// initialisation form in groups above 64, which joins the extremes of two or four wavefronts).  One resident round of
// workgroups covers the matrix; ids are dealt out so that an XCD works on whole rows (scale, zero and B are then fetched by
// one L2 each: 49 -> 46 us at 11008 x 4096 forward).
//  * A lane works on one row and 32 consecutive columns, one group: s, b and 1 / s are per-lane values, extremes and
//    error sums need no exchange, 32 codes are `bits` whole words, and the matrix op's registers are the lane's columns in
//    order (its M axis stands for the columns, see jm).  Only the 2-byte weights and results change lanes, through a 4 KiB
//    tile of LDS, so that every load and store instruction covers whole cache lines.
//  * Memory: the weights of the next row block are in flight while this one is worked on, its factors and parameters from the
//    middle of this one on.  Loads and stores return in order of issue on one counter, so nothing may be waited for between
//    a request and its use a row block later: no copies of requested registers at the loop's end, no request on a branch.
//  * The stated rank sums sum_k B[p,k] A[k,j], k ascending, one rounding per step, are a chain of K = 1 binary32 matrix ops
//    with the bfloat16 product exact: 64 cycles of the vector unit's time per k and 32 rows x 64 columns.  Forms whose result
//    needs the codes alone (forward, packing) take near sums instead, from bfloat16 matrix ops (16 k at once, products
//    exact, binary32 accumulation in the hardware's own order), and near quotients x (1/s), and settle what they cannot
//    decide: a code is that of the stated arithmetic unless the near quotient w' lies within `tol` of a tie k + 1/2.
//      tol = |gamma| D / s + 4 u |b| / s + 8 u R,   u = 2^-24, R = 2^(n-1) + 1 >= |w| wherever the code is not clear of the grid.
//      D = 4 r u S bounds the difference of the two sums, S = sum_k |B[p,k] A[k,j]| <= max |A| of the wavefront's columns x
//      sum_k |B[p,k]|.  The stated sum is (r - 1) u S off at most (products exact).  A matrix op adds in an order and width of
//      its own; taken for granted is that it forms exact products and adds them to the accumulator in steps of 4 or more, a
//      step's terms aligned to the largest and cut to 24 bits or more, below 2 u S lost of each, the step's result rounded or
//      cut, 2 u S more: 2 r u S, and 2 u S for each of at most r / 4 steps (+ 2 where half of the last op's products are zeros).
//      Measured: 7.8 u S at ranks 8 to 32, 15.6 at 64, 63 at 256, one large product beside others just below its last place; on
//      random ones 1 to 4 u S, 11 at rank 256 with exponents 60 apart.  Subnormal factors are not lost.
//      The rest: Wc is rounded once on either side (u |Wc| each, |Wc| <= |b| + R s), gamma acc where gamma is no power of two (in
//      D), the stated x and w once (u R each); near: 1 / s, which multiplies Wc - b as a whole (u R), b / s (u |b| / s), the sum
//      (u R): 3 u |b| / s + 6 u R.
//    An infinity or NaN in A or B makes tol one, and nothing passes.  What is undecided depends on the layer's state.  In the
//    middle of a run (B moved, scales no simple fractions of the weights) 2 % of the row blocks hold such a weight at 4 bits,
//    24 % at 8 (counted, groups of 128).  At the start, B = 0 and min / max scales of bfloat16 weights, 2 to 7 weights of a row
//    block, and some in 80 to 99 % of them, lie exactly on ties; but sums of nothing are not near, they are the stated ones:
//    a row block whose rows of B are all zero (or whose A is) takes W0 and the stated quotient and leaves nothing undecided, as
//    the layers without a rank term do.
//    Undecided weights are settled by the stated sum, one of every lane at a time, from the operands in registers (ranks above
//    what they hold: one at a time, from memory); a row block with more than 3 in a lane is repeated by the stated arithmetic, and
//    the next 3 go there directly.  (Most in a lane 1 / 3 / 8, packing 11008 x 4096: 16 a row block 61 / 48 / 48 us, 128 61 / 61 /
//    69.  Every weight on a tie: 61, going there directly 48.)
//    us, weights from HBM; chain with sums through LDS / here: forward 11008 x 4096, rank 16, in the middle of a run 46 / 37, at
//    the start 46 / 37, 8 bits 45 / 39; 4096 x 11008 at rank 64 100 / 50; 4096 x 4096, groups of 64, 20.4 / 14.0; packing
//    11008 x 4096 49 / 32, at the start 47 / 32, 8 bits 45 / 39.  (Every undecided row block repeated, ties of the start
//    included: forward 86 at the start, packing 63 and at 8 bits 50.)  Slower than the chain, 0.7 to 0.9 times: weights held on
//    ties by a B that is not zero but too small to move them.
//    Error sums, which no single code decides, use the near values (but where a quotient overflows): 45 / 18 with
//    much of the weight in the memory-side cache, 23 from HBM.
//  * Forms that need the quotient itself (backward: the factor; export) do not spend the 11-instruction IEEE expansion per
//    weight: with the correctly rounded reciprocal r = RN(1 / s) (hardware estimate, one Newton step, then the
//    choice among the result and its two neighbours by the exact residual 1 - s r),
//    q = x r;  t = fma(-s, q, x);  w = fma(t, r, q)  after clamping x to +-1024 s.
//    q is within one unit of x / s and the corrected w is the correctly rounded quotient
//    (Markstein's theorem on division by multiplication with the reciprocal and one exact-remainder correction), so codes
//    and mask are those of the stated arithmetic.  |x| > 1024 s lies beyond every code grid, where code, mask and
//    factor depend on the sign of x alone.  Scales outside [2^-60, 2^60] take the IEEE divide instead (wave-uniform
//    branch).  l4q_check_fast_divide compares the sequence with the IEEE divide on the GPU for every significand of s.
//  * Wq and Wq^T leave in the blocked layout the GEMM reads (32 k-values of all rows together), 1 KiB per store instruction.
//  * gamma a power of two (alpha = 2 r, the usual choice): gamma acc is exact, and W0 + gamma acc is one fused
//    multiply-add with the same bits.
// Shapes: bfloat16, rank a multiple of 8, group size >= 32 (so rows are whole runs of 32); anything else runs
// merge_quant_tile_kernel.
#include <type_traits>

#include "l4q_device.h"
#include "l4q_kernels.h"

namespace l4q {

namespace {

constexpr int MS_COLS = 256;                     // columns per workgroup: 4 wavefronts x 64
constexpr int MS_THREADS = 256;
// Wavefronts per SIMD, and workgroups per compute unit of the one resident round, of a form.  As few as keep the memory busy: a
// wavefront starts with a fetch of A and of its first row block that nothing hides, and more registers mean no spills.  us at 2 / 3 /
// 4, weights from HBM, 11008 x 4096 and 13824 x 5120: forward 39 / 39 / 42 and 64 / 63 / 67, rank 64 48 / 140 / 183 and 76 / 216 /
// 292; backward 57 / 56 / 59 and 97 / 92 / 100, rank 64 92 / 91 / 135; codes 43 / 42 / 50 and 70 / 69 / 79; error sums 23 / 24 / 23
// and 39 / 38 / 39 (and fewer pairs to add); initialisation 30 / 29 / 27 and 44 / 41 / 40; packing 32 / 32 / 65 and 51 / 51 / 103.
// 4096 x 4096 and 2048 x 2048 within 1 us of the best.
template <int MODE, int ACH> constexpr int ms_waves() {
  return MODE == 5 ? 4 : MODE == 4 || (MODE == 1 && ACH > 1) ? 2 : 3;
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x32_t __attribute__((ext_vector_type(32)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// the value of another lane of the same 16 (DPP control word)
template <int CTRL> __device__ __forceinline__ uint32_t lane_swap(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
// the values of lanes l % 32 and 32 + l % 32
__device__ __forceinline__ uint2 both_halves(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto t = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return make_uint2(t[0], t[1]);
#else
  return make_uint2(v, v);
#endif
}
__device__ __forceinline__ float2 both_halves(float v) {
  const uint2 t = both_halves(__float_as_uint(v));
  return make_float2(__uint_as_float(t.x), __uint_as_float(t.y));
}
__device__ __forceinline__ float half_sum(float v) {
  const float2 t = both_halves(v);
  return t.x + t.y;
}

// What one row block (32 rows x 64 columns) needs of the factors and the quantizer parameters.  Those of the next row block
// are requested as soon as the current one has consumed its own, before its streaming phase.
template <int ACH>
struct FactorLoads {
  u32x4 b[ACH > 0 ? ACH : 1];  // B[p, 16 c + 8 h .. + 7] of chunk c
  float s, z;                  // scale / zero of row p = p0 + lane % 32, group of this lane's 32 columns
};

// Bytes of LDS per wavefront: a tile of 32 rows x 128 bytes, in 16-byte pieces; backward: a second one for the factor;
// export: 32 rows x 256 bytes (binary32); initialisation: two sets of 32 pairs behind the tile.
template <int MODE> constexpr int ms_wave_lds() { return MODE == 2 || MODE == 3 ? 8192 : MODE == 5 ? 4096 + 512 : 4096; }
template <int MODE> constexpr int ms_lds() { return 4 * ms_wave_lds<MODE>(); }

// MODE 1: forward (dequantized Wq, [ld_wq / 32][o][32]).  MODE 2: backward (Wq^T, [ld_wqT / 32][i][32]; optionally the
// factor [o, i] and B^T).  MODE 3: export (any of int8 codes, binary32 merged weight, mask; all [o, i]).  MODE 4: error
// sums, one pair per wavefront.  MODE 5: scale / zero from the groups' extremes.  MODE 6: packed codes of BITS bits.
// Grid: 256-column strips x partitions of the row blocks; wavefront w of a workgroup walks the row blocks
// [nrb part / parts, nrb (part + 1) / parts) of its 64 columns.
// ACH: 16-k chunks of the rank whose A values a wavefront keeps in registers for its whole run (1: ranks up to 16;
// 4: ranks up to 64, further chunks are loaded where they are used; 0: no rank term, Wc = W0, and A and B are not read).
template <int MODE, bool GAMMA_POW2, int ACH, int BITS = 0>
__device__ __forceinline__ void merge_quant_stream_body(const LayerDims& d, const bf16_t* __restrict__ W0,
                                                        const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                        const float* __restrict__ scale,
                                                        const float* __restrict__ zero,
                                                        const MergeQuantOut<bf16_t>& out, int nrb,
                                                        unsigned char* lds_all) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  [[maybe_unused]] unsigned char* tile = lds_all + wave * ms_wave_lds<MODE>();
  // Workgroup ids go round-robin over the 8 XCDs: each XCD gets a contiguous run of row partitions with all their strips
  const int strips = (int)((d.i + MS_COLS - 1) / MS_COLS), parts = (int)gridDim.x / strips;
  const int total = (int)gridDim.x, xcd = (int)blockIdx.x & 7, at_xcd = (int)blockIdx.x >> 3;
  const int id = xcd * (total >> 3) + (xcd < (total & 7) ? xcd : total & 7) + at_xcd;
  const int strip = id % strips, part = id / strips;
  const int jw = strip * MS_COLS + wave * 64;  // first column of this wavefront
  const int i = (int)d.i, o = (int)d.o, r = d.r, g = d.g;
  const int G = i / g;
  const int rb_begin = (int)((int64_t)nrb * part / parts);
  const int rb_end = (int)((int64_t)nrb * (part + 1) / parts);
  if constexpr (MODE == 2) {
    // B^T for this partition's rows (zeros from o to its leading dimension), dealt out over the strips; where rows are whole
    // 16-byte pieces, 8 ranks of a row per thread.  (All of it on the first strip's workgroups, by elements: an 11008 x
    // 4096 weight at rank 16 67 us, here 60; rank 256 without a rank term of the pass's own 128, here 35.)
    if (out.bT) {
      const int ld = (int)out.ld_bT, rank = out.bT_rank;
      const int pa = rb_begin * 32, pe = rb_end * 32 < ld ? rb_end * 32 : ld;
      const int np = pe - pa, step = strips * MS_THREADS;
      if (rank % 8 == 0) {
        for (int idx = strip * MS_THREADS + (int)threadIdx.x; idx < rank / 8 * np; idx += step) {
          const int k = idx / np * 8, p2 = pa + idx % np;
          u32x4 v = {0u, 0u, 0u, 0u};
          if (p2 < o) v = *reinterpret_cast<const u32x4*>(B + (int64_t)p2 * rank + k);
#pragma unroll
          for (int e = 0; e < 8; ++e) out.bT[(int64_t)(k + e) * ld + p2] = (bf16_t)(e & 1 ? v[e / 2] >> 16 : v[e / 2]);
        }
      } else {
        for (int idx = strip * MS_THREADS + (int)threadIdx.x; idx < rank * np; idx += step) {
          const int k = idx / np, p2 = pa + idx % np;
          out.bT[(int64_t)k * ld + p2] = p2 < o ? B[(int64_t)p2 * rank + k] : (bf16_t)0;
        }
      }
    }
  }
  double err_q = 0.0, err_c = 0.0;  // MODE 4: this lane's share of the wavefront's sums
  float* const err_out = MODE == 4 ? out.errors + 2 * ((int64_t)id * 4 + wave) : nullptr;
  if (jw >= i) {  // a whole wavefront past the last column (MODE 5's barriers count the wavefronts that are left)
    if (MODE == 4 && lane < 2) err_out[lane] = 0.f;
    return;
  }

  // A lane works on row p0 + lane % 32 and the 32 consecutive columns from jl; i is a multiple of 32, so they are all
  // inside or all outside, and of one group.
  const int l32 = lane & 31, h = lane >> 5;
  const int jl = jw + 32 * h;
  const bool col_ok = jl < i;
  const int qtab = jl / g;
  // The matrix op's M axis is the columns: M index m = 8 q + 4 hh + e of column block b ends in register 4 q + e of half-wave
  // hh.  With m standing for column 32 hh + 16 b + 4 q + e the registers of a lane are its 32 columns in order.
  const int jm = jw + 32 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3);  // + 16 b

  const __amdgpu_buffer_rsrc_t rsW0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W0), 0, o * i * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, r * i * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(B), 0, o * r * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(scale), 0, o * G * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsZ = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(zero), 0, o * G * 4, 0x00020000);
  constexpr unsigned OOB = 0x80000000u;
  constexpr bool FILTER = MODE == 1 || MODE == 4 || MODE == 6, CHECKED = FILTER && MODE != 4;
  constexpr bool REST = ACH > 0 && !(MODE <= 2 && ACH == 1);  // ranks above 16 ACH (the forward and backward forms have ACH = 4 for them)
  constexpr bool FACTOR = MODE == 2 && ACH > 0;  // (the layers without a rank term take no factor)

  // Memory role of a row-major tile: instruction t, lane = row 8 t + lane / 8, piece lane % 8 (whole 128-byte lines).  Piece
  // c of row p lies at position c ^ (p % 8) of its row in LDS, so that 8 consecutive lanes meet all banks in either role.
  const int mr = lane >> 3, mc = lane & 7;
  const bool mcol_ok = jw + 8 * mc < i;
  // LDS offsets of the two roles, recomputed from one base each per row block: left to itself the compiler keeps
  // every address of the loop in a register of its own and spills the sums for them
  uint32_t mem_base = (uint32_t)(wave * ms_wave_lds<MODE>() + mr * 128 + ((mc ^ mr) << 4));                     // + 1024 t
  uint32_t row_base = (uint32_t)(wave * ms_wave_lds<MODE>() + l32 * 128 + (((4 * h) ^ (l32 & 7)) << 4));        // ^ 16 c
  auto lds16 = [&](uint32_t at) -> u32x4& { return *reinterpret_cast<u32x4*>(lds_all + at); };

  // every load of row block rb; past the wavefront's range (or the matrix) the offsets are out of range: nothing moves
  FactorLoads<ACH> F;
  auto load_b = [&](int p, bool row_ok, int k0) {  // (rank a multiple of 8: a lane's 8 values are all inside or all outside)
    return __builtin_amdgcn_raw_buffer_load_b128(
        rsB, (int)(row_ok & (k0 + 8 * h < r) ? (unsigned)((p * r + k0 + 8 * h) * 2) : OOB), 0, 0);
  };
  auto request_factors = [&](int rb) {
    const int p = rb * 32 + l32;
    const bool row_ok = (rb < rb_end) & (p < o);
#pragma unroll
    for (int c = 0; c < ACH; ++c) F.b[c] = load_b(p, row_ok, 16 * c);
    if (MODE == 5) return;
    const unsigned vt = row_ok & col_ok ? (unsigned)((p * G + qtab) * 4) : OOB;
    F.s = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsS, (int)vt, 0, 0));
    F.z = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsZ, (int)vt, 0, 0));
  };
  u32x4 next_w[4];
  auto request_weights = [&](int rb) {  // (rows from o on lie past the end of the buffer)
    const unsigned vw = (rb < rb_end) & mcol_ok ? (unsigned)(((rb * 32 + mr) * i + jw + 8 * mc) * 2) : OOB;
#pragma unroll
    for (int t = 0; t < 4; ++t) next_w[t] = __builtin_amdgcn_raw_buffer_load_b128(rsW0, (int)(vw + (unsigned)(t * 16 * i)), 0, 0);
  };
  auto lds_order = [&] {  // a wavefront's own LDS accesses stay in program order; the compiler has to keep it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  request_weights(rb_begin);
  request_factors(rb_begin);

  // A of the first ACH rank chunks, two bfloat16 per register, loaded once per wavefront.  FILTER: operand fragments of the
  // bfloat16 matrix op, A[16 c + 8 h + e, jm + 16 b] at [8 c + 4 b + e / 2].  Else A[16 c + k, jm + 16 h] at [8 c + k / 2].
  uint32_t apk[ACH > 0 ? 8 * ACH : 1];
  const unsigned voffA = jm + 16 * h < i ? (unsigned)((jm + 16 * h) * 2) : OOB;
  // chunk k0 .. k0 + 15 as fragments
  auto load_fragments = [&](int k0, uint32_t (&f)[8]) {
    uint32_t raw[16];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        raw[8 * b + e] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
            rsA, (int)(jm < i && k0 + 8 * h < r ? (unsigned)((8 * h * i + jm + 16 * b) * 2) : OOB), (k0 + e) * i * 2, 0);
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = raw[2 * q] | (raw[2 * q + 1] << 16);
  };
  if constexpr (FILTER) {
#pragma unroll
    for (int c = 0; c < ACH; ++c) {
      uint32_t f[8] = {};
      if (c == 0 || 16 * c < r) load_fragments(16 * c, f);
#pragma unroll
      for (int q = 0; q < 8; ++q) apk[8 * c + q] = f[q];
    }
  } else {
#pragma unroll
    for (int c = 0; c < ACH; ++c) {
      uint32_t araw[16];
#pragma unroll
      for (int k = 0; k < 16; ++k)  // steps past the rank: a valid row is read; the B factor of that step is zero
        araw[k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsA, (int)voffA, (16 * c + k < r ? 16 * c + k : r - 1) * i * 2, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) apk[8 * c + k] = araw[2 * k] | (araw[2 * k + 1] << 16);
    }
  }
  [[maybe_unused]] const float sum_tol = fabsf(d.gamma) * (float)r * 0x1p-22f;  // CHECKED: |gamma| D / S
  float top_a = 0.f;                                                            // max |A| of the wavefront's columns
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  [[maybe_unused]] u16x2 a_max = {0, 0};  // of this lane's part of it (magnitudes of bfloat16 order as integers, NaN above infinity)
  auto take_max = [](u16x2& m, uint32_t v) { m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v & 0x7FFF7FFFu)); };
  auto all_max = [&](const u16x2& m) {
    uint32_t w = m[0] > m[1] ? m[0] : m[1];
    auto take_lane = [&](uint32_t v) { w = w > v ? w : v; };
    take_lane(lane_swap<0xB1>(w));   // quad_perm: lane ^ 1
    take_lane(lane_swap<0x4E>(w));   // quad_perm: lane ^ 2
    take_lane(lane_swap<0x141>(w));  // row_half_mirror
    take_lane(lane_swap<0x140>(w));  // row_mirror
    uint32_t top = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)w, 16 * q);
      top = top > v ? top : v;
    }
    return __uint_as_float(top << 16);
  };
  if constexpr (CHECKED && ACH > 0) {
#pragma unroll
    for (int q = 0; q < 8 * ACH; ++q) take_max(a_max, apk[q]);
    top_a = all_max(a_max);
  }

  auto odd_even = [](uint32_t v, int k) { return __uint_as_float(k & 1 ? v & 0xFFFF0000u : v << 16); };
  // one chunk of the stated sum: k ascending, RN(acc + b a) each; rank steps past r have a zero factor.  Each half-wave holds
  // 8 of the 16 values of B, and both need all of them.
  auto chain = [&](f32x32_t& sum, const u32x4& bq, const uint32_t* a) {
    uint32_t bw[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint2 t = both_halves(bq[q]);
      bw[q] = t.x;
      bw[4 + q] = t.y;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
      sum = __builtin_amdgcn_mfma_f32_32x32x1f32(odd_even(a[k >> 1], k), odd_even(bw[k >> 1], k), sum, 0, 0, 0);
  };
  // chunks from k_first on, loaded where they are used
  auto chain_rest = [&](f32x32_t& sum, int p, bool row_ok, int k_first) {
    for (int k0 = k_first; k0 < r; k0 += 16) {
      const u32x4 bq = load_b(p, row_ok, k0);
      uint32_t araw[16], a[8];
#pragma unroll
      for (int k = 0; k < 16; ++k)
        araw[k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsA, (int)voffA, (k0 + k < r ? k0 + k : r - 1) * i * 2, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) a[k] = araw[2 * k] | (araw[2 * k + 1] << 16);
      chain(sum, bq, a);
    }
  };

  // nothing is outstanding where the loop is entered: else its waits are set for the entry's count of requests, which has no stores
  // between, and each iteration waits for the last one's stores
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
  uint32_t no_bits = 0;
  asm volatile("" : "+s"(no_bits));
  int rb = rb_begin;
  // CHECKED: row blocks ahead that go straight to the stated sums.  From the start where A is not in registers, a wavefront has one
  // or two row blocks, so that little hides the settling (1 us a weight at rank 64, 2 at 256), and the weights to settle are many:
  // at 8 bits, or at high ranks in a launch that leaves units idle.  us, stated / near sums, in the middle of a run (at the start of
  // one the near sums would have been faster, as their last figure says): packing, 8 bits, 1024 x 1024 rank 24 5.9 / 7.8, 64 7.6 /
  // 12.7 (5.2), 2048 x 2048 rank 64 11.8 / 14.9 (7.6), 4 bits, 1024 x 1024 rank 256 17 / 25 (9), 72 9.3 / 7.0; forward, 8 bits, 1024 x
  // 1024 rank 72 12.3 / 13.7 (8.3), 1536 x 1536 rank 72 18.3 / 15.0, 128 22.3 / 26.0, 4 bits, 1024 x 1024 rank 256 20 / 26 (13),
  // 128 15.4 / 15.7 (10), 2048 x 2048 rank 256 34 / 29; two row blocks, 8 bits, 4096 x 2048: packing rank 64 20.1 / 21.5 (12), 96
  // 25 / 28 (14), 128 30 / 43, forward rank 72 28 / 21, 128 37 / 39.
  const bool idle_units = (int)gridDim.x <= 256, high_rank = r >= (MODE == 1 ? 136 : 128);
  const bool many = d.bits == 8 ? (2 * parts >= nrb && r >= (MODE == 1 ? 128 : 96)) || (parts >= nrb && (MODE != 1 || idle_units))
                                : parts >= nrb && high_rank && idle_units;
  [[maybe_unused]] int direct = CHECKED && REST && r > 16 * ACH && many ? rb_end - rb_begin : 0;
  do {  // (no partition is empty)
    const int p0 = rb * 32, p = p0 + l32;
    const bool row_ok = p < o;
    asm volatile("" : "+v"(mem_base), "+v"(row_base));
    if constexpr (ACH > 0) {  // (A stays packed: unpacked ahead of the loop it is spilled)
#pragma unroll
      for (int k = 0; k < 8 * ACH; ++k) asm volatile("" : "+v"(apk[k]));
    }
    // ---- this row block's weights: memory role -> one row per lane
#pragma unroll
    for (int t = 0; t < 4; ++t) lds16(mem_base + 1024 * t) = next_w[t];
    if constexpr (FILTER) request_weights(rb + 1);
    lds_order();
    u32x4 w0[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) w0[c] = lds16(row_base ^ (16 * c));

    // ---- rank sums
    f32x16_t near[2];  // FILTER: near[b][e] of column 16 b + e
    f32x32_t sum;
    float bsum = 0x1p-118f;  // CHECKED: sum_k |B[p,k]| of this lane's k; above what subnormal ones come to, which the op drops
    uint32_t bany = 0;       // CHECKED: any bit of their magnitudes
    if constexpr (FILTER) {
#pragma unroll
      for (int e = 0; e < 16; ++e) near[0][e] = near[1][e] = 0.f;
      auto add_chunk = [&](const u32x4& bq, const uint32_t* a) {
        const bf16x8_t fb = __builtin_bit_cast(bf16x8_t, bq);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const u32x4 fa = {a[4 * b], a[4 * b + 1], a[4 * b + 2], a[4 * b + 3]};
          near[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fa), fb, near[b], 0, 0, 0);
        }
        if constexpr (CHECKED) {
          typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const uint32_t pair = bq[q] & 0x7FFF7FFFu;
            bsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair),
                                                   __builtin_bit_cast(bf16x2_t, 0x3F803F80u), bsum, false);
            bany |= pair;
          }
        }
      };
#pragma unroll
      for (int c = 0; c < ACH; ++c)
        if (c == 0 || 16 * c < r) add_chunk(F.b[c], apk + 8 * c);  // (uniform)
      [[maybe_unused]] u16x2 m = a_max;
      for (int k0 = 16 * ACH; REST && k0 < r && (!CHECKED || direct == 0); k0 += 16) {
        uint32_t f[8];
        load_fragments(k0, f);
        add_chunk(load_b(p, row_ok, k0), f);
        if constexpr (CHECKED) {  // (here and not ahead of the row blocks: another fetch of A, 14.1 us against 10.3 at 256 x 256, rank 72)
#pragma unroll
          for (int q = 0; q < 8; ++q) take_max(m, f[q]);
        }
      }
      if constexpr (CHECKED && REST) {
        if (r > 16 * ACH) top_a = all_max(m);
      }
    } else if constexpr (ACH > 0) {
#pragma unroll
      for (int e = 0; e < 32; ++e) sum[e] = 0.f;
#pragma unroll
      for (int c = 0; c < ACH; ++c)
        if (c == 0 || 16 * c < r) chain(sum, F.b[c], apk + 8 * c);  // (uniform)
      if constexpr (REST) chain_rest(sum, p, row_ok, 16 * ACH);
    }

    // ---- this lane's group: s, b, RN(1 / s), 1024 s
    // (by an op, into registers of their own, so that the next row block's can be fetched into F's: otherwise the loop ends in
    // copies that wait for that fetch)
    const float s = __uint_as_float(__float_as_uint(F.s) ^ no_bits), b = __uint_as_float(__float_as_uint(F.z) ^ no_bits);
    [[maybe_unused]] u32x4 b_now[ACH > 0 ? ACH : 1];
    if constexpr (CHECKED) {
#pragma unroll
      for (int c = 0; c < ACH; ++c) b_now[c] = F.b[c] ^ no_bits;
    }
    const bool bad_scale = MODE != 5 && row_ok && col_ok && !scale_in_fast_range(s);
    const bool slow = __builtin_amdgcn_ballot_w64(bad_scale) != 0;  // wave-uniform
    const float rc = MODE == 5 ? 0.f : exact_reciprocal(s);
    const float hi = s * 1024.f;
    const float nbr = -(b * rc);                                   // FILTER
    if constexpr (!FILTER) request_weights(rb + 1);  // (not before the rank sums: they need the registers)
    request_factors(rb + 1);

    // ---- stream: 32 columns per lane
    float eq = 0.f, ec = 0.f;                                                   // MODE 4
    float lo = __builtin_huge_valf(), top = -__builtin_huge_valf();             // MODE 5: extremes of the lane's columns
    uint32_t words[BITS + 1];                                                   // MODE 6: the lane's columns are BITS whole words
    const uint32_t row_mask = row_ok ? 0xFFFFFFFFu : 0u;                        // MODE 2: zeros below the last row
    u32x4 code8[2], mask8[2], wc4;                                              // MODE 3
    if (MODE == 3) lds_order();  // (its binary32 tile takes the place of the weights)
    float off[4] = {};                                                          // CHECKED: largest |w - code| of 8 columns
    // Merged weights and quotients of columns 8 c .. 8 c + 7.  FORM 0: the stated sums, IEEE divide; 1: the stated sums, quotient
    // by the reciprocal; 2: near sums and quotients; 3: no rank term, quotient by the reciprocal.
    auto stream_columns = [&](auto form_tag) {
      constexpr int FORM = decltype(form_tag)::value;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (FORM == 0) __builtin_amdgcn_sched_barrier(0);
        float wq[8], fg[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int n = 8 * c + e;
          const float wv = odd_even(w0[c][e >> 1], e);
          float wc;
          if constexpr (ACH == 0 || FORM == 3) wc = wv + 0.f;  // (as W0 + gamma 0: a weight of -0 becomes +0)
          else if constexpr (FORM == 2) wc = fmaf(d.gamma, near[n / 16][n % 16], wv);
          else wc = GAMMA_POW2 ? fmaf(d.gamma, sum[n], wv) : wv + d.gamma * sum[n];
          if constexpr (MODE == 5) {
            lo = fminf(lo, wc);
            top = fmaxf(top, wc);
            continue;
          }
          const float x = wc - b;
          const float w = FORM == 2 ? fmaf(wc, rc, nbr) : FORM == 0 ? __fdiv_rn(x, s) : fast_quotient(x, s, rc, hi);
          const float cl = __builtin_amdgcn_fmed3f(w, d.qn, d.qp);
          if constexpr (MODE == 6) {
            // cl + 1.5 2^23 rounds to an integer, ties to even, whose low bits are 0x4B400000 + code; field u = code - Q_N
            constexpr uint32_t C = (1u << (BITS - 1)) - 0x4B400000u;
            const float tf = cl + 12582912.f;
            const uint32_t t = __float_as_uint(tf);
            if (FORM == 2 && ACH > 0) off[c] = fmaxf(off[c], fabsf(cl - (tf - 12582912.f)));
            const int at = BITS * n, k = at / 32, sh = at % 32;
            if (n == 0) {
#pragma unroll
              for (int q = 0; q <= BITS; ++q) words[q] = 0;
            }
            if (sh + BITS <= 32) words[k] += (t << sh) + (C << sh);  // (the constants of a word join at compile time)
            else {
              const uint32_t u = t + C;
              words[k] += u << sh;
              words[k + 1] += u >> (32 - sh);
            }
            continue;
          }
          const float code = rintf(cl);
          if (CHECKED && FORM == 2 && ACH > 0) off[c] = fmaxf(off[c], fabsf(cl - code));
          if (MODE == 1 || MODE == 2) wq[e] = fmaf(code, s, b);
          if (MODE == 4) {
            if (FORM == 2) {  // (in units of s)
              eq += fabsf(w - code);
              ec += fabsf(w - cl);
            } else {
              eq += fabsf(wc - fmaf(code, s, b));
              ec += fabsf(wc - fmaf(cl, s, b));
            }
          }
          if (FACTOR) fg[e] = cl == w ? code - w : code;  // in range = the clamp changed nothing
          if (MODE == 3) {
            const uint32_t byte = (uint32_t)(uint8_t)(int8_t)(int)code, in = cl == w ? 1u : 0u;
            if (n % 4 == 0) code8[n / 16][n / 4 % 4] = mask8[n / 16][n / 4 % 4] = 0;
            code8[n / 16][n / 4 % 4] |= byte << (8 * (n % 4));
            mask8[n / 16][n / 4 % 4] |= in << (8 * (n % 4));
            wc4[n % 4] = __float_as_uint(wc);
            if (n % 4 == 3 && out.wcomb)  // 16-byte piece q of row p of the binary32 tile: position q ^ (p % 16)
              lds16(wave * ms_wave_lds<MODE>() + l32 * 256 + (((8 * h + n / 4) ^ (l32 & 15)) << 4)) = wc4;
          }
        }
        // each piece goes back to LDS as it is finished (a lane's own row: nobody else reads or writes it), over the weights it
        // was made from
        if (FACTOR) {
          typedef _Float16 h2 __attribute__((ext_vector_type(2)));
          typedef float f2 __attribute__((ext_vector_type(2)));
          u32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const f2 q = {fg[2 * e], fg[2 * e + 1]};
            v[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(q, h2));
          }
          lds16((row_base ^ (16 * c)) + 4096) = v;
        }
        if (MODE == 1 || MODE == 2) {
          u32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = pack_bf16x2(wq[2 * e], wq[2 * e + 1]);
            if (MODE == 2) v[e] &= row_mask;
          }
          lds16(row_base ^ (16 * c)) = v;
        }
      }
    };
    // CHECKED: the elements of these lanes within reach of a tie by the stated arithmetic, one of every lane at a time: from
    // registers alone where they hold all of A (a fetch waits for everything the wavefront has in flight: 8 bits, packing
    // 44.6 us against 38.8), else one of one lane.  (All lanes' there, from memory, 8 or 32 ranks at a time: packing 11008 x 4096
    // at rank 64, 8 bits, 76 us against 73, forward 5120 x 5120 at rank 256 115 / 102; four lanes' at a time 77.)  False (and
    // nothing relied on) where a lane has many.
    auto settle = [&](bool unsettled, float edge) {
      uint32_t mine = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (__builtin_amdgcn_ballot_w64(unsettled && !(off[c] < edge)) == 0) continue;
#pragma unroll
        for (int n = 8 * c; n < 8 * c + 8; ++n) {
          const float wc = fmaf(d.gamma, near[n / 16][n % 16], odd_even(w0[n / 8][n % 8 / 2], n));
          const float cl = __builtin_amdgcn_fmed3f(fmaf(wc, rc, nbr), d.qn, d.qp);
          mine |= !(fabsf(cl - rintf(cl)) < edge) ? 1u << n : 0u;
        }
      }
      if (!unsettled) mine = 0;
      if (__builtin_amdgcn_ballot_w64(__builtin_popcount(mine) > 3) != 0) return false;
      for (;;) {
        const uint64_t todo = __builtin_amdgcn_ballot_w64(mine != 0);
        if (todo == 0) return true;
        bool live = mine != 0;
        const int n = live ? __builtin_ctz(mine) : 0;
        float acc = 0.f;
        if (!REST || r <= 16 * ACH) {
          const int from = 4 * (8 * (n % 16 / 4) + 4 * h + n % 4);  // the lane of its column's M index, times 4
#pragma unroll
          for (int c = 0; c < ACH; ++c) {
            uint32_t bw[8], aw[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint2 v = both_halves(b_now[c][q]);
              bw[q] = v.x;
              bw[4 + q] = v.y;
#pragma unroll
              for (int side = 0; side < 2; ++side) {
                const int lo16 = __builtin_amdgcn_ds_bpermute(from + 128 * side, (int)apk[8 * c + q]);
                const int hi16 = __builtin_amdgcn_ds_bpermute(from + 128 * side, (int)apk[8 * c + 4 + q]);
                aw[4 * side + q] = (uint32_t)(n < 16 ? lo16 : hi16);
              }
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) acc = fmaf(odd_even(bw[k / 2], k), odd_even(aw[k / 2], k), acc);
          }
        } else if constexpr (REST) {
          // of the first lane alone, lane = k: one round trip for up to 256 products (exact, but for some below 2^-126, on which no
          // code depends), added in order
          const int at = __builtin_ctzll(todo), col = jw + 32 * (at >> 5) + __builtin_amdgcn_readlane(n, at);
          live = lane == at;
          float prod[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int k = 64 * c + lane;
            const uint32_t bv = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsB, (int)(k < r ? (unsigned)(((p0 + (at & 31)) * r + k) * 2) : OOB), 0, 0);
            const uint32_t av = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsA, (int)(k < r ? (unsigned)((k * i + col) * 2) : OOB), 0, 0);
            prod[c] = odd_even(bv, 0) * odd_even(av, 0);
          }
#pragma unroll
          for (int c = 0; c < 4; ++c)
            for (int k0 = 0; 64 * c + k0 < r && k0 < 64; k0 += 8) {
#pragma unroll
              for (int k = 0; k < 8; ++k)
                acc += __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(prod[c]), k0 + k));
            }
        }
        uint32_t pick[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) pick[q] = w0[q / 4][q % 4];
#pragma unroll
        for (int half = 8; half > 0; half /= 2)
#pragma unroll
          for (int q = 0; q < half; ++q) pick[q] = n & (2 * half) ? pick[q + half] : pick[q];
        const float wv = __uint_as_float(n & 1 ? pick[0] & 0xFFFF0000u : pick[0] << 16);
        const float code = rintf(__builtin_amdgcn_fmed3f(fast_quotient(wv + d.gamma * acc - b, s, rc, hi), d.qn, d.qp));
        if constexpr (MODE == 1) {
          if (live) *reinterpret_cast<bf16_t*>(lds_all + ((row_base ^ (16 * (n / 8))) + 2 * (n % 8))) = f32_to_bf16(fmaf(code, s, b));
        }
        if constexpr (MODE == 6) {
          const uint64_t field = live ? (uint64_t)((1u << BITS) - 1u) << (BITS * n % 32) : 0;
          const uint64_t u = (uint64_t)(uint32_t)((int)code + (1 << (BITS - 1))) << (BITS * n % 32);
          const int k = BITS * n / 32;
#pragma unroll
          for (int q = 0; q < BITS; ++q) {
            const uint32_t f = q == k ? (uint32_t)field : q == k + 1 ? (uint32_t)(field >> 32) : 0u;
            words[q] = (words[q] & ~f) | ((q == k ? (uint32_t)u : (uint32_t)(u >> 32)) & f);
          }
        }
        if (live) mine &= mine - 1;
      }
    };
    if constexpr (FILTER) {
      bool exact = slow || direct > 0;
      direct = direct > 0 ? direct - 1 : 0;
      // (uniform) no rank term in this row block: its sums are zeros, and W0 and the stated quotient leave nothing undecided
      const bool no_term = CHECKED && (ACH == 0 || top_a == 0.f || __builtin_amdgcn_ballot_w64(bany != 0) == 0);
      // within tol of a tie the near sum does not settle the code (see the top of the file)
      const float tol = fmaf(rc, fmaf(top_a * half_sum(bsum), sum_tol, 0x1p-22f * fabsf(b)), 0x1p-21f * (1.f - d.qn));
      const float edge = 0.5f - tol;
      if constexpr (CHECKED && REST) {
        // more than 2 weights of a row block within reach (2 tol of its 2048) take longer, one after the other, than its stated sums:
        // the rest of the run goes there (8 bits, 4096 x 4096, packing / forward at rank 256 161 / 168 us without, chain 90 / 98; at
        // rank 128, 1.6 a row block, 51 / 51 without, chain 52 / 58)
        if (r > 16 * ACH && !exact && !no_term && __builtin_popcountll(__builtin_amdgcn_ballot_w64(tol > 0x1.2p-11f)) >= 32) {
          exact = true;
          direct = 1 << 30;
        }
      }
      if constexpr (CHECKED) {
        if (!exact && no_term) stream_columns(std::integral_constant<int, 3>{});
      }
      if constexpr (ACH > 0) {
        if (!exact && !no_term) stream_columns(std::integral_constant<int, 2>{});
      }
      if constexpr (MODE == 4) {
        eq *= s;
        ec *= s;
        // a quotient has overflowed, W / s or b / s alone, where the errors themselves need not: the stated form
        if (!exact) exact = __builtin_amdgcn_ballot_w64(row_ok & col_ok & !(eq + ec < __builtin_huge_valf())) != 0;
      }
      if constexpr (CHECKED && ACH > 0) {
        const bool unsettled = row_ok & col_ok & !(fmaxf(fmaxf(off[0], off[1]), fmaxf(off[2], off[3])) < edge);
        if (!exact && !no_term && __builtin_amdgcn_ballot_w64(unsettled) != 0)
          direct = __builtin_amdgcn_ballot_w64(unsettled && !(edge > 0.f)) != 0 || !settle(unsettled, edge) ? 3 : 0;
        exact |= direct == 3;  // (set just now)
      }
      if (exact) {
        if constexpr (ACH > 0) {
#pragma unroll
          for (int e = 0; e < 32; ++e) sum[e] = 0.f;
          chain_rest(sum, p, row_ok, 0);
        }
        eq = ec = 0.f;
        if (!slow) stream_columns(std::integral_constant<int, 1>{});
        else stream_columns(std::integral_constant<int, 0>{});
      }
    } else {
      if (!slow) stream_columns(std::integral_constant<int, 1>{});
      else stream_columns(std::integral_constant<int, 0>{});
    }

    if constexpr (MODE == 1) {
      // ---- Wq in blocks of 32 columns, [j / 32][p][j % 32]: a half-wave's tile is 2 KiB of consecutive addresses; through
      //      LDS, so that a store instruction covers 1 KiB (64 bytes per lane straight from the registers: 16-byte pieces
      //      of lines, which took a bare copy from 29 to 35 us)
      lds_order();
      const __amdgpu_buffer_rsrc_t rsOut = __builtin_amdgcn_make_buffer_rsrc(out.wq, 0, o * i * 2, 0x00020000);
      const int sr = lane >> 2, sc = lane & 3;  // instruction t: rows 16 (t % 2) + sr of column block t / 2
      const uint32_t out_base = (uint32_t)(wave * ms_wave_lds<MODE>() + sr * 128 + ((sc ^ (sr & 7)) << 4));
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 16 * (t & 1) + sr;
        const u32x4 v = lds16((out_base ^ (64 * (t >> 1))) + 2048 * (t & 1));
        const bool ok = p0 + row < o && jw + 32 * (t >> 1) < i;
        const unsigned vo = ok ? (unsigned)((((jw >> 5) + (t >> 1)) * o + p0 + row) * 64 + sc * 16) : OOB;
        __builtin_amdgcn_raw_buffer_store_b128(v, rsOut, (int)vo, 0, 0);
      }
      lds_order();
    }
    if constexpr (MODE == 2) {
      // ---- the factor as it came, Wq^T in blocks of 32 rows, [p / 32][j][p % 32]: 64 columns are 4 KiB of consecutive
      //      addresses.  The transposing read gives 16 lanes a column each of 4 rows (see l4q_gemm_core.h).
      lds_order();
      if (FACTOR && out.fgrad) {
        const __amdgpu_buffer_rsrc_t rsF = __builtin_amdgcn_make_buffer_rsrc(out.fgrad, 0, o * i * 2, 0x00020000);
        const unsigned vf = mcol_ok ? (unsigned)(((p0 + mr) * i + jw + 8 * mc) * 2) : OOB;
#pragma unroll
        for (int t = 0; t < 4; ++t)  // (rows from o on: past the end of the buffer)
          __builtin_amdgcn_raw_buffer_store_b128(lds16(mem_base + 4096 + 1024 * t), rsF,
                                                 (int)(vf + (unsigned)(t * 16 * i)), 0, 0);
      }
      typedef short s16x4_t __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_ptr_t;
      const int ld = (int)out.ld_wqT;
      const __amdgpu_buffer_rsrc_t rsT = __builtin_amdgcn_make_buffer_rsrc(out.wqT, 0, i * ld * 2, 0x00020000);
      const int tg = lane >> 4, tj = lane & 15;  // rows 8 tg .. 8 tg + 7, column 16 t + tj
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        u32x2 v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int rowm = 4 * u + (tj >> 2);  // row % 8
          unsigned char* q = tile + (8 * tg + rowm) * 128 + (((2 * t + ((tj >> 1) & 1)) ^ rowm) << 4) + (tj & 1) * 8;
          v[u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr_t)q));
        }
        const bool ok = jw + 16 * t < i;  // (uniform)
        const unsigned vo = ok ? (unsigned)(((rb * i + jw + 16 * t + tj) * 32 + 8 * tg) * 2) : OOB;
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{v[0][0], v[0][1], v[1][0], v[1][1]}, rsT, (int)vo, 0, 0);
      }
      lds_order();
    }
    if constexpr (MODE == 3) {
      const unsigned at = row_ok && col_ok ? (unsigned)(p * i + jl) : OOB;
      const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(out.codes, 0, o * i, 0x00020000);
      const __amdgpu_buffer_rsrc_t rsMask = __builtin_amdgcn_make_buffer_rsrc(out.mask, 0, o * i, 0x00020000);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (out.codes) __builtin_amdgcn_raw_buffer_store_b128(code8[q], rsC, (int)(at + 16u * q), 0, 0);
        if (out.mask) __builtin_amdgcn_raw_buffer_store_b128(mask8[q], rsMask, (int)(at + 16u * q), 0, 0);
      }
      if (out.wcomb) {
        const __amdgpu_buffer_rsrc_t rsWc = __builtin_amdgcn_make_buffer_rsrc(out.wcomb, 0, o * i * 4, 0x00020000);
        lds_order();
        const int sr = lane >> 4, sc = lane & 15;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int row = 4 * t + sr;
          const u32x4 v = *reinterpret_cast<const u32x4*>(tile + row * 256 + ((sc ^ (row & 15)) << 4));
          const unsigned vo = p0 + row < o && jw + 4 * sc < i ? (unsigned)(((p0 + row) * i + jw + 4 * sc) * 4) : OOB;
          __builtin_amdgcn_raw_buffer_store_b128(v, rsWc, (int)vo, 0, 0);
        }
      }
      lds_order();
    }
    if constexpr (MODE == 4) {
      err_q += row_ok && col_ok ? (double)eq : 0.0;
      err_c += row_ok && col_ok ? (double)ec : 0.0;
    }
    if constexpr (MODE == 5) {
      // ---- extremes over the half-waves (groups above 32), then over the wavefronts that share a group: through LDS, two
      //      sets in turn, so that one barrier per row block is enough
      if (g > 32) {
        const float2 l = both_halves(lo), t = both_halves(top);
        lo = fminf(l.x, l.y);
        top = fmaxf(t.x, t.y);
      }
      const int span = g > 64 ? g / 64 : 1;  // wavefronts of a group; its first one finishes it
      if (g > 64) {
        const int set = 4096 + 256 * ((rb - rb_begin) & 1);
        if (h == 0) *reinterpret_cast<float2*>(tile + set + 8 * l32) = make_float2(lo, top);
        __syncthreads();
        if (wave % span == 0) {
          for (int q = 1; q < span; ++q) {
            const float2 t = *reinterpret_cast<const float2*>(tile + q * ms_wave_lds<MODE>() + set + 8 * l32);
            lo = fminf(lo, t.x);
            top = fmaxf(top, t.y);
          }
        }
      }
      if (wave % span == 0 && row_ok && col_ok && (g == 32 || h == 0)) {
        // (a group of nothing but NaN has the extremes of an empty one, as in the general pass)
        float s0, b0 = 0.f;
        if (out.init_method == 0) {         // asymmetric min / max
          s0 = __fdiv_rn(top - lo, d.qp - d.qn);
          b0 = lo - s0 * d.qn;
        } else if (out.init_method == 1) {  // symmetric
          s0 = __fdiv_rn(fmaxf(fabsf(lo), fabsf(top)), -d.qn);
        } else {                            // L4Q_init (Eq. l4q_quant_init)
          s0 = fmaxf(fabsf(__fdiv_rn(lo, d.qn)), fabsf(__fdiv_rn(top, d.qp)));
        }
        out.init_scale[(int64_t)p * G + qtab] = s0;
        out.init_zero[(int64_t)p * G + qtab] = b0;
      }
      lds_order();
    }
    if constexpr (MODE == 6) {
      const int pack_row = BITS * (i / 32) * 4;  // bytes of a packed row
      const __amdgpu_buffer_rsrc_t rsPack = __builtin_amdgcn_make_buffer_rsrc(out.packed, 0, o * pack_row, 0x00020000);
      const unsigned vo = row_ok && col_ok ? (unsigned)(p * pack_row + (jl >> 5) * (4 * BITS)) : OOB;
      constexpr int QUADS = BITS / 4;
#pragma unroll
      for (int q = 0; q < QUADS; ++q)
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{words[4 * q], words[4 * q + 1], words[4 * q + 2], words[4 * q + 3]}, rsPack,
                                               (int)(vo + 16u * q), 0, 0);
      if constexpr (BITS % 4 == 1)
        __builtin_amdgcn_raw_buffer_store_b32(words[4 * QUADS], rsPack, (int)(vo + 16u * QUADS), 0, 0);
      if constexpr (BITS % 4 == 2)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{words[4 * QUADS], words[4 * QUADS + 1]}, rsPack, (int)(vo + 16u * QUADS), 0, 0);
      if constexpr (BITS % 4 == 3)
        __builtin_amdgcn_raw_buffer_store_b96(u32x3{words[4 * QUADS], words[4 * QUADS + 1], words[4 * QUADS + 2]}, rsPack,
                                              (int)(vo + 16u * QUADS), 0, 0);
      lds_order();
    }
    if constexpr (MODE == 4) lds_order();
  } while (++rb < rb_end);
  if constexpr (MODE == 4) {
    for (int off = 32; off > 0; off >>= 1) {
      err_q += __shfl_xor(err_q, off, 64);
      err_c += __shfl_xor(err_c, off, 64);
    }
    if (lane == 0) {
      err_out[0] = (float)err_q;
      err_out[1] = (float)err_c;
    }
  }
#endif
}

template <int ACH>
__global__ __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(ms_waves<1, ACH>(), ms_waves<1, ACH>())))
void merge_quant_stream_fwd_kernel(LayerDims d, const bf16_t* __restrict__ W0, const bf16_t* __restrict__ A,
                                   const bf16_t* __restrict__ B, const float* __restrict__ scale,
                                   const float* __restrict__ zero, MergeQuantOut<bf16_t> out, int nrb) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_all[ms_lds<1>()];
  merge_quant_stream_body<1, false, ACH>(d, W0, A, B, scale, zero, out, nrb, lds_all);
}
template <bool GAMMA_POW2, int ACH>
__global__ __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(ms_waves<2, ACH>(), ms_waves<2, ACH>())))
void merge_quant_stream_bwd_kernel(LayerDims d, const bf16_t* __restrict__ W0, const bf16_t* __restrict__ A,
                                   const bf16_t* __restrict__ B, const float* __restrict__ scale,
                                   const float* __restrict__ zero, MergeQuantOut<bf16_t> out, int nrb) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_all[ms_lds<2>()];
  merge_quant_stream_body<2, GAMMA_POW2, ACH>(d, W0, A, B, scale, zero, out, nrb, lds_all);
}
// MODE 3 .. 6: the export, statistics and packing forms
template <bool GAMMA_POW2, int MODE, int BITS = 0>
__global__ __launch_bounds__(MS_THREADS) __attribute__((amdgpu_waves_per_eu(ms_waves<MODE, 1>(), ms_waves<MODE, 1>())))
void merge_quant_stream_export_kernel(LayerDims d, const bf16_t* __restrict__ W0, const bf16_t* __restrict__ A,
                                      const bf16_t* __restrict__ B, const float* __restrict__ scale,
                                      const float* __restrict__ zero, MergeQuantOut<bf16_t> out, int nrb) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_all[ms_lds<MODE>()];
  merge_quant_stream_body<MODE, GAMMA_POW2, 1, BITS>(d, W0, A, B, scale, zero, out, nrb, lds_all);
}

// ------------------------------------------------------------------ check of the reciprocal-based quotient
// For significand m of s (bits 0 .. 22) and three exponents, compares exact_reciprocal(s) with the IEEE 1 / s and
// fast_quotient with the IEEE x / s for x = s t pushed -5 .. +5 units in the last place, t every rounding tie k + 1/2
// (-128 <= k < 128) and every grid end of 2 .. 8 bits.  counts[0] += wrong reciprocals, counts[1] += wrong quotients,
// counts[2] += quotients compared.
__global__ __launch_bounds__(256) void check_fast_divide_kernel(uint32_t first, uint32_t count,
                                                                unsigned long long* __restrict__ counts) {
  const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
  unsigned long long bad_r = 0, bad_q = 0, n = 0;
  if (idx < count) {
    const uint32_t m = (first + idx) & 0x7FFFFFu;
    const int expos[3] = {127 - 9, 127, 127 + 6};
    for (int ei = 0; ei < 3; ++ei) {
      const float s = __uint_as_float(((uint32_t)expos[ei] << 23) | m);
      const float rc = exact_reciprocal(s);
      if (__float_as_uint(rc) != __float_as_uint(__fdiv_rn(1.f, s))) ++bad_r;
      const float hi = s * 1024.f;
      for (int t2 = -256; t2 < 256 + 14; ++t2) {
        float t;
        if (t2 < 256) {
          if ((t2 & 1) == 0) continue;  // odd halves: k + 1/2
          t = 0.5f * (float)t2;
        } else {
          const int n2 = 2 + (t2 - 256) / 2;
          t = (t2 - 256) & 1 ? (float)((1 << (n2 - 1)) - 1) : -(float)(1 << (n2 - 1));
        }
        const float x0 = s * t;
        for (int u = -5; u <= 5; ++u) {
          const float x = __uint_as_float(__float_as_uint(x0) + (uint32_t)u);  // sign-magnitude: +-u ulps in magnitude
          const float want = __fdiv_rn(x, s);
          const float got = fast_quotient(x, s, rc, hi);
          if (__float_as_uint(want) != __float_as_uint(got)) ++bad_q;
          ++n;
        }
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    bad_r += __shfl_xor(bad_r, off, 64);
    bad_q += __shfl_xor(bad_q, off, 64);
    n += __shfl_xor(n, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&counts[0], bad_r);
    atomicAdd(&counts[1], bad_q);
    atomicAdd(&counts[2], n);
  }
}

}  // namespace

bool merge_quant_stream_supported(const LayerDims& d, const MergeQuantOut<bf16_t>& out) {
  const bool misc = out.codes || out.wcomb || out.mask;
  const bool fwd = out.wq && !out.wqT && !out.fgrad && !misc;
  const bool bwd = !out.wq && out.wqT && !misc;
  const bool exp = !out.wq && !out.wqT && !out.fgrad && misc;
  // A and B are addressed with byte offsets below 2^31 (W0 and the outputs stay below 2^30 by the library's size limits,
  // but a factor of rank 256 next to a few rows or columns does not)
  if ((d.i > d.o ? d.i : d.o) * d.r * 2 >= (1ll << 31)) return false;
  if (out.packed || out.errors || out.init_scale)  // each of them alone
    return d.r % 8 == 0 && d.g >= 32 && (!out.packed || d.i % 32 == 0) && (!out.init_scale || d.g <= 256);
  if (d.r == 0 && out.fgrad) return false;  // (the instance without a rank term takes no factor)
  const bool blocks = (!out.wq || out.ld_wq % 32 == 0) && (!out.wqT || out.ld_wqT % 32 == 0);
  return (fwd || bwd || exp) && blocks && d.r % 8 == 0 && d.g >= 32;
}

int64_t launch_merge_quant_stream(const LayerDims& d, const bf16_t* W0, const bf16_t* A, const bf16_t* B,
                                  const float* scale, const float* zero, const MergeQuantOut<bf16_t>& out,
                                  hipStream_t stream) {
  const int mode = out.wq ? 1 : out.wqT ? 2 : out.errors ? 4 : out.init_scale ? 5 : out.packed ? 6 : 3;
  const int64_t rows = mode == 2 && out.ld_wqT > d.o ? out.ld_wqT : d.o;
  const int nrb = (int)((rows + 31) / 32);
  const int strips = (int)((d.i + MS_COLS - 1) / MS_COLS);
  const bool wide = d.r > 16 && (mode == 1 || mode == 2);
  const int waves = mode == 1 ? (d.r == 0 ? ms_waves<1, 0>() : wide ? ms_waves<1, 4>() : ms_waves<1, 1>())
                  : mode == 2 ? (d.r == 0 ? ms_waves<2, 0>() : ms_waves<2, 1>())
                  : mode == 4 ? ms_waves<4, 1>() : mode == 5 ? ms_waves<5, 1>() : mode == 6 ? ms_waves<6, 1>() : ms_waves<3, 1>();
  int parts = waves * device_compute_units() / strips;
  // (two or four times as many, shorter runs, each with its own fetch of A: forward and packing 2 .. 17 % slower, backward the
  // same at 11008 x 4096, 22 -> 25 us at 4096 x 4096)
  if (parts < 1) parts = 1;
  if (parts > nrb) parts = nrb;
  dim3 grid((unsigned)(strips * parts));
  // gamma acc is exact when gamma is a power of two >= 1 (no underflow of the product)
  const uint32_t gb = __builtin_bit_cast(uint32_t, d.gamma);
  const bool pow2 = (gb & 0x807FFFFFu) == 0 && d.gamma >= 1.f && d.gamma <= 1048576.f;
#define L4Q_MS_LAUNCH(K, ...) \
  hipLaunchKernelGGL((K<__VA_ARGS__>), grid, dim3(MS_THREADS), 0, stream, d, W0, A, B, scale, zero, out, nrb)
#define L4Q_MS_POW2(K, ...) do { if (pow2) L4Q_MS_LAUNCH(K, true, __VA_ARGS__); else L4Q_MS_LAUNCH(K, false, __VA_ARGS__); } while (0)
#define L4Q_MS_PACK(BITS) L4Q_MS_LAUNCH(merge_quant_stream_export_kernel, false, 6, BITS)
  if (mode == 1 && d.r == 0) L4Q_MS_LAUNCH(merge_quant_stream_fwd_kernel, 0);  // (r = 0: the QAT-LoRA layer's passes)
  else if (mode == 1 && wide) L4Q_MS_LAUNCH(merge_quant_stream_fwd_kernel, 4);
  else if (mode == 1) L4Q_MS_LAUNCH(merge_quant_stream_fwd_kernel, 1);
  else if (mode == 2 && d.r == 0) L4Q_MS_LAUNCH(merge_quant_stream_bwd_kernel, false, 0);
  else if (mode == 2 && wide) L4Q_MS_POW2(merge_quant_stream_bwd_kernel, 4);
  else if (mode == 2) L4Q_MS_POW2(merge_quant_stream_bwd_kernel, 1);
  else if (mode == 3) L4Q_MS_POW2(merge_quant_stream_export_kernel, 3);
  else if (mode == 4) L4Q_MS_LAUNCH(merge_quant_stream_export_kernel, false, 4);
  else if (mode == 5) L4Q_MS_POW2(merge_quant_stream_export_kernel, 5);
  else if (d.bits == 2) L4Q_MS_PACK(2);
  else if (d.bits == 3) L4Q_MS_PACK(3);
  else if (d.bits == 4) L4Q_MS_PACK(4);
  else if (d.bits == 5) L4Q_MS_PACK(5);
  else if (d.bits == 6) L4Q_MS_PACK(6);
  else if (d.bits == 7) L4Q_MS_PACK(7);
  else L4Q_MS_PACK(8);
#undef L4Q_MS_PACK
#undef L4Q_MS_POW2
#undef L4Q_MS_LAUNCH
  return (int64_t)strips * parts * 4;
}

void launch_check_fast_divide(uint32_t first, uint32_t count, unsigned long long* counts, hipStream_t stream) {
  hipLaunchKernelGGL(check_fast_divide_kernel, dim3((count + 255u) / 256u), dim3(256), 0, stream, first, count, counts);
}

}  // namespace l4q

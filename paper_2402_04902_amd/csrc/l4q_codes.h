// Packed integer codes -> bfloat16 matrix operands, shared by the kernels of the fully quantized layer.
#pragma once

#include "l4q_device.h"
#include "l4q_gemm_core.h"

namespace l4q {

typedef gemm::bf16x8_t bf16x8_t;

// Operand fragment f (8 consecutive codes) of a 16-byte chunk of packed codes, as bf16 values without a convert.
// 4 bits: byte r holds codes 2r (low nibble) and 2r + 1; times 0x1001 puts a copy of the byte 12 bits up, so one mask
// leaves code 2r in bits 0..3 and code 2r + 1 in bits 16..19, and OR-ing 0x4300 into both halves makes the bf16 pair
// 128 + u (the caller's K0 takes the 128 and the code offset out again).  8 bits: code - 128, converted.
typedef uint32_t code_chunk_t __attribute__((ext_vector_type(4)));
template <int BITS>
__device__ __forceinline__ bf16x8_t code_fragment(const code_chunk_t& w, int f) {
  code_chunk_t d;
  if (BITS == 4) {
    const uint32_t v = w[f];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t spread = __builtin_amdgcn_ubfe(v, 8 * r, 8) * 0x1001u;
      // ((x & mask) | bias as one v_and_or_b32: the constants are made opaque so that they stay in registers - the op
      // takes no literals; the op itself is left to the compiler: as inline assembly it would hide that a vector op wrote
      // the register, and the wait states a matrix op needs before it reads such a register would be missing)
      uint32_t mask = 0x000F000Fu, bias = 0x43004300u;
      asm("" : "+s"(mask));
      asm("" : "+v"(bias));
      d[r] = (spread & mask) | bias;
    }
  } else if (BITS == 2) {
    // the chunk's first two dwords hold 32 codes; fragment f is the 16-bit half f % 2 of dword f / 2, its code pairs are
    // 4-bit fields: times 0x4001 puts a copy 14 bits up, the mask leaves code 2r in bits 0..1 and code 2r + 1 in bits
    // 16..17 (the caller's K0 is 128 + 2)
    const uint32_t v = w[f >> 1];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t spread = __builtin_amdgcn_ubfe(v, 16 * (f & 1) + 4 * r, 4) * 0x4001u;
      d[r] = (spread & 0x00030003u) | 0x43004300u;
    }
  } else if (BITS == 3) {
    // the chunk's first three dwords hold 32 codes; fragment f is the 24-bit window from bit 24 f, its code pairs are
    // 6-bit fields: times 0x2001 puts a copy 13 bits up, the mask leaves code 2r in bits 0..2 and code 2r + 1 in bits
    // 16..18 (the caller's K0 is 128 + 4)
    const uint32_t win = f == 0 ? w[0] : f == 1 ? (w[0] >> 24) | (w[1] << 8) : f == 2 ? (w[1] >> 16) | (w[2] << 16) : w[2] >> 8;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t spread = __builtin_amdgcn_ubfe(win, 6 * r, 6) * 0x2001u;
      d[r] = (spread & 0x00070007u) | 0x43004300u;
    }
  } else {
    // (u - 128 is the signed byte u ^ 0x80; its binary32 value has its significant bits in the upper half: exact)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t v = w[(2 * f + h) & 3] ^ 0x80808080u;  // 4 codes
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const uint32_t lo = __float_as_uint((float)(int8_t)(v >> (16 * r)));
        const uint32_t hi = __float_as_uint((float)(int8_t)(v >> (16 * r + 8)));
        d[2 * h + r] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
      }
    }
  }
  return __builtin_bit_cast(bf16x8_t, d);
}

}  // namespace l4q

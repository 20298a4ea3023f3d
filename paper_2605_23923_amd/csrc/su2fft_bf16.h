// Split-BF16 operands and products, shared by the BF16x3 contraction kernels.
//
// Instruction: V_MFMA_F32_16X16X32_BF16, A 16x32, B 32x16, lane l holding
// A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16], i = 0..7, and
// the accumulator D[4 (l / 16) + r][l % 16] (all measured).
//
// Tables (hi in the low 16 bits, lo in the high 16 bits of a 32-bit word):
//   forward: [tile][k / 8][column j = coff + i][k % 8]  (a lane's 8 nodes are
//            one aligned 32-byte load), rows k >= N zero;
//   inverse: the tile-major [tile][k][lsum] layout of the other paths.
#pragma once

#include "su2fft_mfma.h"

namespace su2 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ unsigned short bf16_rne_bits(float f) {
  unsigned int u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

__device__ __forceinline__ floatx4 mfma_bf16(u16x8 a, u16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                  0);
}

// split eight FP32 values into their bf16 hi and lo parts
__device__ __forceinline__ void split8(const float* v, u16x8& hi, u16x8& lo) {
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const unsigned short h = bf16_rne_bits(v[i]);
    hi[i] = h;
    lo[i] = bf16_rne_bits(v[i] - bf16_bits_to_f32(h));
  }
}

// four table words in one 16-byte load, at any word's alignment
typedef unsigned word4 __attribute__((ext_vector_type(4), aligned(4)));

// eight table words -> hi and lo operands
__device__ __forceinline__ void unpack8(const unsigned* w, u16x8& hi, u16x8& lo) {
#pragma unroll
  for (int i = 0; i < 8; i++) {
    hi[i] = (unsigned short)(w[i] & 0xffffu);
    lo[i] = (unsigned short)(w[i] >> 16);
  }
}
__device__ __forceinline__ void unpack8(const word4 (&w)[2], u16x8& hi, u16x8& lo) {
  const unsigned a[8] = {w[0].x, w[0].y, w[0].z, w[0].w, w[1].x, w[1].y, w[1].z, w[1].w};
  unpack8(a, hi, lo);
}

}  // namespace su2

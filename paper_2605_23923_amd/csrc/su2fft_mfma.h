// Matrix-core primitives shared by the contraction kernels.
//
// Operand layout per 64-lane wave of V_MFMA_F32_16X16X4_F32 /
// V_MFMA_F64_16X16X4_F64 (16x4 by 4x16 blocks): A[i][kk] in lane i + 16 kk,
// B[kk][j] in lane j + 16 kk.  Accumulator element r of lane (j + 16 g) is
// D[4 g + r][j] for the FP32 instruction and D[g + 4 r][j] for the FP64 one
// (both measured).
#pragma once

#include "su2fft_internal.h"

namespace su2 {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

template <class T>
struct acc4;
template <>
struct acc4<float> {
  typedef floatx4 type;
};
template <>
struct acc4<double> {
  typedef doublex4 type;
};

__device__ __forceinline__ floatx4 mfma16x16x4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mfma16x16x4(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <class T>
__device__ __forceinline__ int acc_row(int lane, int r) {
  return sizeof(T) == 4 ? 4 * (lane >> 4) + r : (lane >> 4) + 4 * r;
}

// compute units of the current device (read once per process)
inline int device_cus() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    cus = (hipGetDevice(&dev) == hipSuccess &&
           hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
              ? n
              : 256;
  }
  return cus;
}

}  // namespace su2

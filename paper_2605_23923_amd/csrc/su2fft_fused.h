// The beta contractions for the smallest grids (N <= 16), inside the kernels
// that transform a whole signal per workgroup (su2fft_ring_radix.hip,
// su2fft_ring_fast.hip).  Below that size a call is two kernels of a few
// microseconds, most of it launch and cold-miss latency, and the products are
// so few that vector FMAs beat the matrix cores, whose columns one signal
// leaves empty.  The FMA chains run in the matrix cores' order (node by node,
// degree by degree), whose 16x16x4 FP32 and FP64 products round like
// sequential FMAs (measured on random operands), so the results keep the bits
// of the two-kernel path.
#pragma once

#include "su2fft_internal.h"

namespace su2 {

// Sl: the signal's ring spectra in LDS, [tile][node][PT].  One coefficient per
// thread and step (loading the first step's column before the rings measured
// no gain).
template <class T, int N, int NT>
__device__ __forceinline__ void fused_contract_forward(const cpx<T>* Sl, cpx<T>* __restrict__ out,
                                                       const BetaParams<T>& p, int t) {
  constexpr int LM = (N / 2 + 1) / 2;  // degrees of the longest pair
  for (int idx = t; idx < p.ntiles * PT * LM; idx += NT) {
    const int pos = idx / LM, j = idx % LM;
    const PairInfo q = p.pairs[pos];
    if (j >= q.L) continue;
    const T* d = p.tab + q.tab + q.coff + j;
    const cpx<T>* s = Sl + pos / PT * N * PT + pos % PT;
    T a[N];
#pragma unroll
    for (int k = 0; k < N; k++) a[k] = d[k * q.lsum];
    cpx<T> v = {T(0), T(0)};
#pragma unroll
    for (int k = 0; k < N; k++) {
      const cpx<T> x = s[k * PT];
      v.re = __builtin_elementwise_fma(a[k], x.re, v.re);
      v.im = __builtin_elementwise_fma(a[k], x.im, v.im);
    }
    const T ts = p.table_signs && q.tsign < 0 ? T(-1) : T(1);
    out[coef_index_of(p.so3, q.tl0 + 2 * j, q.tm, q.tn)] = {ts * v.re, ts * v.im};
  }
}

// Cl: the signal's coefficients in LDS; the spectra S'_k(m, n) into Sl.  A
// thread keeps its pair and takes every (NT / pairs)-th node.
template <class T, int N, int NT>
__device__ __forceinline__ void fused_contract_inverse(const cpx<T>* Cl, cpx<T>* Sl, const BetaParams<T>& p, int t) {
  constexpr int LM = (N / 2 + 1) / 2;
  const int np = p.ntiles * PT, groups = NT > np ? NT / np : 1;
  if (NT > np && t >= groups * np) return;
  for (int pos = t % np; pos < np; pos += NT) {
    const PairInfo q = p.pairs[pos];
    cpx<T> c[LM];
#pragma unroll
    for (int j = 0; j < LM; j++) {
      const int tl = q.tl0 + 2 * j;
      // (2l+1) or 1, times the sign of a mirror column of a stored table
      const T sc = (p.scale_mode == 0 ? T(tl + 1) : T(1)) * (p.table_signs && q.tsign < 0 ? T(-1) : T(1));
      const cpx<T> v = Cl[j < q.L ? coef_index_of(p.so3, tl, q.tm, q.tn) : 0];
      c[j] = j < q.L ? cpx<T>{v.re * sc, v.im * sc} : cpx<T>{T(0), T(0)};
    }
    for (int k = NT > np ? t / np : 0; k < N; k += groups) {
      const T* d = p.tab + q.tab + (long long)k * q.lsum + q.coff;
      cpx<T> v = {T(0), T(0)};
#pragma unroll
      for (int j = 0; j < LM; j++) {
        const T a = j < q.L ? d[j] : T(0);
        v.re = __builtin_elementwise_fma(a, c[j].re, v.re);
        v.im = __builtin_elementwise_fma(a, c[j].im, v.im);
      }
      Sl[(pos / PT * N + k) * PT + pos % PT] = v;
    }
  }
}

}  // namespace su2

// What the small-batch contraction kernels share (su2fft_beta_small.hip,
// su2fft_beta_bf16_small.hip): which pairs and signals a wave's 16 product
// columns hold, how its sums leave, and the counts their dispatch goes by.
#pragma once

#include "su2fft_mfma.h"

namespace su2 {

// column cc of a wave's products: which of its MIR pairs, which signal of the
// tile's BT, and re or im
template <int MIR>
struct SmallCols {
  static constexpr int BT = 8 / MIR;
  __device__ static __forceinline__ int mir(int cc) { return cc / (2 * BT); }
  __device__ static __forceinline__ int sig(int cc) { return cc % (2 * BT) / 2; }
};

// What the kernels need of the wave's pair at list position `at` and of its
// mirror, and the table column the products read: the pair's own, or its
// mirror's where the pair is a pad.
template <class T, int MIR>
struct SmallPairs {
  struct Pair {
    int tm, tn, tl0, L, tsign;
  };
  Pair q0, q1;
  int pos0, pos1, L, lsum;
  long long tab, itab;  // the column's block in the row-major tables; its first value in the inverse-layout one
  int coff;             // its column in the block
  __device__ __forceinline__ SmallPairs(const BetaParams<T>& p, int at) {
    pos0 = at;
    pos1 = MIR == 2 ? p.ntiles * PT - 1 - at : at;
    const PairInfo a = p.pairs[pos0], b = p.pairs[pos1];
    q0 = {a.tm, a.tn, a.tl0, a.L, a.tsign};
    q1 = {b.tm, b.tn, b.tl0, b.L, b.tsign};
    if (p.real && mirrored_pair(a.tm, a.tn)) q0.L = q1.L = 0;
    const bool own = q0.L > 0;
    // the self-mirror middle tile stores both columns of a couple (2m = 0: the
    // same values up to sign); reading the first, the second needs its sign
    if (MIR == 2 && own && b.towner) q1.tsign = (((b.tm - b.tn) / 2) & 1) ? -1 : 1;
    L = own ? q0.L : q1.L;
    lsum = own ? a.lsum : b.lsum;
    tab = own ? a.tab : b.tab;
    coff = own ? a.coff : b.coff;
    itab = own ? a.itab : b.itab;
  }
  __device__ __forceinline__ Pair pick(int mir) const {
    if (MIR == 1) return q0;
    return {mir ? q1.tm : q0.tm, mir ? q1.tn : q0.tn, mir ? q1.tl0 : q0.tl0, mir ? q1.L : q0.L,
            mir ? q1.tsign : q0.tsign};
  }
};

// one real of degree j's sum of pair q out to a coefficient vector (`out` at re
// or im of it); half-spectrum real plans also write the mirror
// (-1)^{m-n} conj(fhat) at (-m, -n)
template <class T, int MIR>
__device__ __forceinline__ void store_coef_small(T* __restrict__ out, const BetaParams<T>& p,
                                                 const typename SmallPairs<T, MIR>::Pair& q, int j, int im, T sum) {
  if (j >= q.L) return;
  const T v = (p.table_signs && q.tsign < 0 ? T(-1) : T(1)) * sum;
  out[2 * coef_index_of(p.so3, q.tl0 + 2 * j, q.tm, q.tn)] = v;
  if (MIR == 1 && p.real && (q.tm != 0 || q.tn != 0)) {
    const T sg = ((((q.tm - q.tn) / 2) & 1) ? T(-1) : T(1)) * (im ? T(-1) : T(1));
    out[2 * coef_index_of(p.so3, q.tl0 + 2 * j, -q.tm, -q.tn)] = sg * v;
  }
}

// one real of degree j's scaled coefficient of pair q as the inverse multiplies
// it (zero past the pair's degrees or the signals)
template <class T, int MIR>
__device__ __forceinline__ T load_coef_small(const T* __restrict__ c, const BetaParams<T>& p,
                                             const typename SmallPairs<T, MIR>::Pair& q, int j, int im, bool in) {
  const int tl = q.tl0 + 2 * j;
  const bool ok = in && j < q.L;
  T v = c[ok ? 2 * coef_index_of(p.so3, tl, q.tm, q.tn) : 0];
  if (MIR == 1 && p.real) {  // Hermitian part: (c_{mn} + (-1)^{m-n} conj(c_{-m,-n})) / 2
    const T sg = ((((q.tm - q.tn) / 2) & 1) ? T(-1) : T(1)) * (im ? T(-1) : T(1));
    v = T(0.5) * (v + sg * c[ok ? 2 * coef_index_of(p.so3, tl, -q.tm, -q.tn) : 0]);
  }
  // (2l+1) or 1, times the sign of a mirror column of a stored table
  const T sc = (p.scale_mode == 0 ? T(tl + 1) : T(1)) * (p.table_signs && q.tsign < 0 ? T(-1) : T(1));
  return ok ? v * sc : T(0);
}

// rows (node, signal) of PT pairs in the inverse's stage buffers
template <class T, int BT>
struct SmallStage {
  static constexpr int PB = 2 * PT + 2, NRS = BT * PB + 4;
};

// a staged block of 16 nodes out to S in 16-byte stores
template <class T, int MIR, int NT>
__device__ __forceinline__ void store_rows_small(cpx<T>* __restrict__ S, const BetaParams<T>& p, const T* stage, int tile,
                                                 int kb, int b0, int nb, int tid) {
  constexpr int BT = SmallCols<MIR>::BT;
  typedef SmallStage<T, BT> ST;
  constexpr int VC = 16 / (int)sizeof(cpx<T>), VPR = PT / VC;
  typedef T vec16 __attribute__((ext_vector_type(16 / sizeof(T))));
  const int mirs = MIR == 2 && p.ntiles - 1 - tile == tile ? 1 : MIR;  // a self-mirror tile once
  for (int v = tid; v < mirs * 16 * BT * VPR; v += NT) {
    const int pv = v % VPR, bb = v / VPR % BT, kk = v / (VPR * BT) % 16, h = v / (VPR * BT * 16);
    const int k = 16 * kb + kk;
    if (k >= p.N || bb >= nb) continue;
    const T* src = stage + (h * 16 + kk) * ST::NRS + bb * ST::PB + 2 * pv * VC;
    vec16 x;
#pragma unroll
    for (int e = 0; e < 2 * VC; e++) x[e] = src[e];
    const int t = h ? p.ntiles - 1 - tile : tile;
    *reinterpret_cast<vec16*>(S + (((size_t)t * p.N + k) * p.batch + b0 + bb) * PT + pv * VC) = x;
  }
}

// pairs of a wave: a pair and its mirror where the plan's list is
// point-symmetric and every pair carries spectra
template <class T>
inline bool small_mirrored(const BetaParams<T>& p) { return p.sym && !p.real; }

// pair tiles (with their mirrors) of a launch
template <class T>
inline long long small_units(const BetaParams<T>& p) {
  return small_mirrored(p) ? (p.ntiles + 1) / 2 : p.ntiles - p.tile0;
}
// enough tiles that workgroups of one tile each reach three of four CUs
template <class T>
inline bool small_fills(const BetaParams<T>& p) { return 4 * small_units(p) >= 3LL * device_cus(); }

// Inverse: 16-node blocks per workgroup (`have` tiles x signal groups to share out): the fewest
// block times, counting the coefficient gather at a workgroup's start as two,
// with two workgroups per CU at a time
inline int small_inverse_blocks(long long have, int NB) {
  const long long slots = 2LL * device_cus();
  int blocks = NB;
  long long best = 0;
  for (int b = NB; b >= 1; b--) {
    const long long nsplit = (NB + b - 1) / b, cost = (have * nsplit + slots - 1) / slots * (b + 2);
    if (b == NB || cost < best) {
      best = cost;
      blocks = b;
    }
  }
  return blocks;
}

}  // namespace su2

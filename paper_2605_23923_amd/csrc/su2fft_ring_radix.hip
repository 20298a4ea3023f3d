// Ring FFT (stage 1, Proposition 4.2 / Proposition 6.1) for every N = 2^a 3^b
// that the register-resident kernels (N = 16, 32, 64, 128) and the N = 256
// kernels do not take: N = 2, 4, 6, 8, 12, 18, 24, 36, 48, 54, 72, 96, 108,
// 144, 162, 192, 216.
//
// Forward, per ring (signal b, node k), with w = e^{+2 pi i / N}:
//   G[j, q]  = sum_l f[k, j, l] w^{q l}                    (gamma)
//   H[p, q]  = sum_j G[j, q] w^{(p + delta) j}             (alpha; delta = 1/2 on odd q,
//                                                           the half-integer n; 0 in SO(3) plans)
//   S_k(m,n) = W_k rho_{mn} H[p, q]
// and the inverse is the conjugate transpose network without W_k (or with it,
// the adjoint).
//
// A ring is cut in R slices, one workgroup each, so that a slice fits LDS: two or
// more per CU at most lengths, one (95-160 KB) at N = 192 and 216, at N = 144 in
// FP64, in the FP32 inverse and the FP64 forward at N = 108 and in the FP64 forward at
// N = 162.  The forward is cut by gamma frequency (slice s holds
// q = R q' + s; the first radix-R step of the gamma transform is taken while
// the samples are read), the inverse by output row (slice s holds
// j = R j' + s; the bins fold into an (N / R)-point alpha transform while the
// spectra are read).  Every slice reads the whole ring: the slices of one
// ring are numbered side by side on one XCD, so all but the first read it
// from that XCD's L2.
//
// Inside a slice each axis is one four-step transform of two in-register DFTs
// (length = A1 x A2, both at most 18).  The slice stays in LDS between the
// four phases, and every phase writes each of its DFTs back to the slots it
// read, so one barrier separates two phases and no second buffer is needed:
//   forward  1  load, radix-R step, radix-GB DFT over l2 (c = l1 + GA l2), twiddle
//            2  radix-GA DFT over l1 -> q' = q2 + GB q1 at column GA q2 + q1
//            3  half-bin shift, radix-AB DFT over j2 (j = j1 + AA j2), twiddle
//            4  radix-AA DFT over j1 -> p = p2 + AB p1 at row AA p2 + p1
//            5  the retained bins, phases and weights, to S in pair order
//   inverse  1  gather and fold the bins, radix-A2 DFT over b (p' = a + A1 b), twiddle
//            2  radix-A1 DFT over a -> j' = k2 + A2 k1 at row A1 k2 + k1, half-bin shift
//            3  radix-G2 DFT over g2 (q = g1 + G1 g2), twiddle
//            4  radix-G1 DFT over g1 -> l = u2 + G2 u1, to the samples
// Row pitches are odd (and the inverse's column groups of G1 are padded to
// odd length), so that lanes over consecutive rows meet distinct banks.
//
// What bounds it: HBM in principle, and the traffic is N^2 + P values per ring
// (counters: 1.01 times that at N = 54, 1.08 at N = 72, 1.00 at N = 192, whose
// slices read their ring again from L2).  Full batches take 1.0-1.5 times as long
// as a copy of those bytes at N = 24 to 48 and 1.5-1.7 at N = 54 to 96 (vector
// ALUs 58 % busy at N = 72); N = 192 and 216 take 2.3-2.9 times, one workgroup
// per CU, nothing covering its loads, steps and stores.  Ring stage alone, forward /
// inverse, against one-radix-per-pass kernels with run-time sizes before: N = 54
// FP64, 106 signals 291 / 293 -> 105 / 99 us; N = 72 FP32, 44 signals 140 / 142 ->
// 49 / 54 us; N = 96 FP32, 18 signals 93 / 83 -> 48 / 53 us; N = 192 FP32, 2 signals
// 278 / 280 -> 63 / 74 us; N = 216 FP64, 2 signals 799 / 968 -> 234 / 228 us.
#include <algorithm>

#include "su2fft_fused.h"

namespace su2 {

#define SU2_DEV __device__ __forceinline__

// Every multiply-add below is written out, and the compiler forms none of its
// own: which ones it picks depends on the code around them, and a length's rings
// have the same bits in its own launch, in a list beside other lengths and in the
// one-kernel calls.
#pragma clang fp contract(off)
template <class T>
SU2_DEV T fma_of(T a, T b, T c) { return __builtin_elementwise_fma(a, b, c); }
template <class T>
SU2_DEV cpx<T> mul(cpx<T> a, cpx<T> w) {
  return {fma_of(a.re, w.re, -(a.im * w.im)), fma_of(a.re, w.im, a.im * w.re)};
}
template <class T>
SU2_DEV cpx<T> mul_conj(cpx<T> a, cpx<T> w) {  // a conj(w)
  return {fma_of(a.re, w.re, a.im * w.im), fma_of(a.im, w.re, -(a.re * w.im))};
}
template <class T>
SU2_DEV cpx<T> mul_add(cpx<T> a, cpx<T> w, cpx<T> c) {  // a w + c
  return {fma_of(a.re, w.re, fma_of(-a.im, w.im, c.re)), fma_of(a.re, w.im, fma_of(a.im, w.re, c.im))};
}

// e^{2 pi i k / 288}, the first octant: every root that the DFTs and the
// half-bin shifts below need (lengths dividing 288) follows by symmetry
struct Octant {
  static constexpr double c[37] = {
      1.0, 0.9997620270799090923, 0.9990482215818577624, 0.99785892323860350674, 0.9961946980917455323,
      0.9940563382223196121, 0.99144486137381041114, 0.9883615104677607085, 0.98480775301220805937,
      0.98078528040323044913, 0.97629600711993336597, 0.97134206981326143451, 0.96592582628906828675,
      0.96004985438592867412, 0.95371695074822692114, 0.94693012949510566426, 0.93969262078590838405,
      0.93200786928279850264, 0.92387953251128675613, 0.91531147911944714241, 0.90630778703664996324,
      0.89687274153268830389, 0.88701083317822170105, 0.8767267557075077174, 0.86602540378443864676,
      0.85491187067294659555, 0.84339144581288570127, 0.83146961230254523708, 0.81915204428899178968,
      0.80644460426748256644, 0.79335334029123516458, 0.77988448309288180111, 0.7660444431189780352,
      0.75183980747897739641, 0.73727733681012404138, 0.72236396205975558059, 0.7071067811865475244};
  static constexpr double s[37] = {
      0.0, 0.021814885034561121843, 0.043619387365335999782, 0.065403129230143066815, 0.087155742747658173558,
      0.10886687485196457597, 0.13052619222005159155, 0.15212338618991670154, 0.17364817766693034885,
      0.19509032201612826785, 0.21643961393810287976, 0.23768589232617309353, 0.25881904510252076235,
      0.27982901403099205675, 0.30070579950427312162, 0.3214394653031615807, 0.34202014332566873304,
      0.36243803828370164506, 0.38268343236508977173, 0.40274668985873723482, 0.42261826174069943619,
      0.442288690219001282, 0.46174861323503393056, 0.48098876891938764278, 0.5, 0.51877325816052144952,
      0.53729960834682383184, 0.55557023301960222474, 0.57357643635104609611, 0.59130964836358237728,
      0.60876142900872063942, 0.62592347218405906344, 0.64278760968653932632, 0.65934581510006886843,
      0.67559020761566024435, 0.69151305578226937776, 0.7071067811865475244};
};
constexpr int root_step(int k, int n) {
  return ((k % n + n) % n) * (288 / n);
}
constexpr double root_re(int k, int n) {
  const int u = root_step(k, n);           // 0..287
  const int v = u > 144 ? 288 - u : u;     // cos is even
  const int w = v > 72 ? 144 - v : v;      // cos(pi - x) = -cos x
  const double r = w <= 36 ? Octant::c[w] : Octant::s[72 - w];
  return v > 72 ? -r : r;
}
constexpr double root_im(int k, int n) {
  const int u = root_step(k, n);
  const int v = u > 144 ? 288 - u : u;
  const int w = v > 72 ? 144 - v : v;
  const double r = w <= 36 ? Octant::s[w] : Octant::c[72 - w];
  return u > 144 ? -r : r;
}

// a e^{SIGN 2 pi i K / LEN} for compile-time K, LEN
template <class T, int K, int LEN, int SIGN>
SU2_DEV cpx<T> rot(cpx<T> a) {
  static_assert(288 % LEN == 0, "root table");
  constexpr int u = root_step(SIGN * K, LEN);
  if constexpr (u == 0) return a;
  else if constexpr (u == 72) return {-a.im, a.re};
  else if constexpr (u == 144) return {-a.re, -a.im};
  else if constexpr (u == 216) return {a.im, -a.re};
  else {
    constexpr T wr = T(root_re(SIGN * K, LEN)), wi = T(root_im(SIGN * K, LEN));
    return mul(a, cpx<T>{wr, wi});
  }
}

constexpr int inverse_mod(int a, int m) {
  for (int i = 1; i < m; i++)
    if (a * i % m == 1) return i;
  return 0;  // not coprime
}
// In-register DFT of length R: a[q] <- sum_n a[n] e^{SIGN 2 pi i q n / R}, by
// R = P Q.  Coprime P and Q (6 = 2 x 3, 12 = 4 x 3, 18 = 2 x 9) need no twiddles
// between them under the prime-factor index maps n = Q n1 + P n2 and
// q = EP k1 + EQ k2 (mod R; I. J. Good, 1958), which also saves their rounding:
// the rings' errors are 1-8 % smaller than with twiddles.
template <class T, int R, int SIGN>
struct Dft {
  static constexpr int P = R == 9 ? 3 : (R == 12 || R == 16 ? 4 : 2), Q = R / P;
  static constexpr int EP = Q * inverse_mod(Q % P, P), EQ = P * inverse_mod(P % Q, Q);
  static constexpr bool PRIME_FACTOR = EP != 0 && EQ != 0;
  template <int N1, int K2>
  SU2_DEV static void twiddle(cpx<T> (&y)[P][Q]) {
    if constexpr (N1 < P) {
      y[N1][K2] = rot<T, N1 * K2, R, SIGN>(y[N1][K2]);
      if constexpr (K2 + 1 < Q) twiddle<N1, K2 + 1>(y);
      else twiddle<N1 + 1, 1>(y);
    }
  }
  SU2_DEV static void run(cpx<T>* a) {
    cpx<T> y[P][Q];
#pragma unroll
    for (int n1 = 0; n1 < P; n1++) {
#pragma unroll
      for (int n2 = 0; n2 < Q; n2++) y[n1][n2] = a[PRIME_FACTOR ? (Q * n1 + P * n2) % R : P * n2 + n1];
      Dft<T, Q, SIGN>::run(y[n1]);
    }
    if constexpr (!PRIME_FACTOR) twiddle<1, 1>(y);
#pragma unroll
    for (int k2 = 0; k2 < Q; k2++) {
      cpx<T> z[P];
#pragma unroll
      for (int n1 = 0; n1 < P; n1++) z[n1] = y[n1][k2];
      Dft<T, P, SIGN>::run(z);
#pragma unroll
      for (int k1 = 0; k1 < P; k1++) a[PRIME_FACTOR ? (EP * k1 + EQ * k2) % R : k2 + Q * k1] = z[k1];
    }
  }
};
template <class T, int SIGN>
struct Dft<T, 1, SIGN> {
  SU2_DEV static void run(cpx<T>*) {}
};
template <class T, int SIGN>
struct Dft<T, 2, SIGN> {
  SU2_DEV static void run(cpx<T>* a) {
    const cpx<T> t = a[0];
    a[0] = cadd(t, a[1]);
    a[1] = csub(t, a[1]);
  }
};
template <class T, int SIGN>
struct Dft<T, 3, SIGN> {
  SU2_DEV static void run(cpx<T>* a) {
    constexpr T h = T(root_im(1, 3));
    const cpx<T> t1 = cadd(a[1], a[2]), t2 = csub(a[1], a[2]);
    const cpx<T> m = {fma_of(T(-0.5), t1.re, a[0].re), fma_of(T(-0.5), t1.im, a[0].im)};
    a[0] = cadd(a[0], t1);
    a[1] = {fma_of(-T(SIGN) * h, t2.im, m.re), fma_of(T(SIGN) * h, t2.re, m.im)};
    a[2] = {fma_of(T(SIGN) * h, t2.im, m.re), fma_of(-T(SIGN) * h, t2.re, m.im)};
  }
};
template <class T, int SIGN>
struct Dft<T, 4, SIGN> {
  SU2_DEV static void run(cpx<T>* a) {
    const cpx<T> s02 = cadd(a[0], a[2]), d02 = csub(a[0], a[2]);
    const cpx<T> s13 = cadd(a[1], a[3]), d13 = rot<T, 1, 4, SIGN>(csub(a[1], a[3]));
    a[0] = cadd(s02, s13);
    a[2] = csub(s02, s13);
    a[1] = cadd(d02, d13);
    a[3] = csub(d02, d13);
  }
};

// 8 = 2 x 4, the products with the eighth roots inside the last additions
template <class T, int SIGN>
struct Dft<T, 8, SIGN> {
  SU2_DEV static void run(cpx<T>* a) {
    constexpr T h = T(root_re(1, 8)), g = T(SIGN) * h;
    cpx<T> e[4] = {a[0], a[2], a[4], a[6]}, o[4] = {a[1], a[3], a[5], a[7]};
    Dft<T, 4, SIGN>::run(e);
    Dft<T, 4, SIGN>::run(o);
    o[2] = rot<T, 1, 4, SIGN>(o[2]);
    a[0] = cadd(e[0], o[0]);
    a[4] = csub(e[0], o[0]);
    a[2] = cadd(e[2], o[2]);
    a[6] = csub(e[2], o[2]);
    const T p = o[1].re - T(SIGN) * o[1].im, q = o[1].im + T(SIGN) * o[1].re;
    const T r = -o[3].re - T(SIGN) * o[3].im, t = -o[3].im + T(SIGN) * o[3].re;
    a[1] = {fma_of(h, p, e[1].re), fma_of(h, q, e[1].im)};
    a[5] = {fma_of(-h, p, e[1].re), fma_of(-h, q, e[1].im)};
    a[3] = {fma_of(h, r, e[3].re), fma_of(h, t, e[3].im)};
    a[7] = {fma_of(-h, r, e[3].re), fma_of(-h, t, e[3].im)};
  }
};

// a[j] *= e^{SIGN pi i j / LEN} where `odd`, j = 1 .. LEN - 1
template <class T, int LEN, int SIGN, int J = 1>
SU2_DEV void half_bins(cpx<T>* a, bool odd) {
  if constexpr (J < LEN) {
    constexpr T c = T(root_re(SIGN * J, 2 * LEN)), s = T(root_im(SIGN * J, 2 * LEN));
    const T wr = odd ? c : T(1), wi = odd ? s : T(0);
    a[J] = mul(a[J], cpx<T>{wr, wi});
    half_bins<T, LEN, SIGN, J + 1>(a, odd);
  }
}

// Shapes per N and type: R slices per ring (N / R = M), NTR threads per
// slice, RPW slices per workgroup; forward gamma M = GA GB and alpha N = AA AB;
// inverse alpha M = A1 A2 and gamma N = G1 G2.  From N = 24 up the shapes are the
// fastest of up to 24 per (N, type, direction) at 1 signal and at about 400 MB
// of samples (geometric mean): few slices (each reads the whole ring), enough
// threads that a phase is one to three instances per thread, and AA a
// multiple of 4 where the pruning of the last alpha DFT pays.  At N = 12, 24 and
// 36 they are the fastest of those whose rounding error is no larger than that of
// one radix per pass (N = 36 FP32, forward / inverse at 256 signals 34.7 / 33.7 ->
// 31.1 / 31.3 us with errors 5-8 % smaller; N = 12 costs up to 5 % of a call for
// 1-10 %).
template <int R_, int NTR_, int RPW_, int GA_, int GB_, int AA_, int AB_>
struct RadixFwd {
  static constexpr int R = R_, NTR = NTR_, RPW = RPW_, GA = GA_, GB = GB_, AA = AA_, AB = AB_;
};
template <int R_, int NTR_, int RPW_, int A1_, int A2_, int G1_, int G2_>
struct RadixInv {
  static constexpr int R = R_, NTR = NTR_, RPW = RPW_, A1 = A1_, A2 = A2_, G1 = G1_, G2 = G2_;
};
template <class T, int N, bool FWD>
struct RadixCfg;
template <class T> struct RadixCfg<T, 2, true> : RadixFwd<1, 16, 16, 2, 1, 2, 1> {};
template <class T> struct RadixCfg<T, 2, false> : RadixInv<1, 16, 16, 2, 1, 2, 1> {};
template <class T> struct RadixCfg<T, 4, true> : RadixFwd<1, 16, 16, 4, 1, 4, 1> {};
template <class T> struct RadixCfg<T, 4, false> : RadixInv<1, 16, 16, 4, 1, 4, 1> {};
template <class T> struct RadixCfg<T, 6, true> : RadixFwd<1, 32, 8, 3, 2, 3, 2> {};
template <class T> struct RadixCfg<T, 6, false> : RadixInv<1, 32, 8, 3, 2, 2, 3> {};
template <class T> struct RadixCfg<T, 8, true> : RadixFwd<1, 32, 8, 4, 2, 4, 2> {};
template <> struct RadixCfg<float, 8, false> : RadixInv<1, 32, 8, 4, 2, 8, 1> {};
template <> struct RadixCfg<double, 8, false> : RadixInv<1, 32, 8, 4, 2, 2, 4> {};
template <class T> struct RadixCfg<T, 12, true> : RadixFwd<1, 64, 4, 3, 4, 3, 4> {};
template <class T> struct RadixCfg<T, 12, false> : RadixInv<1, 64, 4, 4, 3, 4, 3> {};
template <class T> struct RadixCfg<T, 18, true> : RadixFwd<1, 64, 4, 6, 3, 6, 3> {};
template <class T> struct RadixCfg<T, 18, false> : RadixInv<1, 64, 4, 6, 3, 3, 6> {};
template <> struct RadixCfg<float, 24, true> : RadixFwd<1, 96, 1, 4, 6, 12, 2> {};
template <> struct RadixCfg<float, 24, false> : RadixInv<1, 96, 1, 4, 6, 3, 8> {};
template <> struct RadixCfg<float, 36, true> : RadixFwd<1, 192, 1, 3, 12, 12, 3> {};
template <> struct RadixCfg<float, 36, false> : RadixInv<1, 192, 1, 9, 4, 3, 12> {};
template <> struct RadixCfg<float, 48, true> : RadixFwd<1, 192, 1, 8, 6, 12, 4> {};
template <> struct RadixCfg<float, 48, false> : RadixInv<1, 192, 1, 12, 4, 3, 16> {};
template <> struct RadixCfg<float, 54, true> : RadixFwd<1, 256, 1, 9, 6, 9, 6> {};
template <> struct RadixCfg<float, 54, false> : RadixInv<1, 256, 1, 18, 3, 6, 9> {};
template <> struct RadixCfg<float, 72, true> : RadixFwd<1, 512, 1, 18, 4, 12, 6> {};
template <> struct RadixCfg<float, 72, false> : RadixInv<1, 512, 1, 12, 6, 6, 12> {};
template <> struct RadixCfg<float, 96, true> : RadixFwd<1, 768, 1, 12, 8, 12, 8> {};
template <> struct RadixCfg<float, 96, false> : RadixInv<2, 576, 1, 12, 4, 8, 12> {};
template <> struct RadixCfg<float, 108, true> : RadixFwd<2, 384, 1, 18, 3, 12, 9> {};
template <> struct RadixCfg<float, 108, false> : RadixInv<1, 1024, 1, 18, 6, 9, 12> {};
template <> struct RadixCfg<float, 144, true> : RadixFwd<3, 576, 1, 16, 3, 12, 12> {};
template <> struct RadixCfg<float, 144, false> : RadixInv<3, 576, 1, 12, 4, 12, 12> {};
template <> struct RadixCfg<float, 162, true> : RadixFwd<3, 512, 1, 18, 3, 18, 9> {};
template <> struct RadixCfg<float, 162, false> : RadixInv<3, 576, 1, 9, 6, 9, 18> {};
template <> struct RadixCfg<float, 192, true> : RadixFwd<2, 768, 1, 16, 6, 16, 12> {};
template <> struct RadixCfg<float, 192, false> : RadixInv<3, 1024, 1, 16, 4, 12, 16> {};
template <> struct RadixCfg<float, 216, true> : RadixFwd<3, 1024, 1, 18, 4, 12, 18> {};
template <> struct RadixCfg<float, 216, false> : RadixInv<3, 1024, 1, 18, 4, 18, 12> {};
template <> struct RadixCfg<double, 24, true> : RadixFwd<1, 96, 1, 4, 6, 12, 2> {};
template <> struct RadixCfg<double, 24, false> : RadixInv<1, 96, 1, 4, 6, 3, 8> {};
template <> struct RadixCfg<double, 36, true> : RadixFwd<1, 192, 1, 3, 12, 12, 3> {};
template <> struct RadixCfg<double, 36, false> : RadixInv<1, 192, 1, 9, 4, 3, 12> {};
template <> struct RadixCfg<double, 48, true> : RadixFwd<1, 384, 1, 8, 6, 8, 6> {};
template <> struct RadixCfg<double, 48, false> : RadixInv<1, 384, 1, 8, 6, 6, 8> {};
template <> struct RadixCfg<double, 54, true> : RadixFwd<1, 256, 1, 9, 6, 6, 9> {};
template <> struct RadixCfg<double, 54, false> : RadixInv<1, 256, 1, 18, 3, 3, 18> {};
template <> struct RadixCfg<double, 72, true> : RadixFwd<3, 256, 1, 8, 3, 8, 9> {};
template <> struct RadixCfg<double, 72, false> : RadixInv<2, 384, 1, 9, 4, 9, 8> {};
template <> struct RadixCfg<double, 96, true> : RadixFwd<2, 384, 1, 12, 4, 8, 12> {};
template <> struct RadixCfg<double, 96, false> : RadixInv<3, 384, 1, 8, 4, 12, 8> {};
template <> struct RadixCfg<double, 108, true> : RadixFwd<2, 512, 1, 18, 3, 12, 9> {};
template <> struct RadixCfg<double, 108, false> : RadixInv<3, 512, 1, 9, 4, 9, 12> {};
template <> struct RadixCfg<double, 144, true> : RadixFwd<3, 576, 1, 16, 3, 12, 12> {};
template <> struct RadixCfg<double, 144, false> : RadixInv<3, 768, 1, 12, 4, 12, 12> {};
template <> struct RadixCfg<double, 162, true> : RadixFwd<3, 512, 1, 18, 3, 18, 9> {};
template <> struct RadixCfg<double, 162, false> : RadixInv<6, 512, 1, 9, 3, 9, 18> {};
template <> struct RadixCfg<double, 192, true> : RadixFwd<4, 768, 1, 16, 3, 16, 12> {};
template <> struct RadixCfg<double, 192, false> : RadixInv<4, 768, 1, 8, 6, 16, 12> {};
template <> struct RadixCfg<double, 216, true> : RadixFwd<6, 768, 1, 12, 3, 12, 18> {};
template <> struct RadixCfg<double, 216, false> : RadixInv<6, 768, 1, 12, 3, 18, 12> {};

// Column q of the bin map (RadixRingParams::cols): retained bins are
// p = ps mod N for ps in [-nneg, npos); bin ps has pair hi + ps (ps < 0),
// zero (ps = 0) or lo + ps (ps > 0) and phase i^{e0 + 3 ps}.
struct RadixCol {
  int hi, zero, lo, nneg, npos, e0;
};
SU2_DEV RadixCol radix_col(const int4& w) {
  return {w.x, w.y, w.z, (w.w >> 2) & 127, (w.w >> 9) & 127, w.w & 3};
}
SU2_DEV int radix_pair(const RadixCol& c, int ps) { return ps < 0 ? c.hi + ps : (ps == 0 ? c.zero : c.lo + ps); }

// Samples are written once: non-temporal stores keep them from evicting the
// spectra (N = 96 FP32, 56 signals: inverse ring 257 -> 181 us).  The
// forward's sample reads are plain: runs of GA values share cache lines with
// their neighbours', and non-temporal reads measured 10-16 % slower.
template <class T>
SU2_DEV void nt_store(T* a, T v) { __builtin_nontemporal_store(v, a); }
template <class T>
SU2_DEV void nt_store(cpx<T>* a, cpx<T> v) {
  __builtin_nontemporal_store(v.re, &a->re);
  __builtin_nontemporal_store(v.im, &a->im);
}

// v i^e s
template <class T>
SU2_DEV cpx<T> ipow_times(cpx<T> v, int e, T s) {
  const T ss = (e & 2) ? -s : s;
  const T c = (e & 1) ? T(0) : ss, d = (e & 1) ? ss : T(0);
  return mul(v, cpx<T>{c, d});
}

// One slice s of one ring; t is the thread's index among the slice's NTR.
// buf: LDS values of the slice; tw: e^{i pi u / N}, u = 0 .. 2N - 1, in LDS;
// twg the same in device memory (uniform reads).
template <class C>
struct RadixThreads {
  static constexpr int NTR = C::NTR;
  static constexpr int iters(int total) { return (total + NTR - 1) / NTR; }
  SU2_DEV static bool in(int idx, int total) { return total % NTR == 0 || idx < total; }
};

template <class T, int N_, class C_>
struct RadixForward : RadixThreads<C_> {
  typedef C_ C;
  typedef RadixThreads<C> TH;
  using TH::in;
  using TH::iters;
  static constexpr int N = N_, R = C::R, M = N / R, NTR = C::NTR, B = N / 2;
  static constexpr int GA = C::GA, GB = C::GB, AA = C::AA, AB = C::AB;
  static_assert(GA * GB == M && AA * AB == N && R * M == N, "shape");
  static constexpr int FP = M | 1;  // row pitch
  static constexpr int LDS = N * FP;
  // rows p1 of the last alpha DFT that can hold retained bins (p < N/4 or
  // p >= 3N/4): known at compile time where 4 divides AA
  SU2_DEV static constexpr bool kept_p1(int p1) { return AA % 4 != 0 || p1 < AA / 4 || p1 >= 3 * AA / 4; }
  // instances of phase 1 whose loads are issued together
  static constexpr int BATCH1 = sizeof(T) == 4 ? 2 : 1;

  template <bool REAL>
  SU2_DEV static cpx<T> sample(const cpx<T>* x, int idx) {
    // (opaque_zero: the transforms round real samples exactly as complex
    // samples with a zero imaginary part)
    if constexpr (REAL) return {reinterpret_cast<const T*>(x)[idx], opaque_zero<T>()};
    else return x[idx];
  }

  // the samples of phase-1 instance (row j, l1), radix-R step taken:
  // y[c] w^{-s l1} for c = l1 + GA l2 with y[c] = w^{s c} sum_i x[c + i M] w^{s i M}
  template <bool REAL>
  SU2_DEV static void load1(const cpx<T>* x, const cpx<T>* twg, int s, int j, int l1, cpx<T> (&a)[GB]) {
#pragma unroll
    for (int l2 = 0; l2 < GB; l2++) {
      a[l2] = sample<REAL>(x, j * N + l1 + GA * l2);
      if constexpr (R > 1) {
        if (l2 > 0) a[l2] = mul(a[l2], twg[2 * ((s * GA * l2) % N)]);
#pragma unroll
        for (int i = 1; i < R; i++)
          a[l2] = mul_add(sample<REAL>(x, j * N + l1 + GA * l2 + i * M), twg[2 * ((s * (GA * l2 + i * M)) % N)], a[l2]);
      }
    }
  }

  template <bool REAL>
  SU2_DEV static void forward1_as(const cpx<T>* x, cpx<T>* buf, const cpx<T>* tw, const cpx<T>* twg, int s, int t) {
    constexpr int TOTAL = N * GA, IT = iters(TOTAL), U = IT < BATCH1 ? IT : BATCH1;
#pragma unroll 1
    for (int i0 = 0; i0 < IT; i0 += U) {
      cpx<T> a[U][GB];
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int idx = t + NTR * (i0 + u);
        if ((IT % U == 0 || i0 + u < IT) && in(idx, TOTAL)) load1<REAL>(x, twg, s, idx / GA, idx % GA, a[u]);
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int idx = t + NTR * (i0 + u);
        if (!((IT % U == 0 || i0 + u < IT) && in(idx, TOTAL))) continue;
        const int j = idx / GA, l1 = idx % GA;
        Dft<T, GB, 1>::run(a[u]);
#pragma unroll
        for (int q2 = 0; q2 < GB; q2++) {
          // w_M^{l1 q2} w_N^{l1 s}
          if (q2 > 0 || R > 1) a[u][q2] = mul(a[u][q2], tw[2 * l1 * (R * q2 + s)]);
          buf[j * FP + l1 + GA * q2] = a[u][q2];
        }
      }
    }
  }
  SU2_DEV static void forward1(const cpx<T>* x, cpx<T>* buf, const cpx<T>* tw, const cpx<T>* twg, int s, int real_io,
                              int t) {
    if (real_io) forward1_as<true>(x, buf, tw, twg, s, t);
    else forward1_as<false>(x, buf, tw, twg, s, t);
  }

  SU2_DEV static void forward2(cpx<T>* buf, int t) {
    constexpr int TOTAL = N * GB;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      cpx<T>* row = buf + (idx % N) * FP + GA * (idx / N);
      cpx<T> a[GA];
#pragma unroll
      for (int l1 = 0; l1 < GA; l1++) a[l1] = row[l1];
      Dft<T, GA, 1>::run(a);
#pragma unroll
      for (int q1 = 0; q1 < GA; q1++) row[q1] = a[q1];
    }
  }

  // gamma frequency of forward column c
  SU2_DEV static int forward_q(int c, int s) { return R * (c / GA + GB * (c % GA)) + s; }

  SU2_DEV static void forward3(cpx<T>* buf, const cpx<T>* tw, int s, int so3, int t) {
    constexpr int TOTAL = M * AA;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      const int c = idx % M, j1 = idx / M;
      const int odd = so3 ? 0 : (R % 2 == 0 ? s & 1 : forward_q(c, s) & 1);
      cpx<T>* col = buf + j1 * FP + c;
      cpx<T> a[AB];
#pragma unroll
      for (int j2 = 0; j2 < AB; j2++) a[j2] = col[AA * j2 * FP];
      half_bins<T, AB, 1>(a, odd != 0);
      Dft<T, AB, 1>::run(a);
#pragma unroll
      for (int p2 = 0; p2 < AB; p2++) col[AA * p2 * FP] = mul(a[p2], tw[(2 * p2 + odd) * j1]);
    }
  }

  SU2_DEV static void forward4(cpx<T>* buf, int t) {
    constexpr int TOTAL = M * AB;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      cpx<T>* col = buf + (idx / M) * AA * FP + idx % M;
      cpx<T> a[AA];
#pragma unroll
      for (int j1 = 0; j1 < AA; j1++) a[j1] = col[j1 * FP];
      Dft<T, AA, 1>::run(a);
#pragma unroll
      for (int p1 = 0; p1 < AA; p1++)
        if (kept_p1(p1)) col[p1 * FP] = a[p1];
    }
  }

  // S points at (tile 0, node k, signal b); tile_step values to the next tile
  SU2_DEV static void forward5(const cpx<T>* buf, cpx<T>* S, size_t tile_step, const int4* cols, T Wk, int s, int t) {
    constexpr int TOTAL = M * B;
#pragma unroll 2
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      const int qp = idx / B;
      const RadixCol col = radix_col(cols[R * qp + s]);
      const int ps = idx % B - col.nneg;
      if (ps >= col.npos) continue;
      const int p = ps < 0 ? ps + N : ps;
      const cpx<T> v = buf[(AA * (p % AB) + p / AB) * FP + (qp % GB) * GA + qp / GB];
      const int pair = radix_pair(col, ps);
      S[(size_t)(pair / PT) * tile_step + pair % PT] = ipow_times(v, (col.e0 + 3 * ps) & 3, Wk);
    }
  }

};

template <class T, int N_, class C_>
struct RadixInverse : RadixThreads<C_> {
  typedef C_ C;
  typedef RadixThreads<C> TH;
  using TH::in;
  using TH::iters;
  static constexpr int N = N_, R = C::R, M = N / R, NTR = C::NTR, B = N / 2;
  static constexpr int A1 = C::A1, A2 = C::A2, G1 = C::G1, G2 = C::G2;
  static_assert(A1 * A2 == M && G1 * G2 == N && R * M == N, "shape");
  static constexpr int G1P = G2 == 1 || N <= 24 ? G1 : (G1 | 1);  // column group pitch (short rows need no pad)
  static constexpr int IP = (G2 * G1P) | 1;            // row pitch
  static constexpr int LDS = M * IP;
  // folded bins p = p' + r M: false where none is retained for any p'
  SU2_DEV static constexpr bool kept_fold(int r) { return !(4 * r * M >= N && 4 * (r * M + M - 1) < 3 * N); }
  static constexpr int BATCH1 = sizeof(T) == 4 ? 2 : 1;

  SU2_DEV static int inverse_col(int q) { return (q / G1) * G1P + q % G1; }

  SU2_DEV static void inverse1(const cpx<T>* S, size_t tile_step, cpx<T>* buf, const cpx<T>* tw, const cpx<T>* twg,
                              const int4* cols, T scale, int s, int t) {
    constexpr int TOTAL = N * A1, IT = iters(TOTAL), U = IT < BATCH1 ? IT : BATCH1;
#pragma unroll 1
    for (int i0 = 0; i0 < IT; i0 += U) {
      cpx<T> v[U][A2];
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int idx = t + NTR * (i0 + u);
        if (!((IT % U == 0 || i0 + u < IT) && in(idx, TOTAL))) continue;
        const int q = idx / A1, a = idx % A1;
        const RadixCol col = radix_col(cols[q]);
#pragma unroll
        for (int b = 0; b < A2; b++) {
          v[u][b] = {T(0), T(0)};
#pragma unroll
          for (int r = 0; r < R; r++) {
            if (!kept_fold(r)) continue;
            const int p = a + A1 * b + r * M;
            const int ps = p < B ? p : p - N;
            cpx<T> h = {T(0), T(0)};
            if (ps >= -col.nneg && ps < col.npos) {
              const int pair = radix_pair(col, ps);
              h = ipow_times(S[(size_t)(pair / PT) * tile_step + pair % PT], -(col.e0 + 3 * ps) & 3, scale);
            }
            // w^{-s (A1 b + r M)}; the rest, w^{-s a}, rides on the twiddle
            if (R > 1 && (b > 0 || r > 0)) h = mul_conj(h, twg[2 * ((s * (A1 * b + r * M)) % N)]);
            v[u][b] = cadd(v[u][b], h);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int idx = t + NTR * (i0 + u);
        if (!((IT % U == 0 || i0 + u < IT) && in(idx, TOTAL))) continue;
        const int q = idx / A1, a = idx % A1;
        Dft<T, A2, -1>::run(v[u]);
#pragma unroll
        for (int k2 = 0; k2 < A2; k2++) {
          if (k2 > 0 || R > 1) v[u][k2] = mul_conj(v[u][k2], tw[2 * a * (s + R * k2)]);
          buf[(a + A1 * k2) * IP + inverse_col(q)] = v[u][k2];
        }
      }
    }
  }

  SU2_DEV static void inverse2(cpx<T>* buf, const cpx<T>* tw, int s, int so3, int t) {
    constexpr int TOTAL = N * A2;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      const int q = idx % N, k2 = idx / N;
      cpx<T>* col = buf + A1 * k2 * IP + inverse_col(q);
      cpx<T> v[A1];
#pragma unroll
      for (int a = 0; a < A1; a++) v[a] = col[a * IP];
      Dft<T, A1, -1>::run(v);
      const bool odd = !so3 && (q & 1);
#pragma unroll
      for (int k1 = 0; k1 < A1; k1++) {
        const cpx<T> w = tw[odd ? R * (k2 + A2 * k1) + s : 0];
        col[k1 * IP] = mul_conj(v[k1], w);
      }
    }
  }

  SU2_DEV static void inverse3(cpx<T>* buf, const cpx<T>* tw, int t) {
    constexpr int TOTAL = M * G1;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      const int g1 = idx / M;
      cpx<T>* row = buf + (idx % M) * IP + g1;
      cpx<T> v[G2];
#pragma unroll
      for (int g2 = 0; g2 < G2; g2++) v[g2] = row[g2 * G1P];
      Dft<T, G2, -1>::run(v);
#pragma unroll
      for (int u2 = 0; u2 < G2; u2++) row[u2 * G1P] = u2 > 0 ? mul_conj(v[u2], tw[2 * g1 * u2]) : v[u2];
    }
  }

  template <bool REAL>
  SU2_DEV static void inverse4_as(const cpx<T>* buf, cpx<T>* x, int s, int t) {
    constexpr int TOTAL = M * G2;
#pragma unroll 1
    for (int i = 0; i < iters(TOTAL); i++) {
      const int idx = t + NTR * i;
      if (!in(idx, TOTAL)) continue;
      const int u2 = idx % G2, row = idx / G2;
      const cpx<T>* src = buf + row * IP + u2 * G1P;
      cpx<T> v[G1];
#pragma unroll
      for (int g1 = 0; g1 < G1; g1++) v[g1] = src[g1];
      Dft<T, G1, -1>::run(v);
      const int j = R * (row / A1 + A2 * (row % A1)) + s;
#pragma unroll
      for (int u1 = 0; u1 < G1; u1++) {
        if constexpr (REAL) {
          keep_value(v[u1].im);  // formed all the same: the real part rounds as in the complex case
          nt_store(&reinterpret_cast<T*>(x)[j * N + u2 + G2 * u1], v[u1].re);
        } else {
          nt_store(&x[j * N + u2 + G2 * u1], v[u1]);
        }
      }
    }
  }
  SU2_DEV static void inverse4(const cpx<T>* buf, cpx<T>* x, int s, int real_io, int t) {
    if (real_io) inverse4_as<true>(buf, x, s, t);
    else inverse4_as<false>(buf, x, s, t);
  }
};

// Workgroup blk, sub-group sub -> ring and slice.  R = 1: RPW consecutive
// rings per workgroup.  R > 1 (RPW = 1): ids are dealt to the XCDs round robin
// (id % 8), so a ring's slices take consecutive slots of one XCD.
template <int R, int RPW>
__device__ __forceinline__ void radix_slot(int blk, int sub, int* ring, int* slice) {
  if (R == 1) {
    *ring = blk * RPW + sub;
    *slice = 0;
  } else {
    const int x = blk % NXCD, r = blk / NXCD;
    *ring = (r / R) * NXCD + x;
    *slice = r % R;
  }
}
template <int R, int RPW>
inline unsigned radix_grid(long long rings) {
  return R == 1 ? (unsigned)((rings + RPW - 1) / RPW) : (unsigned)((rings + NXCD - 1) / NXCD * NXCD * R);
}

// dynamic LDS of a workgroup: the column table where it fits (it does not in
// the FP64 inverse at N = 192), the roots, the slices
template <class T, int N, bool FWD, class C, int RPW = C::RPW>
constexpr size_t radix_lds_values() {
  return 2 * N + (size_t)RPW * std::conditional<FWD, RadixForward<T, N, C>, RadixInverse<T, N, C>>::type::LDS;
}
template <class T, int N, bool FWD, class C, int RPW = C::RPW>
constexpr bool radix_cols_in_lds() {
  return sizeof(int4) * N + radix_lds_values<T, N, FWD, C, RPW>() * sizeof(cpx<T>) <= 160 * 1024;
}

// workgroup blk of a launch of one length: RPW slices, NT threads
template <class T, int N, bool FWD, class C, int RPW = C::RPW, int NT = C::NTR * RPW>
__device__ __forceinline__ void radix_workgroup(const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out,
                                                const RadixRingParams<T>& p, int blk, unsigned char* smem_raw) {
  typedef typename std::conditional<FWD, RadixForward<T, N, C>, RadixInverse<T, N, C>>::type X;
  constexpr int NTR = C::NTR;
  // the column table and the roots, in LDS for the whole workgroup (a column's
  // entry read from memory would put its latency in front of the spectra's)
  constexpr bool CL = radix_cols_in_lds<T, N, FWD, C, RPW>();
  int4* lcols = reinterpret_cast<int4*>(smem_raw);
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(lcols + (CL ? N : 0));
  if constexpr (CL)
    for (int u = threadIdx.x; u < N; u += NT) lcols[u] = p.cols[u];
  const int4* cols = CL ? lcols : p.cols;
  for (int u = threadIdx.x; u < 2 * N; u += NT) tw[u] = p.tw[u];
  const int sub = NT == NTR ? 0 : threadIdx.x / NTR, t = NT == NTR ? threadIdx.x : threadIdx.x - sub * NTR;
  const bool live = NT == NTR * RPW || sub < RPW;  // threads beyond the slices only take part in the barriers
  cpx<T>* buf = tw + 2 * N + (live ? sub : 0) * X::LDS;
  int ring, s;
  radix_slot<C::R, RPW>(blk, sub, &ring, &s);
  // forward rings node-major over the signals, inverse rings signal-major:
  // the orders of the register-resident kernels, for the same reasons
  const bool ok = live && ring < p.batch * N;
  const int rr = ok ? ring : 0;
  const int b = FWD ? rr % p.batch : rr / N, k = FWD ? rr / p.batch : rr % N;
  const size_t x0 = ring_offset(p.soff, b, N) + (size_t)k * N * N;
  const size_t s0 = ((size_t)k * p.batch + b) * PT, tile_step = (size_t)N * p.batch * PT;
  __syncthreads();
  if constexpr (FWD) {
    const cpx<T>* x = p.real_io ? reinterpret_cast<const cpx<T>*>(reinterpret_cast<const T*>(in) + x0) : in + x0;
    if (ok) X::forward1(x, buf, tw, p.tw, s, p.real_io, t);
    __syncthreads();
    if (live) X::forward2(buf, t);
    __syncthreads();
    if (live) X::forward3(buf, tw, s, p.so3, t);
    __syncthreads();
    if (live) X::forward4(buf, t);
    __syncthreads();
    if (ok) X::forward5(buf, out + s0, tile_step, cols, p.W[k], s, t);
  } else {
    cpx<T>* x = p.real_io ? reinterpret_cast<cpx<T>*>(reinterpret_cast<T*>(out) + x0) : out + x0;
    if (ok) X::inverse1(in + s0, tile_step, buf, tw, p.tw, cols, p.adjoint ? p.W[k] : T(1), s, t);
    __syncthreads();
    if (live) X::inverse2(buf, tw, s, p.so3, t);
    __syncthreads();
    if (live) X::inverse3(buf, tw, t);
    __syncthreads();
    if (ok) X::inverse4(buf, x, s, p.real_io, t);
  }
}

template <class T, int N, bool FWD, class C>
__global__ __launch_bounds__((C::NTR * C::RPW)) void ring_radix_kernel(const cpx<T>* __restrict__ in,
                                                                       cpx<T>* __restrict__ out, RadixRingParams<T> p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  radix_workgroup<T, N, FWD, C>(in, out, p, blockIdx.x, smem_raw);
}

template <class T, int N, bool FWD, class C = RadixCfg<T, N, FWD>>
static hipError_t launch_radix(const RadixRingParams<T>& p, const cpx<T>* in, cpx<T>* out, hipStream_t s) {
  constexpr size_t smem = (radix_cols_in_lds<T, N, FWD, C>() ? sizeof(int4) * N : 0) +
                          radix_lds_values<T, N, FWD, C>() * sizeof(cpx<T>);
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  if (smem > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)ring_radix_kernel<T, N, FWD, C>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((ring_radix_kernel<T, N, FWD, C>), dim3(radix_grid<C::R, C::RPW>((long long)p.batch * N)),
                     dim3(C::NTR * C::RPW), smem, s, in, out, p);
  return hipGetLastError();
}

template <class T, bool FWD>
static hipError_t launch_radix_any(const RadixRingParams<T>& p, const cpx<T>* in, cpx<T>* out, hipStream_t s) {
  switch (p.N) {
#define SU2_RADIX_CASE(NN) \
  case NN: return launch_radix<T, NN, FWD>(p, in, out, s);
    SU2_RADIX_CASE(2) SU2_RADIX_CASE(4) SU2_RADIX_CASE(6) SU2_RADIX_CASE(8) SU2_RADIX_CASE(12) SU2_RADIX_CASE(18)
    SU2_RADIX_CASE(24) SU2_RADIX_CASE(36) SU2_RADIX_CASE(48) SU2_RADIX_CASE(54) SU2_RADIX_CASE(72) SU2_RADIX_CASE(96)
    SU2_RADIX_CASE(108) SU2_RADIX_CASE(144) SU2_RADIX_CASE(162) SU2_RADIX_CASE(192) SU2_RADIX_CASE(216)
#undef SU2_RADIX_CASE
  }
  return hipErrorInvalidValue;
}

// ---- several lengths in one launch (mixed plans) ----
//
// Groups of a few rings leave the chip idle one launch after another.  Here a
// workgroup takes its group and workgroup number from a list and runs its
// length's shape, with as many rings as fit the list's workgroup (the shape's own
// threads per ring, so that the compiler forms the same products and sums and
// the bits are those of the length's own launch).  Up to N = 54: longer rings
// want more threads and LDS than the short ones beside them can share.
template <class T>
constexpr int radix_list_threads() { return sizeof(T) == 4 ? 256 : 384; }  // the longest shape's
template <class T, int N, bool FWD>
struct RadixListShape {
  typedef RadixCfg<T, N, FWD> C;
  static_assert(C::R == 1, "whole rings");
  static constexpr int NT = radix_list_threads<T>(), RPW = NT / C::NTR;
  static_assert(RPW == NT / RadixCfg<T, N, !FWD>::NTR, "one list for both directions");
  static constexpr size_t smem = sizeof(int4) * N + radix_lds_values<T, N, FWD, C, RPW>() * sizeof(cpx<T>);
  static_assert(smem <= 64 * 1024, "no attribute needed");
};
#define SU2_RADIX_LIST(X) X(2) X(4) X(6) X(8) X(12) X(18) X(24) X(36) X(48) X(54)

template <class T, bool FWD>
__global__ __launch_bounds__(radix_list_threads<T>()) void ring_radix_list_kernel(
    const int2* __restrict__ items, const RadixListGroup<T>* __restrict__ groups, const cpx<T>* __restrict__ in,
    cpx<T>* __restrict__ out, int dir) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int2 w = items[blockIdx.x];
  const RadixRingParams<T> p = groups[w.x].p[dir];
  const cpx<T>* src = FWD ? in : groups[w.x].S;
  cpx<T>* dst = FWD ? groups[w.x].S : out;
  switch (p.N) {
#define SU2_RADIX_CASE(NN)                                                                                         \
  case NN:                                                                                                         \
    radix_workgroup<T, NN, FWD, RadixCfg<T, NN, FWD>, RadixListShape<T, NN, FWD>::RPW, radix_list_threads<T>()>(   \
        src, dst, p, w.y, smem_raw);                                                                               \
    break;
    SU2_RADIX_LIST(SU2_RADIX_CASE)
#undef SU2_RADIX_CASE
  }
}

template <class T>
int radix_list_blocks(int N, long long rings) {
  switch (N) {
#define SU2_RADIX_CASE(NN) \
  case NN: return (int)radix_grid<1, RadixListShape<T, NN, true>::RPW>(rings);
    SU2_RADIX_LIST(SU2_RADIX_CASE)
#undef SU2_RADIX_CASE
  }
  return 0;
}
template int radix_list_blocks<float>(int, long long);
template int radix_list_blocks<double>(int, long long);

template <class T>
size_t radix_list_smem(int N) {
  switch (N) {
#define SU2_RADIX_CASE(NN) \
  case NN: return std::max(RadixListShape<T, NN, true>::smem, RadixListShape<T, NN, false>::smem);
    SU2_RADIX_LIST(SU2_RADIX_CASE)
#undef SU2_RADIX_CASE
  }
  return 0;
}
template size_t radix_list_smem<float>(int);
template size_t radix_list_smem<double>(int);

template <class T>
hipError_t launch_radix_list(bool forward, int dir, const int2* items, int n, size_t smem,
                             const RadixListGroup<T>* groups, const cpx<T>* in, cpx<T>* out, hipStream_t s) {
  const dim3 grid(n), block(radix_list_threads<T>());
  if (forward)
    hipLaunchKernelGGL((ring_radix_list_kernel<T, true>), grid, block, smem, s, items, groups, in, out, dir);
  else
    hipLaunchKernelGGL((ring_radix_list_kernel<T, false>), grid, block, smem, s, items, groups, in, out, dir);
  return hipGetLastError();
}
template hipError_t launch_radix_list<float>(bool, int, const int2*, int, size_t, const RadixListGroup<float>*,
                                             const cpx<float>*, cpx<float>*, hipStream_t);
template hipError_t launch_radix_list<double>(bool, int, const int2*, int, size_t, const RadixListGroup<double>*,
                                              const cpx<double>*, cpx<double>*, hipStream_t);

// ---- whole signals: rings and contraction in one kernel (N <= 12) ----
//
// One workgroup per signal: its rings, one sub-group each, into spectra kept in LDS,
// and the contraction from there (su2fft_fused.h); the inverse the other way
// round.  The spectra go to the plan's workspace as well, where the stage by
// stage launches leave them.
template <class T, int N, bool FWD>
struct FusedShape {
  typedef RadixCfg<T, N, FWD> C;
  typedef typename std::conditional<FWD, RadixForward<T, N, C>, RadixInverse<T, N, C>>::type X;
  static_assert(C::R == 1, "whole rings");
  static constexpr int NT = N == 12 ? 768 : 512, NTR = C::NTR;  // 12 wavefronts for the 12 rings at N = 12
  static_assert(N * NTR <= NT, "a sub-group per ring");
};

template <class T, int N, bool FWD>
static size_t fused_smem(const BetaParams<T>& q) {
  typedef FusedShape<T, N, FWD> F;
  return sizeof(int4) * N +
         (2 * N + (size_t)q.ntiles * PT * N + (size_t)N * F::X::LDS + (FWD ? 0 : q.ncoef)) * sizeof(cpx<T>);
}

template <class T, int N, bool FWD>
__global__ __launch_bounds__((FusedShape<T, N, FWD>::NT)) void radix_fused_kernel(const cpx<T>* __restrict__ in,
                                                                                cpx<T>* __restrict__ out,
                                                                                cpx<T>* __restrict__ Sg,
                                                                                RadixRingParams<T> p, BetaParams<T> q) {
  typedef FusedShape<T, N, FWD> F;
  typedef typename F::X X;
  constexpr int NT = F::NT;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  int4* cols = reinterpret_cast<int4*>(smem_raw);
  cpx<T>* tw = reinterpret_cast<cpx<T>*>(cols + N);
  const int ns = q.ntiles * PT * N;
  cpx<T>* Sl = tw + 2 * N;
  cpx<T>* bufs = Sl + ns;
  const int t = threadIdx.x, b = blockIdx.x, k = t / F::NTR, tr = t - k * F::NTR;
  const size_t x0 = ring_offset(p.soff, b, N), c0 = coef_offset(q.coff, b, q.ncoef);
  for (int u = t; u < N; u += NT) cols[u] = p.cols[u];
  for (int u = t; u < 2 * N; u += NT) tw[u] = p.tw[u];
  const bool ok = k < N;
  cpx<T>* buf = bufs + (ok ? k : 0) * X::LDS;
  const size_t xk = x0 + (size_t)k * N * N;
  if constexpr (FWD) {
    __syncthreads();
    const cpx<T>* x = p.real_io ? reinterpret_cast<const cpx<T>*>(reinterpret_cast<const T*>(in) + xk) : in + xk;
    if (ok) X::forward1(x, buf, tw, p.tw, 0, p.real_io, tr);
    __syncthreads();
    if (ok) X::forward2(buf, tr);
    __syncthreads();
    if (ok) X::forward3(buf, tw, 0, p.so3, tr);
    __syncthreads();
    if (ok) X::forward4(buf, tr);
    __syncthreads();
    if (ok) X::forward5(buf, Sl + k * PT, (size_t)N * PT, cols, p.W[k], 0, tr);
    __syncthreads();
    fused_contract_forward<T, N, NT>(Sl, out + c0, q, t);
    for (int e = t; e < ns; e += NT)
      Sg[((size_t)(e / PT) * p.batch + b) * PT + e % PT] = Sl[e];
  } else {
    cpx<T>* Cl = bufs + N * X::LDS;
    for (int e = t; e < (int)q.ncoef; e += NT) Cl[e] = in[c0 + e];
    __syncthreads();
    fused_contract_inverse<T, N, NT>(Cl, Sl, q, t);
    __syncthreads();
    for (int e = t; e < ns; e += NT)
      Sg[((size_t)(e / PT) * p.batch + b) * PT + e % PT] = Sl[e];
    cpx<T>* x = p.real_io ? reinterpret_cast<cpx<T>*>(reinterpret_cast<T*>(out) + xk) : out + xk;
    if (ok) X::inverse1(Sl + k * PT, (size_t)N * PT, buf, tw, p.tw, cols, p.adjoint ? p.W[k] : T(1), 0, tr);
    __syncthreads();
    if (ok) X::inverse2(buf, tw, 0, p.so3, tr);
    __syncthreads();
    if (ok) X::inverse3(buf, tw, tr);
    __syncthreads();
    if (ok) X::inverse4(buf, x, 0, p.real_io, tr);
    __syncthreads();
  }
}

template <class T, int N, bool FWD>
static hipError_t launch_fused(const RadixRingParams<T>& p, const BetaParams<T>& q, const cpx<T>* in, cpx<T>* out,
                               cpx<T>* Sg, hipStream_t s) {
  const size_t smem = fused_smem<T, N, FWD>(q);
  if (smem > 160 * 1024) return hipErrorInvalidValue;
  if (smem > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)radix_fused_kernel<T, N, FWD>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((radix_fused_kernel<T, N, FWD>), dim3(p.batch), dim3(FusedShape<T, N, FWD>::NT), smem, s, in, out,
                     Sg, p, q);
  return hipGetLastError();
}

template <class T>
hipError_t launch_radix_fused(bool forward, const RadixRingParams<T>& p, const BetaParams<T>& q, const cpx<T>* in,
                              cpx<T>* out, cpx<T>* Sg, hipStream_t s) {
  switch (p.N) {
#define SU2_FUSED_CASE(NN) \
  case NN: return forward ? launch_fused<T, NN, true>(p, q, in, out, Sg, s) : launch_fused<T, NN, false>(p, q, in, out, Sg, s);
    SU2_FUSED_CASE(2) SU2_FUSED_CASE(4) SU2_FUSED_CASE(6) SU2_FUSED_CASE(8) SU2_FUSED_CASE(12)
#undef SU2_FUSED_CASE
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_radix_fused<float>(bool, const RadixRingParams<float>&, const BetaParams<float>&,
                                              const cpx<float>*, cpx<float>*, cpx<float>*, hipStream_t);
template hipError_t launch_radix_fused<double>(bool, const RadixRingParams<double>&, const BetaParams<double>&,
                                               const cpx<double>*, cpx<double>*, cpx<double>*, hipStream_t);

template <class T>
hipError_t launch_ring_forward_radix(const RadixRingParams<T>& p, const cpx<T>* samples, cpx<T>* S, hipStream_t s) {
  return launch_radix_any<T, true>(p, samples, S, s);
}
template <class T>
hipError_t launch_ring_inverse_radix(const RadixRingParams<T>& p, const cpx<T>* S, cpx<T>* samples, hipStream_t s) {
  return launch_radix_any<T, false>(p, S, samples, s);
}

template hipError_t launch_ring_forward_radix<float>(const RadixRingParams<float>&, const cpx<float>*, cpx<float>*,
                                                     hipStream_t);
template hipError_t launch_ring_forward_radix<double>(const RadixRingParams<double>&, const cpx<double>*, cpx<double>*,
                                                      hipStream_t);
template hipError_t launch_ring_inverse_radix<float>(const RadixRingParams<float>&, const cpx<float>*, cpx<float>*,
                                                     hipStream_t);
template hipError_t launch_ring_inverse_radix<double>(const RadixRingParams<double>&, const cpx<double>*, cpx<double>*,
                                                      hipStream_t);

}  // namespace su2

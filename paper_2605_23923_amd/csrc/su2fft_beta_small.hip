// The beta contractions (su2fft_beta.hip) for small batches: the same products
// in the same order, hence the same bits, streamed straight into the matrix
// cores.
//
// With few signals the Wigner-d table is most of the bytes and the tile
// kernels lose twice: their 16- or 32-signal tiles leave most matrix-core
// columns empty, and one staged chunk per workgroup keeps too few bytes in
// flight.  Here a wave owns one pair (m, n) together with its mirror
// (-m, -n), which uses the same table column up to sign: the columns of one
// 16-wide product are 2 pairs x 4 signals x (re, im), every table value is
// read once per 4 signals, by coalesced loads that go directly into operand
// registers, many of them in flight, and the forward has no LDS and no barrier
// at all.  More signals take more waves, which share the table through L2
// (two products side by side per wave measured slower: B = 48 FP64, 12 signals
// inverse 37 against 22 us).  Plans without the symmetric
// pair list, and half-spectrum real plans (whose mirrors carry no spectra),
// take one pair per wave and 8 signals per product.
#include "su2fft_beta_small.h"

namespace su2 {

// Forward: fhat(l)_{mn}[b] = sum_k d^l(beta_k) S_k(m, n)[b].  One wave per
// pair (and mirror): table rows as the A operand, spectra as the B operand,
// KU groups of 4 nodes requested together.  RT row tiles cover the pair's L
// degrees, degree RT i + rt in row i of tile rt, so that a lane's values of
// all row tiles are adjacent and come in one load.
constexpr int SMALL_FWD_WAVES = 4;  // waves (pairs) per workgroup: a quarter of a tile

// a wave's sums out to the coefficient vectors
template <class T, int RT, int MIR>
__device__ __forceinline__ void store_forward_small(cpx<T>* __restrict__ coeffs, const BetaParams<T>& p,
                                                    const SmallPairs<T, MIR>& w, int b0, int lane,
                                                    const typename acc4<T>::type (&acc)[RT]) {
  typedef SmallCols<MIR> Cols;
  const int col = lane & 15, b = b0 + Cols::sig(col);
  const auto q = w.pick(Cols::mir(col));
  if (b >= p.batch) return;
  T* out = reinterpret_cast<T*>(coeffs + coef_offset(p.coff, b, p.ncoef)) + (col & 1);
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int r = 0; r < 4; r++)
      store_coef_small<T, MIR>(out, p, q, RT * acc_row<T>(lane, r) + rt, col & 1, acc[rt][r]);
}

template <class T, int RT, int MIR>
__device__ __forceinline__ void beta_forward_small_pair(const cpx<T>* __restrict__ S, cpx<T>* __restrict__ coeffs,
                                                        const BetaParams<T>& p, const SmallPairs<T, MIR>& w, int b0,
                                                        int lane) {
  typedef typename acc4<T>::type accT;
  typedef SmallCols<MIR> Cols;
  // RT adjacent table values, at any element's alignment
  typedef T rowv __attribute__((ext_vector_type(RT), aligned(sizeof(T))));
  constexpr int KU = RT == 1 ? (sizeof(T) == 4 ? 16 : 8) : (RT == 2 ? 8 : 4);
  const int lrow = lane & 15, lk = lane >> 4, N = p.N;
  // operand addresses of node lk.  Rows past L read the columns after the
  // pair's (or the padding after the table) and are dropped; signals past the
  // batch read the last one and are dropped likewise.
  static_assert(16 * RT <= TABLE_PAD && 15 * RT + 4 <= TABLE_PAD, "a three-value load may take four");
  const T* ta = p.tab + w.tab + w.coff + (long long)lk * w.lsum + RT * lrow;
  const int pos = MIR == 2 && Cols::mir(lrow) ? w.pos1 : w.pos0, bs = min(b0 + Cols::sig(lrow), p.batch - 1);
  const T* tb = reinterpret_cast<const T*>(S + (((size_t)(pos / PT) * N + lk) * p.batch + bs) * PT + pos % PT) + (lrow & 1);
  const long long sa = 4LL * w.lsum, sb = 8LL * p.batch * PT;

  accT acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int r = 0; r < 4; r++) acc[rt][r] = T(0);

  auto load = [&](rowv& a, T& b) {
    a = *reinterpret_cast<const rowv*>(ta);
    ta += sa;
    b = *tb;
    tb += sb;
  };
  auto products = [&](const rowv& a, const T b) {
#pragma unroll
    for (int rt = 0; rt < RT; rt++) acc[rt] = mfma16x16x4(a[rt], b, acc[rt]);
  };
  const int ng = N / 4;  // whole groups of 4 nodes
  int g = 0;
  for (; g + KU <= ng; g += KU) {
    rowv a[KU];
    T b[KU];
#pragma unroll
    for (int u = 0; u < KU; u++) load(a[u], b[u]);
#pragma unroll
    for (int u = 0; u < KU; u++) products(a[u], b[u]);
  }
  if constexpr (KU > 4)
    for (; g + 4 <= ng; g += 4) {
      rowv a[4];
      T b[4];
#pragma unroll
      for (int u = 0; u < 4; u++) load(a[u], b[u]);
#pragma unroll
      for (int u = 0; u < 4; u++) products(a[u], b[u]);
    }
  for (; g < ng; g++) {
    rowv a;
    T b;
    load(a, b);
    products(a, b);
  }
  if (N % 4 != 0) {  // the last N mod 4 nodes, zeros past them
    const bool in = 4 * ng + lk < N;
    rowv a;
#pragma unroll
    for (int rt = 0; rt < RT; rt++) a[rt] = in ? ta[rt] : T(0);
    products(a, in ? *tb : T(0));
  }

  store_forward_small<T, RT, MIR>(coeffs, p, w, b0, lane, acc);
}

// RTMAX: row tiles of the plan's longest pairs (beta_rtmax)
template <class T, int RTMAX, int MIR>
__global__ __launch_bounds__(64 * SMALL_FWD_WAVES) void beta_forward_small_kernel(const cpx<T>* __restrict__ S,
                                                                                  cpx<T>* __restrict__ coeffs,
                                                                                  BetaParams<T> p, int pos_end) {
  constexpr int BT = SmallCols<MIR>::BT, QT = PT / SMALL_FWD_WAVES;
  const int nbt = (p.batch + BT - 1) / BT;
  const int ntl = (pos_end - p.tile0 * PT + PT - 1) / PT;
  const TileSlot sl = contraction_slot(blockIdx.x, ntl, QT * nbt);
  if (!sl.valid) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int at = (p.tile0 + sl.tile) * PT + (sl.bt % QT) * SMALL_FWD_WAVES + wave, b0 = sl.bt / QT * BT;
  if (at >= pos_end) return;
  const SmallPairs<T, MIR> w(p, at);
  if (w.L == 0) return;
  const int rt = (w.L + 15) / 16;  // uniform
  if constexpr (RTMAX >= 4) {
    if (rt == 4) return beta_forward_small_pair<T, 4, MIR>(S, coeffs, p, w, b0, lane);
    if (rt == 3) return beta_forward_small_pair<T, 3, MIR>(S, coeffs, p, w, b0, lane);
  }
  if constexpr (RTMAX >= 2)
    if (rt == 2) return beta_forward_small_pair<T, 2, MIR>(S, coeffs, p, w, b0, lane);
  beta_forward_small_pair<T, 1, MIR>(S, coeffs, p, w, b0, lane);
}

// Forward with the spectra through LDS, from a few signals on: a wave that
// reads its own pair's values touches a 128-byte line of S per node and signal
// for 8 of its bytes, which soon costs more than the table.  One workgroup of
// 16 waves per pair tile (and its mirror tile) reads whole lines, KG groups of
// 4 nodes at a time into one of two buffers; table values still go straight
// to registers.
constexpr int MID_THREADS = 64 * PT;

template <class T, int RTMAX, int MIR>
struct MidShape {
  static constexpr int BT = SmallCols<MIR>::BT;
  // 70 KB for the two buffers, two workgroups per CU (half of it where the
  // operands of 64 degrees need the registers)
  static constexpr int KG = sizeof(T) == 4 && RTMAX < 4 ? 8 : 4;
  static constexpr int KN = 4 * KG;
  static constexpr int PB = 2 * PT + 2, HALF = KN * BT * PB + 2;  // one of the MIR tiles' rows
  static constexpr int VC = 16 / (int)sizeof(cpx<T>), VPR = PT / VC;  // 16-byte vectors per row
  static constexpr int NV = MIR * KN * BT * VPR, VPT = (NV + MID_THREADS - 1) / MID_THREADS;
};

template <class T, int RTMAX, int RT, int MIR>
__device__ __forceinline__ void beta_forward_mid_body(const cpx<T>* __restrict__ S, cpx<T>* __restrict__ coeffs,
                                                      const BetaParams<T>& p, const SmallPairs<T, MIR>& w, int tile,
                                                      int b0, T* lds, int wave, int lane) {
  typedef typename acc4<T>::type accT;
  typedef SmallCols<MIR> Cols;
  typedef MidShape<T, RTMAX, MIR> MS;
  typedef T rowv __attribute__((ext_vector_type(RT), aligned(sizeof(T))));
  typedef T vec16 __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int KG = MS::KG, KN = MS::KN, BT = MS::BT;
  const int lrow = lane & 15, lk = lane >> 4, N = p.N, tid = wave * 64 + lane;
  const int nb = min(BT, p.batch - b0), ng = (N + 3) / 4, nchunk = (ng + KG - 1) / KG;
  const bool work = w.L > 0;

  // this thread's 16-byte pieces of a chunk of S: row (mir, node, signal), piece pv
  vec16 sv[MS::VPT];
  auto fetch_s = [&](int c) {
#pragma unroll
    for (int i = 0; i < MS::VPT; i++) {
      const int v = tid + MID_THREADS * i, pv = v % MS::VPR, bb = v / MS::VPR % BT, kk = v / (MS::VPR * BT) % KN;
      const int mir = v / (MS::VPR * BT * KN), k = c * KN + kk, t = mir ? p.ntiles - 1 - tile : tile;
      sv[i] = vec16(T(0));
      if (v < MS::NV && k < N && bb < nb)
        sv[i] = *reinterpret_cast<const vec16*>(S + (((size_t)t * N + k) * p.batch + b0 + bb) * PT + pv * MS::VC);
    }
  };
  auto commit_s = [&](int c) {
    T* d = lds + (c & 1) * MIR * MS::HALF;
#pragma unroll
    for (int i = 0; i < MS::VPT; i++) {
      const int v = tid + MID_THREADS * i, pv = v % MS::VPR, bb = v / MS::VPR % BT, kk = v / (MS::VPR * BT) % KN;
      const int mir = v / (MS::VPR * BT * KN);
      if (v < MS::NV)
#pragma unroll
        for (int e = 0; e < 2 * MS::VC; e++) d[mir * MS::HALF + (kk * BT + bb) * MS::PB + 2 * pv * MS::VC + e] = sv[i][e];
    }
  };
  // RT is the tile's: a pair with fewer row tiles reads the columns after its
  // own, or the padding after the table, and drops the rows
  static_assert(16 * RT <= TABLE_PAD && 15 * RT + 4 <= TABLE_PAD, "a three-value load may take four");
  rowv a[KG];
  const T* ta = p.tab + w.tab + w.coff + (long long)lk * w.lsum + RT * lrow;
  const long long sa = 4LL * w.lsum;
  auto fetch_a = [&](int c) {
#pragma unroll
    for (int u = 0; u < KG; u++) {
      const int g = c * KG + u;
#pragma unroll
      for (int rt = 0; rt < RT; rt++) a[u][rt] = T(0);
      if (work && 4 * g + lk < N) a[u] = *reinterpret_cast<const rowv*>(ta + g * sa);
    }
  };
  const int hm = MIR == 2 ? Cols::mir(lrow) : 0;
  const int bofs = hm * MS::HALF + (lk * BT + Cols::sig(lrow)) * MS::PB + 2 * (hm ? PT - 1 - wave : wave) + (lrow & 1);

  accT acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int r = 0; r < 4; r++) acc[rt][r] = T(0);
  fetch_s(0);
  fetch_a(0);
  commit_s(0);
  __syncthreads();
  for (int c = 0; c < nchunk; c++) {
    if (c + 1 < nchunk) fetch_s(c + 1);
    const T* src = lds + (c & 1) * MIR * MS::HALF;
    if (work) {
#pragma unroll
      for (int u = 0; u < KG; u++) {
        if (c * KG + u >= ng) break;
        const T b = src[bofs + 4 * u * BT * MS::PB];
#pragma unroll
        for (int rt = 0; rt < RT; rt++) acc[rt] = mfma16x16x4(a[u][rt], b, acc[rt]);
      }
    }
    if (c + 1 < nchunk) {
      fetch_a(c + 1);
      commit_s(c + 1);
    }
    __syncthreads();
  }
  if (work) store_forward_small<T, RT, MIR>(coeffs, p, w, b0, lane, acc);
}

template <class T, int RTMAX, int MIR>
__global__ __launch_bounds__(MID_THREADS) void beta_forward_mid_kernel(const cpx<T>* __restrict__ S,
                                                                       cpx<T>* __restrict__ coeffs, BetaParams<T> p,
                                                                       int pos_end) {
  typedef MidShape<T, RTMAX, MIR> MS;
  __shared__ __align__(16) T lds[2 * MIR * MS::HALF];
  const int ntl = (pos_end - p.tile0 * PT + PT - 1) / PT;
  const TileSlot sl = contraction_slot(blockIdx.x, ntl, (p.batch + MS::BT - 1) / MS::BT);
  if (!sl.valid) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile = p.tile0 + sl.tile, b0 = sl.bt * MS::BT;
  SmallPairs<T, MIR> w(p, tile * PT + wave);
  if (tile * PT + wave >= pos_end) w.L = 0;  // the second half of a self-mirror tile
  // row tiles of the workgroup's longest pair: one branch for all its waves
  // (barriers inside)
  int rt = 1;
  if constexpr (RTMAX > 1) {
    int L = 0;
    for (int i = 0; i < PT; i++) L = max(L, p.pairs[tile * PT + i].L);
    rt = (L + 15) / 16;
  }
  if constexpr (RTMAX >= 4) {
    if (rt >= 4) return beta_forward_mid_body<T, RTMAX, 4, MIR>(S, coeffs, p, w, tile, b0, lds, wave, lane);
    if (rt == 3) return beta_forward_mid_body<T, RTMAX, 3, MIR>(S, coeffs, p, w, tile, b0, lds, wave, lane);
  }
  if constexpr (RTMAX >= 2)
    if (rt == 2) return beta_forward_mid_body<T, RTMAX, 2, MIR>(S, coeffs, p, w, tile, b0, lds, wave, lane);
  beta_forward_mid_body<T, RTMAX, 1, MIR>(S, coeffs, p, w, tile, b0, lds, wave, lane);
}

// Inverse / adjoint: S'_k(m, n)[b] = sum_l s_l d^l(beta_k) fhat(l)_{mn}[b].
// One workgroup of 16 waves per pair tile (and its mirror tile) and range of
// 16-node blocks; a wave's scaled coefficients are its B operands, the
// inverse-layout table its A operands.  A block's rows are gathered in LDS
// and written as whole PT-pair rows of S.
constexpr int SMALL_INV_THREADS = 64 * PT;

template <class T, int LQ, int MIR>
__global__ __launch_bounds__(SMALL_INV_THREADS) void beta_inverse_small_kernel(const cpx<T>* __restrict__ coeffs,
                                                                               cpx<T>* __restrict__ S, BetaParams<T> p,
                                                                               int ntl, int blocks) {
  typedef typename acc4<T>::type accT;
  typedef SmallCols<MIR> Cols;
  constexpr int BT = Cols::BT;
  typedef SmallStage<T, BT> ST;
  __shared__ __align__(16) T stages[2][MIR * 16 * ST::NRS];
  const int N = p.N, NB = (N + 15) / 16, nsplit = (NB + blocks - 1) / blocks;
  const int nbt = (p.batch + BT - 1) / BT;
  const TileSlot sl = contraction_slot(blockIdx.x, ntl, nsplit * nbt);
  if (!sl.valid) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lrow = lane & 15, lk = lane >> 4;
  const int tile = p.tile0 + sl.tile, b0 = sl.bt / nsplit * BT;
  const int kb0 = sl.bt % nsplit * blocks, kb1 = min(NB, kb0 + blocks);
  const int nb = min(BT, p.batch - b0);
  const SmallPairs<T, MIR> w(p, tile * PT + wave);
  const int L = w.L, G = (L + 3) / 4;

  const T* ta = p.tabi + w.itab + (long long)kb0 * G * 64 + lane;
  T av[LQ];
  auto fetch = [&]() {
#pragma unroll
    for (int s = 0; s < LQ; s++) {
      av[s] = T(0);
      if (s < G) av[s] = ta[64 * s];  // wave-uniform branch
    }
    ta += (long long)G * 64;
  };
  fetch();  // in flight while the coefficients are gathered

  const int mir = MIR == 2 ? Cols::mir(lrow) : 0, sig = Cols::sig(lrow);
  T bop[LQ];
  {
    const auto q = w.pick(mir);
    const T* c = reinterpret_cast<const T*>(coeffs + coef_offset(p.coff, b0 + min(sig, nb - 1), p.ncoef)) + (lrow & 1);
#pragma unroll
    for (int s = 0; s < LQ; s++) {
      bop[s] = T(0);
      if (s < G) bop[s] = load_coef_small<T, MIR>(c, p, q, 4 * s + lk, lrow & 1, sig < nb);
    }
  }

  T* const mine = stages[0] + mir * 16 * ST::NRS + sig * ST::PB + 2 * (mir ? PT - 1 - wave : wave) + (lrow & 1);
  for (int kb = kb0; kb < kb1; kb++) {
    accT acc;
#pragma unroll
    for (int r = 0; r < 4; r++) acc[r] = T(0);
#pragma unroll
    for (int s = 0; s < LQ; s++)
      if (s < G) acc = mfma16x16x4(av[s], bop[s], acc);
    if (kb + 1 < kb1) fetch();  // next block's values, in flight during the stores
    // two stage buffers in turn: one barrier per block
#pragma unroll
    for (int r = 0; r < 4; r++) mine[(kb & 1) * MIR * 16 * ST::NRS + acc_row<T>(lane, r) * ST::NRS] = acc[r];
    __syncthreads();
    store_rows_small<T, MIR, SMALL_INV_THREADS>(S, p, stages[kb & 1], tile, kb, b0, nb, tid);
  }
}

// Forward: these kernels instead of the tile kernel where its grid of tiles and
// 16- or 32-signal groups leaves CUs idle or columns empty, i.e. by signals
// times tiles; with a tile per CU or more, by signals, two groups of 4 (three
// with the long columns of B > 64 in FP32).  Whole calls on inputs not in the
// caches, tile kernel -> these, us:
// FP32 B = 24, 32 signals 23.9 -> 20.6, 52 signals 30.3 -> 30.5; B = 32, 16 signals
// 30.3 -> 26.2, 28 signals 37.6 -> 38.5; B = 48, 8 signals 48 -> 43, 12 signals
// 62 -> 65; B = 64, 1 signal 56 -> 29, 8 signals 89 -> 76, 12 signals 110.4 -> 110.5;
// B = 72, 12 signals 236 -> 210; B = 128, 8 signals 917 -> 806.
// FP64 B = 32, 24 signals 64.3 -> 63.6, 30 signals 69 -> 73; B = 48, 16 signals
// 143 -> 137; B = 54, 12 signals 197.1 -> 196.5; SO(3) B = 64 (whole row tiles),
// 4 signals 94 -> 69, 12 signals 191 -> 197; B = 64, 4 signals 115 -> 104,
// 8 signals 170 -> 166, 9 signals 193 -> 206; B = 96, 4 signals 557 -> 375.
template <class T>
bool beta_small_forward(const BetaParams<T>& p) {
  if (small_fills(p)) return p.batch <= (sizeof(T) == 4 && p.B > 64 ? 12 : 8);
  if (sizeof(T) == 4 || beta_rtmax(p.B) == 1) return p.batch * small_units(p) <= 1600;
  return p.batch * small_units(p) <= (p.B <= 54 ? 2300 : 1200);
}

// Inverse: likewise (its tile kernel also gathers the coefficients through
// eight barriers); up to 8 degrees the tile kernel is as fast and smaller.
// FP32 B = 24, 52 signals 30.0 -> 30.4; B = 32, 16 signals 28.5 -> 25.3, 40 signals
// 47.6 -> 46.8, 60 signals 58 -> 59; B = 36, 44 signals 73.1 -> 72.6; B = 48, 12 signals
// 60 -> 55, 24 signals 110 -> 108; B = 64, 8 signals 77 -> 74, 9 signals 88 -> 94;
// B = 72, 12 signals 257 -> 229; B = 96, 8 signals 469 -> 405.
// FP64 B = 24, 72 signals 55.4 -> 54.4; B = 32, 32 signals 73 -> 69, 45 signals
// 105 -> 110; B = 48, 20 signals 209 -> 197; SO(3) B = 64, 4 signals 84 -> 64,
// 12 signals 172 -> 177; B = 64, 8 signals 166 -> 156, 9 signals 197 -> 205;
// half-spectrum B = 64, 8 signals 106 -> 107; B = 96, 4 signals 586 -> 421.
template <class T>
bool beta_small_inverse(const BetaParams<T>& p) {
  const int lq = beta_lq(p.B);
  if (lq == 2) return false;
  if (small_fills(p)) {
    if (sizeof(T) == 4) return p.batch <= (p.B > 64 ? 12 : 8);
    return p.batch <= (small_mirrored(p) ? 8 : 4);
  }
  if (sizeof(T) == 4) return p.batch <= 40 && p.batch * small_units(p) <= 3600;
  return p.batch * small_units(p) <= (lq == 4 ? 2550 : p.B <= 54 ? 2900 : 1200);
}

// Forward with the spectra through LDS: where the lines of S that the
// LDS-free kernel reads piecemeal outweigh the barriers, and only with enough
// tiles to give most CUs a workgroup.  LDS-free -> through LDS, us: FP32 B = 128,
// 1 signal 144 -> 123, 2 signals 202 -> 132; B = 96, 1 signal 41 -> 46, 3 signals
// 62 -> 49; B = 64, 2 signals 14.9 -> 15.4, 8 signals 37 -> 30; B = 48 (142 tiles),
// 8 signals 15 -> 20.  FP64, whose products take twice as long and whose chunks
// hold half the nodes, B = 64, 2 signals 19 -> 22, 5 signals 43 -> 37; B = 96, 2 signals
// 102 -> 112, 3 signals 128 -> 118.
template <class T>
static bool small_through_lds(const BetaParams<T>& p) {
  return small_fills(p) && p.batch * small_units(p) >= (sizeof(T) == 4 ? 1000 : 1250);
}

template <class T, int MIR>
static hipError_t launch_forward_mid(const BetaParams<T>& p, const cpx<T>* S, cpx<T>* coeffs, hipStream_t s) {
  constexpr int BT = SmallCols<MIR>::BT;
  const int pos_end = MIR == 2 ? p.ntiles * PT / 2 : p.ntiles * PT;
  const int ntl = (pos_end - p.tile0 * PT + PT - 1) / PT, nbt = (p.batch + BT - 1) / BT;
  const dim3 grid(contraction_grid(ntl, nbt)), block(MID_THREADS);
  switch (beta_rtmax(p.B)) {
    case 1: hipLaunchKernelGGL((beta_forward_mid_kernel<T, 1, MIR>), grid, block, 0, s, S, coeffs, p, pos_end); break;
    case 2: hipLaunchKernelGGL((beta_forward_mid_kernel<T, 2, MIR>), grid, block, 0, s, S, coeffs, p, pos_end); break;
    default:  // above B = 64 every list is point-symmetric and every pair carries spectra
      if constexpr (MIR == 1) return hipErrorInvalidValue;
      else hipLaunchKernelGGL((beta_forward_mid_kernel<T, 4, MIR>), grid, block, 0, s, S, coeffs, p, pos_end);
  }
  return hipGetLastError();
}

template <class T, int MIR>
static hipError_t launch_forward_small(const BetaParams<T>& p, const cpx<T>* S, cpx<T>* coeffs, hipStream_t s) {
  constexpr int BT = SmallCols<MIR>::BT;
  const int pos_end = MIR == 2 ? p.ntiles * PT / 2 : p.ntiles * PT;
  const int ntl = (pos_end - p.tile0 * PT + PT - 1) / PT, nbt = (p.batch + BT - 1) / BT;
  const dim3 grid(contraction_grid(ntl, PT / SMALL_FWD_WAVES * nbt)), block(64 * SMALL_FWD_WAVES);
  switch (beta_rtmax(p.B)) {
    case 1: hipLaunchKernelGGL((beta_forward_small_kernel<T, 1, MIR>), grid, block, 0, s, S, coeffs, p, pos_end); break;
    case 2: hipLaunchKernelGGL((beta_forward_small_kernel<T, 2, MIR>), grid, block, 0, s, S, coeffs, p, pos_end); break;
    default:  // above B = 64 every list is point-symmetric and every pair carries spectra
      if constexpr (MIR == 1) return hipErrorInvalidValue;
      else hipLaunchKernelGGL((beta_forward_small_kernel<T, 4, MIR>), grid, block, 0, s, S, coeffs, p, pos_end);
  }
  return hipGetLastError();
}

template <class T, int LQ, int MIR>
static hipError_t launch_inverse_small_lq(const BetaParams<T>& p, const cpx<T>* coeffs, cpx<T>* S, hipStream_t s) {
  constexpr int BT = SmallCols<MIR>::BT;
  const int ntl = MIR == 2 ? (p.ntiles + 1) / 2 : p.ntiles - p.tile0, nbt = (p.batch + BT - 1) / BT;
  const int NB = (p.N + 15) / 16;
  const int blocks = small_inverse_blocks((long long)ntl * nbt, NB);
  const dim3 grid(contraction_grid(ntl, (NB + blocks - 1) / blocks * nbt)), block(SMALL_INV_THREADS);
  hipLaunchKernelGGL((beta_inverse_small_kernel<T, LQ, MIR>), grid, block, 0, s, coeffs, S, p, ntl, blocks);
  return hipGetLastError();
}

template <class T, int MIR>
static hipError_t launch_inverse_small(const BetaParams<T>& p, const cpx<T>* coeffs, cpx<T>* S, hipStream_t s) {
  switch (beta_lq(p.B)) {
    case 4: return launch_inverse_small_lq<T, 4, MIR>(p, coeffs, S, s);
    case 8: return launch_inverse_small_lq<T, 8, MIR>(p, coeffs, S, s);
    case 16:  // B > 64
      if constexpr (MIR == 2) return launch_inverse_small_lq<T, 16, MIR>(p, coeffs, S, s);
  }
  return hipErrorInvalidValue;
}

template <class T>
hipError_t launch_beta_forward_small(const BetaParams<T>& p, const cpx<T>* S, cpx<T>* coeffs, hipStream_t s) {
  if (small_mirrored(p))
    return small_through_lds(p) ? launch_forward_mid<T, 2>(p, S, coeffs, s) : launch_forward_small<T, 2>(p, S, coeffs, s);
  return small_through_lds(p) ? launch_forward_mid<T, 1>(p, S, coeffs, s) : launch_forward_small<T, 1>(p, S, coeffs, s);
}
template <class T>
hipError_t launch_beta_inverse_small(const BetaParams<T>& p, const cpx<T>* coeffs, cpx<T>* S, hipStream_t s) {
  return small_mirrored(p) ? launch_inverse_small<T, 2>(p, coeffs, S, s) : launch_inverse_small<T, 1>(p, coeffs, S, s);
}

template bool beta_small_forward<float>(const BetaParams<float>&);
template bool beta_small_forward<double>(const BetaParams<double>&);
template bool beta_small_inverse<float>(const BetaParams<float>&);
template bool beta_small_inverse<double>(const BetaParams<double>&);
template hipError_t launch_beta_forward_small<float>(const BetaParams<float>&, const cpx<float>*, cpx<float>*,
                                                     hipStream_t);
template hipError_t launch_beta_forward_small<double>(const BetaParams<double>&, const cpx<double>*, cpx<double>*,
                                                      hipStream_t);
template hipError_t launch_beta_inverse_small<float>(const BetaParams<float>&, const cpx<float>*, cpx<float>*,
                                                     hipStream_t);
template hipError_t launch_beta_inverse_small<double>(const BetaParams<double>&, const cpx<double>*, cpx<double>*,
                                                      hipStream_t);

}  // namespace su2

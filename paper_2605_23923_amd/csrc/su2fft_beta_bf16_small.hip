// The split-BF16 contractions (su2fft_beta_bf16.hip) for small batches: the same
// products in the same order, hence the same bits, with the columns of a
// 16-wide product 2 mirror pairs x 4 signals x (re, im) (su2fft_beta_small.h; one
// pair and 8 signals where mirrors carry no spectra), so that the table, most
// of the bytes, is read once per 4 signals and no column is empty.
#include "su2fft_beta_small.h"
#include "su2fft_bf16.h"

namespace su2 {

constexpr int BS_THREADS = 64 * PT;  // a wave per pair of a tile
constexpr int BS_KC = 32;            // nodes per matrix instruction

// A chunk's operands: 32 nodes of the table's RT row tiles, in the
// node-interleaved layout (a lane's 8 nodes are one aligned 32-byte load)
template <int RT>
struct BfRows {
  uint4 w[RT][2];
  // `src`: the wave's column block at this lane's node group; rows past L read
  // row L - 1 and are dropped at the end, node groups past the last are zero
  __device__ __forceinline__ void load(const unsigned* src, int L, int lrow, bool ok) {
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
      const uint4* r = reinterpret_cast<const uint4*>(src + 8 * min(rt * 16 + lrow, L - 1));
      w[rt][0] = ok ? r[0] : uint4{0, 0, 0, 0};
      w[rt][1] = ok ? r[1] : uint4{0, 0, 0, 0};
    }
  }
  __device__ __forceinline__ void products(const float (&v)[8], floatx4 (&acc)[RT]) const {
    u16x8 bhi, blo, ahi, alo;
    split8(v, bhi, blo);
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
      const unsigned a[8] = {w[rt][0].x, w[rt][0].y, w[rt][0].z, w[rt][0].w,
                             w[rt][1].x, w[rt][1].y, w[rt][1].z, w[rt][1].w};
      unpack8(a, ahi, alo);
      acc[rt] = mfma_bf16(ahi, bhi, acc[rt]);
      acc[rt] = mfma_bf16(ahi, blo, acc[rt]);
      acc[rt] = mfma_bf16(alo, bhi, acc[rt]);
    }
  }
};

// the sums of row tile rt, row i are degree 16 rt + i
template <int RT, int MIR>
__device__ __forceinline__ void store_forward_bf16(cpx<float>* __restrict__ coeffs, const BetaParams<float>& p,
                                                   const SmallPairs<float, MIR>& w, int b0, int lane,
                                                   const floatx4 (&acc)[RT]) {
  typedef SmallCols<MIR> Cols;
  const int col = lane & 15, b = b0 + Cols::sig(col);
  const auto q = w.pick(Cols::mir(col));
  if (b >= p.batch) return;
  float* out = reinterpret_cast<float*>(coeffs + coef_offset(p.coff, b, p.ncoef)) + (col & 1);
#pragma unroll
  for (int rt = 0; rt < RT; rt++)
#pragma unroll
    for (int r = 0; r < 4; r++)
      store_coef_small<float, MIR>(out, p, q, 16 * rt + 4 * (lane >> 4) + r, col & 1, acc[rt][r]);
}

// Forward, bound by the table and spectra bytes in flight: one workgroup of 16
// waves per pair tile (and its mirror tile), S in whole lines through LDS, a chunk of 32 nodes in each of two buffers; the
// table goes straight to registers.
template <int MIR>
struct BfMid {
  static constexpr int BT = SmallCols<MIR>::BT, PB = 2 * PT + 2;
  // a pad after 8 nodes: the wave's four node groups meet different banks
  static constexpr int HALF = BS_KC * BT * PB + 4 * 16 + 2;
  static constexpr int NV = MIR * BS_KC * BT * (PT / 2), VPT = NV / BS_THREADS;  // 16-byte pieces
  static_assert(NV % BS_THREADS == 0, "chunk split");
  __device__ static __forceinline__ int row(int kk, int bb) { return (kk * BT + bb) * PB + (kk >> 3) * 16; }
};

template <int RT, int MIR>
__device__ __forceinline__ void beta_forward_bf16_mid_body(const cpx<float>* __restrict__ S,
                                                           cpx<float>* __restrict__ coeffs,
                                                           const BetaParams<float>& p,
                                                           const unsigned* __restrict__ tabf,
                                                           const SmallPairs<float, MIR>& w, int tile, int b0,
                                                           float* lds, int wave, int lane) {
  typedef SmallCols<MIR> Cols;
  typedef BfMid<MIR> M;
  constexpr int BT = M::BT;
  const int lrow = lane & 15, lg = lane >> 4, N = p.N, NB8 = (N + 7) / 8, tid = wave * 64 + lane;
  const int nb = min(BT, p.batch - b0), nchunk = (N + BS_KC - 1) / BS_KC;
  const bool work = w.L > 0;

  float4 sv[M::VPT];
  auto fetch_s = [&](int c) {
#pragma unroll
    for (int i = 0; i < M::VPT; i++) {
      const int v = tid + BS_THREADS * i, pv = v % (PT / 2), bb = v / (PT / 2) % BT, kk = v / (PT / 2 * BT) % BS_KC;
      const int mir = v / (PT / 2 * BT * BS_KC), k = c * BS_KC + kk, t = mir ? p.ntiles - 1 - tile : tile;
      sv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < N && bb < nb)
        sv[i] = *reinterpret_cast<const float4*>(S + (((size_t)t * N + k) * p.batch + b0 + bb) * PT + 2 * pv);
    }
  };
  auto commit_s = [&](int c) {
    float* d = lds + (c & 1) * MIR * M::HALF;
#pragma unroll
    for (int i = 0; i < M::VPT; i++) {
      const int v = tid + BS_THREADS * i, pv = v % (PT / 2), bb = v / (PT / 2) % BT, kk = v / (PT / 2 * BT) % BS_KC;
      const int mir = v / (PT / 2 * BT * BS_KC);
      float* e = d + mir * M::HALF + M::row(kk, bb) + 4 * pv;
      e[0] = sv[i].x; e[1] = sv[i].y; e[2] = sv[i].z; e[3] = sv[i].w;
    }
  };
  const unsigned* ta = tabf + w.tab / N * NB8 * 8 + ((long long)lg * w.lsum + w.coff) * 8;
  const long long sa = 4LL * w.lsum * 8;
  BfRows<RT> a;
  auto fetch_a = [&](int c) {
    if (work) a.load(4 * c + lg < NB8 ? ta + c * sa : ta, w.L, lrow, 4 * c + lg < NB8);
  };
  const int hm = MIR == 2 ? Cols::mir(lrow) : 0;
  const int bofs = hm * M::HALF + M::row(8 * lg, Cols::sig(lrow)) + 2 * (hm ? PT - 1 - wave : wave) + (lrow & 1);

  floatx4 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; rt++) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
  fetch_s(0);
  fetch_a(0);
  commit_s(0);
  __syncthreads();
  for (int c = 0; c < nchunk; c++) {
    if (c + 1 < nchunk) fetch_s(c + 1);
    const float* src = lds + (c & 1) * MIR * M::HALF + bofs;
    if (work) {
      float v[8];
#pragma unroll
      for (int q = 0; q < 8; q++) v[q] = src[q * BT * M::PB];
      a.products(v, acc);
    }
    if (c + 1 < nchunk) {
      fetch_a(c + 1);
      commit_s(c + 1);
    }
    __syncthreads();
  }
  if (work) store_forward_bf16<RT, MIR>(coeffs, p, w, b0, lane, acc);
}

template <int RTMAX, int MIR>
__global__ __launch_bounds__(BS_THREADS) void beta_forward_bf16_mid_kernel(const cpx<float>* __restrict__ S,
                                                                           cpx<float>* __restrict__ coeffs,
                                                                           BetaParams<float> p,
                                                                           const unsigned* __restrict__ tabf, int ntl) {
  typedef BfMid<MIR> M;
  __shared__ __align__(16) float lds[2 * MIR * M::HALF];
  const TileSlot sl = contraction_slot(blockIdx.x, ntl, (p.batch + M::BT - 1) / M::BT);
  if (!sl.valid) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tile = p.tile0 + sl.tile, b0 = sl.bt * M::BT;
  SmallPairs<float, MIR> w(p, tile * PT + wave);
  if (MIR == 2 && p.ntiles - 1 - tile == tile) {
    // the self-mirror tile stores both columns of a couple: each pair reads its
    // own, as in the tile kernel (these products do not round alike under a
    // change of sign: a handful of 16206 coefficients differed at B = 36)
    w.L = w.q0.L;
    w.q1.L = 0;
  }
  // row tiles of the workgroup's longest pair: one branch for all its waves
  // (barriers inside)
  int rt = 1;
  if constexpr (RTMAX > 1) {
    int L = 0;
    for (int i = 0; i < PT; i++) L = max(L, p.pairs[tile * PT + i].L);
    rt = (L + 15) / 16;
  }
  if constexpr (RTMAX >= 4) {
    if (rt >= 4) return beta_forward_bf16_mid_body<4, MIR>(S, coeffs, p, tabf, w, tile, b0, lds, wave, lane);
    if (rt == 3) return beta_forward_bf16_mid_body<3, MIR>(S, coeffs, p, tabf, w, tile, b0, lds, wave, lane);
  }
  if constexpr (RTMAX >= 2)
    if (rt == 2) return beta_forward_bf16_mid_body<2, MIR>(S, coeffs, p, tabf, w, tile, b0, lds, wave, lane);
  beta_forward_bf16_mid_body<1, MIR>(S, coeffs, p, tabf, w, tile, b0, lds, wave, lane);
}

// Inverse / adjoint: one workgroup of 16 waves per pair tile (and its mirror
// tile) and range of 16-node blocks; a wave's split, scaled coefficients are
// its B operands.  A block's rows are gathered in LDS and written as whole
// PT-pair rows of S.  The table's 8 words per lane come in two 16-byte loads: as
// eight loads they pass over more lines than the L1 holds between them (B = 64,
// 8 signals 69 -> 28 us).
template <int LQ, int MIR>
__global__ __launch_bounds__(BS_THREADS) void beta_inverse_bf16_small_kernel(const cpx<float>* __restrict__ coeffs,
                                                                             cpx<float>* __restrict__ S,
                                                                             BetaParams<float> p,
                                                                             const unsigned* __restrict__ tabi,
                                                                             int ntl, int blocks) {
  typedef SmallCols<MIR> Cols;
  constexpr int BT = Cols::BT;
  typedef SmallStage<float, BT> ST;
  __shared__ __align__(16) float stages[2][MIR * 16 * ST::NRS];
  const int N = p.N, NB = (N + 15) / 16, nsplit = (NB + blocks - 1) / blocks;
  const int nbt = (p.batch + BT - 1) / BT;
  const TileSlot sl = contraction_slot(blockIdx.x, ntl, nsplit * nbt);
  if (!sl.valid) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lrow = lane & 15, lg = lane >> 4;
  const int tile = p.tile0 + sl.tile, b0 = sl.bt / nsplit * BT;
  const int kb0 = sl.bt % nsplit * blocks, kb1 = min(NB, kb0 + blocks);
  const int nb = min(BT, p.batch - b0);
  const SmallPairs<float, MIR> w(p, tile * PT + wave);
  const int L = w.L;

  // table words of a block: 8 consecutive degrees of node 16 kb + lrow (rows
  // past N read row N - 1 and are never stored; degrees past L read the words
  // that follow in the block, or the zeroed table padding, and meet zeros)
  const unsigned* tb = tabi + w.tab + w.coff + 8 * lg;
  word4 aw[LQ][2];
  auto fetch = [&](int kb) {
    const unsigned* trow = tb + (long long)min(16 * kb + lrow, N - 1) * w.lsum;
#pragma unroll
    for (int s = 0; s < LQ; s++) {
      if (32 * s < L) {  // wave-uniform branch
        aw[s][0] = *reinterpret_cast<const word4*>(trow + 32 * s);
        aw[s][1] = *reinterpret_cast<const word4*>(trow + 32 * s + 4);
      }
    }
  };
  fetch(kb0);  // in flight while the coefficients are gathered

  const int mir = MIR == 2 ? Cols::mir(lrow) : 0, sig = Cols::sig(lrow);
  u16x8 bhi[LQ], blo[LQ];
  {
    const auto q = w.pick(mir);
    const float* c =
        reinterpret_cast<const float*>(coeffs + coef_offset(p.coff, b0 + min(sig, nb - 1), p.ncoef)) + (lrow & 1);
#pragma unroll
    for (int s = 0; s < LQ; s++) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; i++) v[i] = load_coef_small<float, MIR>(c, p, q, 32 * s + 8 * lg + i, lrow & 1, sig < nb);
      split8(v, bhi[s], blo[s]);
    }
  }

  float* const mine = stages[0] + mir * 16 * ST::NRS + sig * ST::PB + 2 * (mir ? PT - 1 - wave : wave) + (lrow & 1);
  for (int kb = kb0; kb < kb1; kb++) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < LQ; s++)
      if (32 * s < L) {
        u16x8 ahi, alo;
        unpack8(aw[s], ahi, alo);
        acc = mfma_bf16(ahi, bhi[s], acc);
        acc = mfma_bf16(ahi, blo[s], acc);
        acc = mfma_bf16(alo, bhi[s], acc);
      }
    if (kb + 1 < kb1) fetch(kb + 1);  // next block's words, in flight during the stores
    // two stage buffers in turn: one barrier per block
#pragma unroll
    for (int r = 0; r < 4; r++) mine[(kb & 1) * MIR * 16 * ST::NRS + (4 * lg + r) * ST::NRS] = acc[r];
    __syncthreads();
    store_rows_small<float, MIR, BS_THREADS>(S, p, stages[kb & 1], tile, kb, b0, nb, tid);
  }
}

// Forward: this kernel instead of the tile kernel where its grid of tiles and
// 16-signal groups leaves CUs idle or columns empty: by signals times tiles, further
// with one row tile of degrees (B <= 32); with a tile per CU or more, by signals.
// Whole calls on inputs not in the caches, tile kernel -> this, us: B = 32,
// 32 signals 38.7 -> 35.2 (the contraction alone at 64 signals, the last of this
// kernel's gain: 24.9 -> 19.4 before the tile kernel ran two workgroups per CU);
// B = 36, 20 signals 44.5 -> 43.3 (alone at 48 signals 23 -> 29); B = 48, 12 signals
// 58.8 -> 57.5; B = 54, 8 signals 71 -> 68 (alone at 12 signals 25.4 -> 27.0);
// B = 64, 4 signals 50 -> 40, 8 signals 76 -> 73 (alone at 9 signals 30.9 -> 32.0);
// alone: B = 72, 12 signals 73 -> 48 (16 signals 65 on the tile kernel); B = 96,
// 12 signals 169 -> 133; B = 128, 1 signal 297 -> 113 (the table takes 68 at the copy
// rate), 8 signals 341 -> 254, 12 signals 360 (tile kernel at 13: 361).
bool beta_bf16_small_forward(const BetaParams<float>& p) {
  if (small_fills(p)) return p.batch <= (p.B > 64 && p.B <= 108 ? 12 : 8);
  return p.batch * small_units(p) <= (beta_rtmax(p.B) == 1 ? 2500 : 1800);
}

// Inverse: likewise; further where the 32-degree products of the tile kernel
// are partly empty (B <= 54), less far in half-spectrum plans, whose waves hold one
// pair.  Whole calls: B = 24, 100 signals 51 -> 47; B = 32, 60 signals 67.1 -> 67.1;
// B = 36, 44 signals 80 -> 76; B = 54, 20 signals 162 -> 156; B = 64, 4 signals
// 59 -> 42, 8 signals 85 -> 80; B = 72, 12 signals 258 -> 238; B = 128, 8 signals
// 915 -> 850.  Alone: SO(3) B = 64, 16 signals 29.9 -> 27.1, 24 signals 38.2 -> 42.0;
// B = 64, 9 signals 37.8 -> 38.3; B = 128, 1 signal 297 -> 122, 12 signals 418 -> 440.
// Half-spectrum whole calls: B = 16, 55 signals 21.1 -> 18.5; B = 32, whose second group
// of 8 signals fills the CUs twice, 8 signals 26.4 -> 20.6, 9 signals 26.7 -> 28.0.
bool beta_bf16_small_inverse(const BetaParams<float>& p) {
  if (small_fills(p)) return p.batch <= (p.B > 64 && p.B <= 96 ? 12 : 8);
  if (!small_mirrored(p)) return p.batch * small_units(p) <= (p.B <= 16 ? 1000 : 520);
  return p.batch * small_units(p) <= (p.B <= 54 ? 4000 : 2200);
}

template <int RTMAX, int MIR>
static hipError_t launch_forward_bf16_mid(const BetaParams<float>& p, const unsigned* tabf, const cpx<float>* S,
                                          cpx<float>* coeffs, hipStream_t s) {
  constexpr int BT = SmallCols<MIR>::BT;
  const int ntl = MIR == 2 ? (p.ntiles + 1) / 2 : p.ntiles - p.tile0, nbt = (p.batch + BT - 1) / BT;
  hipLaunchKernelGGL((beta_forward_bf16_mid_kernel<RTMAX, MIR>), dim3(contraction_grid(ntl, nbt)), dim3(BS_THREADS), 0,
                     s, S, coeffs, p, tabf, ntl);
  return hipGetLastError();
}
template <int RTMAX>
static hipError_t launch_forward_bf16(const BetaParams<float>& p, const unsigned* tabf, const cpx<float>* S,
                                      cpx<float>* coeffs, hipStream_t s) {
  if (small_mirrored(p)) return launch_forward_bf16_mid<RTMAX, 2>(p, tabf, S, coeffs, s);
  // above B = 64 every list is point-symmetric and every pair carries spectra
  if constexpr (RTMAX <= 2) return launch_forward_bf16_mid<RTMAX, 1>(p, tabf, S, coeffs, s);
  return hipErrorInvalidValue;
}

template <int LQ, int MIR>
static hipError_t launch_inverse_bf16(const BetaParams<float>& p, const unsigned* tabi, const cpx<float>* coeffs,
                                      cpx<float>* S, hipStream_t s) {
  constexpr int BT = SmallCols<MIR>::BT;
  const int ntl = MIR == 2 ? (p.ntiles + 1) / 2 : p.ntiles - p.tile0, nbt = (p.batch + BT - 1) / BT;
  const int NB = (p.N + 15) / 16, blocks = small_inverse_blocks((long long)ntl * nbt, NB);
  hipLaunchKernelGGL((beta_inverse_bf16_small_kernel<LQ, MIR>),
                     dim3(contraction_grid(ntl, (NB + blocks - 1) / blocks * nbt)), dim3(BS_THREADS), 0, s, coeffs, S, p,
                     tabi, ntl, blocks);
  return hipGetLastError();
}

hipError_t launch_beta_forward_bf16_small(const BetaParams<float>& p, const unsigned* tabf, const cpx<float>* S,
                                          cpx<float>* coeffs, hipStream_t s) {
  switch (beta_rtmax(p.B)) {
    case 1: return launch_forward_bf16<1>(p, tabf, S, coeffs, s);
    case 2: return launch_forward_bf16<2>(p, tabf, S, coeffs, s);
    default: return launch_forward_bf16<4>(p, tabf, S, coeffs, s);
  }
}
hipError_t launch_beta_inverse_bf16_small(const BetaParams<float>& p, const unsigned* tabi, const cpx<float>* coeffs,
                                          cpx<float>* S, hipStream_t s) {
  if (beta_bf16_lq(p.B) == 1)
    return small_mirrored(p) ? launch_inverse_bf16<1, 2>(p, tabi, coeffs, S, s)
                             : launch_inverse_bf16<1, 1>(p, tabi, coeffs, S, s);
  return small_mirrored(p) ? launch_inverse_bf16<2, 2>(p, tabi, coeffs, S, s) : hipErrorInvalidValue;  // B > 64
}

}  // namespace su2

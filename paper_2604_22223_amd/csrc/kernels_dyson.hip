// Dyson equations.
//
// Screened interaction (Eq. eq-screened-coulomb): for every (bosonic node,
// q) solve (I - V P) W = V and return W^C = W - V.  Gauss-Jordan elimination
// with partial pivoting on the augmented system [I - V P | V], two lanes per
// row: lane (row, half 0) holds the row of I - V P, lane (row, half 1) the row
// of V, so a row costs 2 x N_b registers-worth of complex values spread over
// two lanes.  Both halves run the same instruction stream on different
// columns (no divergence): the pivot row is found by a segmented arg-max
// over the unused rows (ties go to the lower row) and broadcast through LDS;
// every row is updated as x <- x - f * pivot_row, with f = a_rs / a_ps for the
// other rows and f = 1 - 1 / a_ps for the pivot row itself (which normalises
// it).  At the end the half-1 lane of the row that pivoted column s holds row
// s of W.
//
// Green's function (Eq. full-green-freq): one thread per (fermionic node, k)
// inverts the n_o x n_o matrix (i w + mu) - H(k) - Sigma(k, i w) in registers
// (in-place Gauss-Jordan with partial pivoting).  The chemical potential for
// the target filling comes from a safeguarded Newton iteration on
// N_e(mu) = -2/N_k sum_{k,m} Re rho_m Tr G(k, i w_m), with
// dN_e/dmu = 2/N_k sum Re rho_m Tr G^2 (dG/dmu = -G^2): steps stay inside the
// sign-change bracket once one is known (bisection otherwise) and are capped
// before.  Each evaluation is one launch that writes per-block partial sums;
// a one-block launch sums them in a fixed order and takes the step, so the
// search is deterministic and needs no grid-wide barrier.
#include <algorithm>
#include <cmath>
#include <utility>

#include "qgw_gj.h"
#include "qgw_internal.h"
#include "qgw_mfma.h"

namespace qgw {

constexpr int pow2_ceil(int n) {
  int p = 1;
  while (p < n) p *= 2;
  return p;
}

// ---------------------------------------------------------------------------
// W^C = (I - V P)^{-1} V - V
// ---------------------------------------------------------------------------
template <int NB>
struct DysonWShape {
  static constexpr int SEG = pow2_ceil(NB);     // lanes per half
  static constexpr int LPM = 2 * SEG;           // lanes per matrix
  static constexpr int MPW = 64 / LPM;          // matrices per block (one wavefront)
  static constexpr int NN = NB * NB;
  static constexpr int SPLIT = (NB + 1) / 2;    // columns of I - V P formed by each half
};

template <typename T>
__device__ __forceinline__ cpx<T> shfl_cpx(cpx<T> v, int src, int width) {
  return mk(__shfl(v.re, src, width), __shfl(v.im, src, width));
}

template <int NB, typename T>
__global__ __launch_bounds__(64) void k_dyson_w(const cpx<T>* __restrict__ vq,
                                                const cpx<T>* __restrict__ pnu,
                                                cpx<T>* __restrict__ wc, int64_t nmat, int nk, int64_t ld,
                                                int* __restrict__ cond) {
  using S = DysonWShape<NB>;
  static_assert(S::SEG <= 32, "a row index must fit the five low bits of a pivot key");
  __shared__ cpx<T> sp[S::MPW * S::NN];
  __shared__ cpx<T> piv[2][S::MPW][2 * NB];
  const int lane = threadIdx.x;
  const int mw = lane / S::LPM;
  const int half = (lane / S::SEG) & 1;
  const int row = lane % S::SEG;
  const int64_t mat0 = int64_t(blockIdx.x) * S::MPW;
  const int64_t mat = mat0 + mw;
  const bool valid = (mat < nmat) && (row < NB);
  const int q = int(valid ? mat % nk : 0);
  const int64_t nload = (nmat - mat0 < S::MPW ? nmat - mat0 : S::MPW) * S::NN;
  for (int e = lane; e < S::MPW * S::NN; e += 64) sp[e] = e < nload ? pnu[mat0 * S::NN + e] : mk(T(0), T(0));
  __syncthreads();
  const cpx<T>* vrow = vq + (int64_t(q) * NB + (row < NB ? row : 0)) * NB;
  cpx<T>* pm = sp + mw * S::NN;
  // I - V P, formed in place of P: in round g, half h forms columns
  // [8 g + 4 h, 8 g + 4 h + 4) of its row; once every lane has read those
  // columns of P they are overwritten by the columns of I - V P.
  constexpr int CW = 4;
#pragma unroll
  for (int g = 0; g < (NB + 2 * CW - 1) / (2 * CW); ++g) {
    const int c0 = (2 * g + half) * CW;
    cpx<T> acc[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) acc[c] = mk(T(row == c0 + c ? 1 : 0), T(0));
    if (valid && c0 < NB) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const cpx<T> v = vrow[j];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          const int col = c0 + c < NB ? c0 + c : NB - 1;
          acc[c] = fms(acc[c], v, pm[j * NB + col]);
        }
      }
    }
    __syncthreads();
    if (valid) {
#pragma unroll
      for (int c = 0; c < CW; ++c)
        if (c0 + c < NB) pm[row * NB + c0 + c] = acc[c];
    }
  }
  __syncthreads();
  cpx<T> x[NB];
  if (valid) {
    if (half == 0) {
#pragma unroll
      for (int c = 0; c < NB; ++c) x[c] = pm[row * NB + c];
    } else {
#pragma unroll
      for (int c = 0; c < NB; ++c) x[c] = vrow[c];
    }
  } else {
#pragma unroll
    for (int c = 0; c < NB; ++c) x[c] = mk(T(0), T(0));
  }
  bool used = false, singular = false;
  int my_step = 0;
  const int partner = lane - half * S::SEG;  // the half-0 lane of this row
#pragma unroll
  for (int s = 0; s < NB; ++s) {
    // the candidates' keys (|Re| + |Im| in FP32 bits, low bits 31 - row: ties go to the lower row) reduced by DPP
    // row shifts over the SEG lanes of half 0 into its first lane (of each 16-lane DPP row), then sent to the
    // matrix's lanes
    int key = (valid && half == 0 && !used) ? ((mag_bits(x[s]) & ~31) | (31 - row)) : int(0x80000000u);
    if constexpr (S::SEG >= 16) key = max(key, dpp_shl_i<0x108>(key));
    if constexpr (S::SEG >= 8) key = max(key, dpp_shl_i<0x104>(key));
    if constexpr (S::SEG >= 4) key = max(key, dpp_shl_i<0x102>(key));
    if constexpr (S::SEG >= 2) key = max(key, dpp_shl_i<0x101>(key));
    if constexpr (S::SEG == 32)  // half 0 spans two DPP rows (one matrix per wave)
      key = max(__builtin_amdgcn_readlane(key, 0), __builtin_amdgcn_readlane(key, 16));
    else
      key = __shfl(key, mw * S::LPM, 64);
    const int idx = 31 - (key & 31);
    const bool is_p = valid && (row == idx);
    if (is_p) {
      if (half == 0) used = true;
      my_step = s;
#pragma unroll
      for (int c = 0; c < NB; ++c) piv[s & 1][mw][half * NB + c] = x[c];
    }
    __syncthreads();
    const cpx<T>* pr = piv[s & 1][mw] + half * NB;
    const cpx<T> pv = piv[s & 1][mw][s];
    const T pn = norm2(pv);
    singular |= !(pn > T(0)) || !isfinite(pn);  // exact zero, NaN or overflow
    const T d = rcp_nr(pn);
    const cpx<T> pinv = mk(pv.re * d, -pv.im * d);
    cpx<T> f = is_p ? mk(T(1), T(0)) - pinv : x[s] * pinv;  // meaningful on half 0
    f = shfl_cpx(f, partner, 64);
    if (valid) {
#pragma unroll
      for (int c = 0; c < NB; ++c) x[c] = fms(x[c], f, pr[c]);
      if (half == 0) x[s] = mk(T(is_p ? 1 : 0), T(0));
    }
  }
  // a singular or non-finite system of an existing matrix raises the condition bit (the output is non-finite)
  if (singular && mat < nmat && row == 0 && half == 0) atomicOr(cond, kCondSingular);
  // W^C row my_step = (row of W) - (row of V); staged in LDS, stored contiguously
  __syncthreads();
  if (valid && half == 1) {
    const cpx<T>* vr = vq + (int64_t(q) * NB + my_step) * NB;
#pragma unroll
    for (int c = 0; c < NB; ++c) sp[mw * S::NN + my_step * NB + c] = x[c] - vr[c];
  }
  __syncthreads();
  for (int e = lane; e < nload; e += 64) {
    const int mi = e / S::NN;
    wc[(mat0 + mi) * ld + (e - mi * S::NN)] = sp[e];
  }
}

// ---------------------------------------------------------------------------
// Register-blocked form of the same solve for N_b = 25 (the five-orbital
// product basis).  One wavefront per (node, q) matrix.  The augmented system
// [I - V P | V] is 25 x 50; its columns are numbered 0..24 for I - V P and
// 25..49 for V (56 with zero padding).  Lane = rg + 8 cg holds
//  * rows rg + 8 s (s < 3, rows 0..23) in columns cg + 8 t (t < 7), and
//  * one entry of row 24, column cg + 8 rg,
// so the last row costs one register pair per lane instead of a mostly empty
// fourth row slot.
//  * V P is formed in that layout: per summation index j a lane reads 3
//    values of V (rows rg + 8 s sit in distinct banks), V(24, j) (one
//    address) and 4 + 1 values of P, and does 13 complex multiply-adds.  P
//    is staged in LDS seven rows at a time, each chunk read into registers
//    while the previous one is used.
//  * Gauss-Jordan step K (a compile-time constant): the lanes holding column
//    K rank their unused rows by |Re| + |Im|, rounded to FP32 and packed with
//    31 - row into one 32-bit key (ties go to the lower row); three DPP
//    shifts inside the 8-lane group and one readlane give the pivot row p.
//    The owners of row p publish it, the owners of column K publish the
//    multipliers (the pivot's own entry less one), and every lane subtracts
//    f_r * (pivot row) with f_r = m_r / a_pK, which normalises the pivot
//    row and clears column K in every other row.
//  * Columns of I - V P left of K are never read again, so a slot whose
//    columns are all <= K drops out of the update.
// LDS holds V (10,000 bytes in FP64) and a 3,072-byte area shared by the P
// chunks and the pivot exchange (two buffers, alternating by step): twelve
// blocks fit a CU.
// ---------------------------------------------------------------------------
struct W25 {
  static constexpr int NB = 25, NS = 3, NT = 7;
  static constexpr int CH = 7;                   // rows of P per staged chunk
  static constexpr int NCH = (NB + CH - 1) / CH;
  static constexpr int ROW = 64;                 // pivot row: 56 columns and 8 zeros
  static constexpr int EX = ROW + 32;            // pivot row and multipliers of one step
  static constexpr int XS = 2 * EX;              // area shared by the P chunks and the pivot exchange
  static constexpr int MIN = int(0x80000000u);
};
static_assert(W25::CH * W25::NB <= W25::XS, "a chunk of P must fit the exchange area");

// The owners of pivot row p = rg + 8 S (S < 3) publish it from the slot
// holding column K on, mark the row as used and record the step; the owner
// of a_pK also stores a_pK - 1 as the pivot row's multiplier.
template <typename T, int K, int S>
__device__ __forceinline__ void gj25_publish(const cpx<T> (&x)[3][7], cpx<T>* xs, int cg, int p, int (&cs)[3],
                                             int (&kof)[3]) {
  constexpr int tk = K / 8;
  xs += (K & 1) * W25::EX;
#pragma unroll
  for (int t = tk; t < W25::NT; ++t) xs[cg + 8 * t] = x[S][t];
  if (cg == K % 8) xs[W25::ROW + p] = mk(x[S][tk].re - T(1), x[S][tk].im);
  cs[S] |= W25::MIN;
  kof[S] = K;
}

// cs[s] = 31 - row for a candidate row, with the sign bit set once the row
// has pivoted, so that a set sign drops it from the max
template <typename T, int K>
__device__ __forceinline__ void gj25_step(cpx<T> (&x)[3][7], cpx<T>& y, int (&cs)[3], int (&kof)[3], int& k24,
                                          int rg, int cg, cpx<T>* xs, bool& singular) {
  constexpr int NS = W25::NS, NT = W25::NT, ROW = W25::ROW, MIN = W25::MIN;
  constexpr int cgk = K % 8, tk = K / 8, t0 = (K + 1) / 8;
  const bool used24 = k24 >= 0;
  int key = (!used24 && rg == tk) ? ((mag_bits(y) & ~31) | (31 - 24)) : MIN;
#pragma unroll
  for (int s = 0; s < NS; ++s) key = max(key, (mag_bits(x[s][tk]) & ~31) | cs[s]);
  key = cg == cgk ? key : MIN;
  key = max(key, dpp_shl_i<0x104>(key));
  key = max(key, dpp_shl_i<0x102>(key));
  key = max(key, dpp_shl_i<0x101>(key));
  const int p = 31 - (__builtin_amdgcn_readlane(key, cgk * 8) & 31);
  const int rgp = p & 7, sp = p >> 3;
  cpx<T>* ex = xs + (K & 1) * W25::EX;  // exchange buffers alternate by step parity
  cpx<T>* mu = ex + ROW;
  if (cg == cgk) {
#pragma unroll
    for (int s = 0; s < NS; ++s) mu[rg + 8 * s] = x[s][tk];
    if (rg == tk) mu[24] = y;
  }
  if (p == 24) {
    if (rg < 7) ex[cg + 8 * rg] = y;
    if (rg == tk && cg == cgk) mu[24] = mk(y.re - T(1), y.im);
    k24 = K;
  } else if (rg == rgp) {
    if (sp == 0)
      gj25_publish<T, K, 0>(x, xs, cg, p, cs, kof);
    else if (sp == 1)
      gj25_publish<T, K, 1>(x, xs, cg, p, cs, kof);
    else
      gj25_publish<T, K, 2>(x, xs, cg, p, cs, kof);
  }
  __syncthreads();
  const cpx<T> pv = ex[K];
  const T pn = norm2(pv);
  singular |= !(pn > T(0)) || !isfinite(pn);  // exact zero, NaN or overflow (the same value in every lane)
  const T d = rcp_nr(pn);
  const cpx<T> pinv = mk(pv.re * d, -pv.im * d);
  cpx<T> f[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) f[s] = mu[rg + 8 * s] * pinv;
  y = fms(y, mu[24] * pinv, ex[cg + 8 * rg]);
#pragma unroll
  for (int t = t0; t < NT; ++t) {
    const cpx<T> pc = ex[cg + 8 * t];
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s][t] = fms(x[s][t], f[s], pc);
  }
}

template <typename T, int... K>
__device__ __forceinline__ void gj25_all(cpx<T> (&x)[3][7], cpx<T>& y, int (&cs)[3], int (&kof)[3], int& k24, int rg,
                                         int cg, cpx<T>* xs, bool& singular, std::integer_sequence<int, K...>) {
  (gj25_step<T, K>(x, y, cs, kof, k24, rg, cg, xs, singular), ...);
}

// MVP: V P on the matrix cores (16x16x4, 2 x 2 tiles over the 25 x 25 product, 7 slices of 4 along the
// contraction; rows, columns and slices past 25 are zero), V from LDS as the A operand and P straight from memory
// as the B operand; I - V P then passes through the V area of LDS into the elimination layout, and the final
// W - V reads V(q) from memory again.  The matrix cores run beside the VALU elimination of the other waves of
// the SIMD and the product no longer streams V and P through LDS, but on gfx950 the FP64 matrix rate equals the
// VALU rate and the 32 x 32 x 28 padding costs 1.8x the product's flops: measured at 24 x 24, r = 53 it takes
// 0.46 ms (FP64) and 0.27 ms (FP32) against 0.42 and 0.25 for the VALU product, so it is an autotuner
// alternative and not the default.
// one matrix; xs: a chunk of P rows, then the pivot exchange; sv: V(q)
template <typename T, bool MVP>
__device__ __forceinline__ void w25_solve(const cpx<T>* __restrict__ vq, const cpx<T>* __restrict__ pnu,
                                          cpx<T>* __restrict__ wc, int64_t mat, int nk, int64_t ld,
                                          int* __restrict__ cond, cpx<T>* xs, cpx<T>* sv) {
  constexpr int NB = W25::NB, NN = NB * NB, NS = W25::NS, NT = W25::NT, CH = W25::CH, NCH = W25::NCH;
  const int lane = threadIdx.x;
  const int rg = lane & 7, cg = lane >> 3;
  const int c24 = cg + 8 * rg;  // this lane's column of row 24
  const int q = int(mat % nk);
  const cpx<T>* vm = vq + int64_t(q) * NN;
  const cpx<T>* pm = pnu + mat * NN;
  // chunk c of P (rows CH c ..) is read into registers one chunk ahead; a
  // chunk has at most 175 entries, three per lane
  static_assert(CH * NB <= 3 * 64, "a chunk of P must fit three entries per lane");
  cpx<T> x[NS][NT], y;
  if constexpr (MVP) {
    using M = Mfma<T>;
    using v4 = typename M::v4;
    const int l16 = lane & 15, l4 = lane >> 4;
    for (int e = lane; e < NN; e += 64) sv[e] = vm[e];
    // B operand of slice ks, column tile ct: P[4 ks + l4][16 ct + l16]
    auto ldp = [&](int ks, int ct) -> cpx<T> {
      const int k = 4 * ks + l4, n = 16 * ct + l16;
      return (k < NB && n < NB) ? pm[k * NB + n] : mk(T(0), T(0));
    };
    v4 cr[2][2], ci[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        cr[a][b] = v4{T(0), T(0), T(0), T(0)};
        ci[a][b] = v4{T(0), T(0), T(0), T(0)};
      }
    cpx<T> b0 = ldp(0, 0), b1 = ldp(0, 1);
    __syncthreads();  // V(q) is in LDS
#pragma unroll 1
    for (int ks = 0; ks < 7; ++ks) {
      const cpx<T> pb[2] = {b0, b1};
      if (ks + 1 < 7) {
        b0 = ldp(ks + 1, 0);
        b1 = ldp(ks + 1, 1);
      }
      const int k = 4 * ks + l4;
      cpx<T> a[2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const int m = 16 * rt + l16;
        a[rt] = (k < NB && m < NB) ? sv[m * NB + k] : mk(T(0), T(0));
      }
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          cr[rt][ct] = M::mac(a[rt].re, pb[ct].re, cr[rt][ct]);
          ci[rt][ct] = M::mac(a[rt].re, pb[ct].im, ci[rt][ct]);
        }
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          cr[rt][ct] = M::mac(-a[rt].im, pb[ct].im, cr[rt][ct]);
          ci[rt][ct] = M::mac(a[rt].im, pb[ct].re, ci[rt][ct]);
        }
    }
    __syncthreads();  // every lane has finished reading V: its area takes A = I - V P
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * rt + M::row(lane, v), col = 16 * ct + l16;
          if (row < NB && col < NB)
            sv[row * NB + col] = mk(T(row == col ? 1 : 0) - cr[rt][ct][v], -ci[rt][ct][v]);
        }
    __syncthreads();
    // A from LDS and the right-hand side V from memory into the elimination layout
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int row = rg + 8 * s;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int c = cg + 8 * t;
        cpx<T> val = mk(T(0), T(0));
        if (t < 4 && c < NB)
          val = sv[row * NB + c];
        else if (c >= NB && c < 2 * NB)
          val = vm[row * NB + c - NB];
        x[s][t] = val;
      }
    }
    y = mk(T(0), T(0));
    if (c24 < NB)
      y = sv[24 * NB + c24];
    else if (c24 < 2 * NB)
      y = vm[24 * NB + c24 - NB];
  } else {
  cpx<T> pre0 = mk(T(0), T(0)), pre1 = pre0, pre2 = pre0;
  auto load_chunk = [&](int c) {
    const int n = min(CH, NB - CH * c) * NB;
    const cpx<T>* src = pm + CH * c * NB;
    if (lane < n) pre0 = src[lane];
    if (lane + 64 < n) pre1 = src[lane + 64];
    if (lane + 128 < n) pre2 = src[lane + 128];
  };
  load_chunk(0);
  for (int e = lane; e < NN; e += 64) sv[e] = vm[e];
  {
    // V P on the columns of I - V P: slots t < 3, t = 3 where cg = 0 (column
    // 24), and row 24 at column c24 < 25
    cpx<T> acc[NS][4], a24 = mk(T(0), T(0));
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[s][t] = mk(T(0), T(0));
    const int j24 = min(c24, NB - 1);
#pragma unroll 1
    for (int c = 0; c < NCH; ++c) {
      const int rows = min(CH, NB - CH * c);
      __syncthreads();  // the previous chunk has been read
      if (lane < rows * NB) xs[lane] = pre0;
      if (lane + 64 < rows * NB) xs[lane + 64] = pre1;
      if (lane + 128 < rows * NB) xs[lane + 128] = pre2;
      if (c + 1 < NCH) load_chunk(c + 1);
      __syncthreads();
#pragma unroll
      for (int jj = 0; jj < CH; ++jj) {
        if (jj < rows) {
          const int j = CH * c + jj;
          cpx<T> v[NS], pj[4];
#pragma unroll
          for (int s = 0; s < NS; ++s) v[s] = sv[(rg + 8 * s) * NB + j];
#pragma unroll
          for (int t = 0; t < 4; ++t) pj[t] = xs[jj * NB + min(cg + 8 * t, NB - 1)];
#pragma unroll
          for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[s][t] = fma(acc[s][t], v[s], pj[t]);
          a24 = fma(a24, sv[24 * NB + j], xs[jj * NB + j24]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int row = rg + 8 * s;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int c = cg + 8 * t;
        cpx<T> val = mk(T(0), T(0));
        if (t < 4 && c < NB)
          val = mk(T(row == c ? 1 : 0) - acc[s][t < 4 ? t : 0].re, -acc[s][t < 4 ? t : 0].im);
        else if (c >= NB && c < 2 * NB)
          val = sv[row * NB + c - NB];
        x[s][t] = val;
      }
    }
    y = mk(T(0), T(0));
    if (c24 < NB)
      y = mk(T(c24 == 24 ? 1 : 0) - a24.re, -a24.im);
    else if (c24 < 2 * NB)
      y = sv[24 * NB + c24 - NB];
  }
  }
  __syncthreads();  // the last chunk has been read: its area takes the pivot exchange
  if (lane < 16) xs[(lane >> 3) * W25::EX + 56 + (lane & 7)] = mk(T(0), T(0));  // pivot-row padding columns
  int cs[NS], kof[NS], k24 = -1;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    cs[s] = 31 - (rg + 8 * s);
    kof[s] = 0;
  }
  bool singular = false;
  gj25_all<T>(x, y, cs, kof, k24, rg, cg, xs, singular, std::make_integer_sequence<int, NB>{});
  if (singular && lane == 0) atomicOr(cond, kCondSingular);
  // row r of the V part is row kof of W; W^C = W - V
  cpx<T>* wm = wc + mat * ld;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int k = kof[s];
#pragma unroll
    for (int t = 3; t < NT; ++t) {
      const int col = cg + 8 * t - NB;
      if (col >= 0 && col < NB) wm[k * NB + col] = x[s][t] - (MVP ? vm : sv)[k * NB + col];
    }
  }
  if (c24 >= NB && c24 < 2 * NB) wm[k24 * NB + c24 - NB] = y - (MVP ? vm : sv)[k24 * NB + c24 - NB];
}

// FP32 asks for five waves per SIMD: its elimination fits 96 VGPRs without spills (97 by default, four waves).
// guarded: only the matrices that the folded solver left marked
template <typename T, bool MVP = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 1))) void k_dyson_w25(
    const cpx<T>* __restrict__ vq, const cpx<T>* __restrict__ pnu, cpx<T>* __restrict__ wc, int64_t nmat, int nk,
    int64_t ld, int* __restrict__ cond, int guarded = 0) {
  __shared__ cpx<T> xs[W25::XS];
  __shared__ cpx<T> sv[W25::NB * W25::NB];
  if constexpr (sizeof(T) == 8) {
    if (guarded && !is_left_mark(wc[int64_t(blockIdx.x) * ld])) return;
  }
  w25_solve<T, MVP>(vq, pnu, wc, blockIdx.x, nk, ld, cond, xs, sv);
}

// ---------------------------------------------------------------------------
// Register-blocked form for 8 < N_b <= 16 (three orbitals, four orbitals): one wavefront per (node, q) matrix,
// the layout and elimination of the N_b = 25 kernel without its spread last row.  Lane = rg + 8 cg holds rows
// rg + 8 s (s < 2) in columns cg + 8 t (t < NT) of [I - V P | V] (columns 0..N_b-1, then N_b..2 N_b-1; rows and
// columns past them are zero).  V(q) and P are staged in LDS; V P is formed in that layout; step K searches column
// K by packed keys in the 8-lane group holding it, the owners of the pivot row and of column K publish them through
// LDS, and every lane subtracts f_r * (pivot row).  Slots whose columns are all in I - V P and left of K drop out of
// the update at compile time.
// ---------------------------------------------------------------------------
template <int NB>
struct WR {
  static_assert(NB > 8 && NB <= 16, "two row slots of eight");
  static constexpr int NS = 2, NT = (2 * NB + 7) / 8, NN = NB * NB;
  static constexpr int ROW = 8 * NT;      // pivot row (all column slots)
  static constexpr int EX = ROW + 16;     // pivot row and the multipliers of one step
  static constexpr int TA = (NB + 7) / 8;  // slots holding columns of I - V P
  static_assert(2 * EX <= NN, "the exchange area reuses the P area");
};

template <typename T, int NB, int K, int S>
__device__ __forceinline__ void wr_publish(const cpx<T> (&x)[2][WR<NB>::NT], cpx<T>* ex, int cg, int p, int (&cs)[2],
                                           int (&kof)[2]) {
  constexpr int tk = K / 8;
#pragma unroll
  for (int t = tk; t < WR<NB>::NT; ++t) ex[cg + 8 * t] = x[S][t];
  if (cg == K % 8) ex[WR<NB>::ROW + p] = mk(x[S][tk].re - T(1), x[S][tk].im);
  cs[S] |= int(0x80000000u);
  kof[S] = K;
}

template <typename T, int NB, int K>
__device__ __forceinline__ void wr_step(cpx<T> (&x)[2][WR<NB>::NT], int (&cs)[2], int (&kof)[2], int rg, int cg,
                                        cpx<T>* xs, bool& singular) {
  constexpr int NT = WR<NB>::NT, ROW = WR<NB>::ROW, MIN = int(0x80000000u);
  constexpr int cgk = K % 8, tk = K / 8;
  constexpr int t0 = (K + 1) / 8 < NB / 8 ? (K + 1) / 8 : NB / 8;  // slots left of t0 hold dead columns only
  int key = MIN;
#pragma unroll
  for (int s = 0; s < 2; ++s) key = max(key, (mag_bits(x[s][tk]) & ~31) | cs[s]);
  key = cg == cgk ? key : MIN;
  key = max(key, dpp_shl_i<0x104>(key));
  key = max(key, dpp_shl_i<0x102>(key));
  key = max(key, dpp_shl_i<0x101>(key));
  const int p = 31 - (__builtin_amdgcn_readlane(key, cgk * 8) & 31);
  cpx<T>* ex = xs + (K & 1) * WR<NB>::EX;  // exchange buffers alternate by step parity
  cpx<T>* mu = ex + ROW;
  if (cg == cgk) {
#pragma unroll
    for (int s = 0; s < 2; ++s) mu[rg + 8 * s] = x[s][tk];
  }
  if (rg == (p & 7)) {
    if ((p >> 3) == 0)
      wr_publish<T, NB, K, 0>(x, ex, cg, p, cs, kof);
    else
      wr_publish<T, NB, K, 1>(x, ex, cg, p, cs, kof);
  }
  __syncthreads();
  const cpx<T> pv = ex[K];
  const T pn = norm2(pv);
  singular |= !(pn > T(0)) || !isfinite(pn);  // exact zero, NaN or overflow (the same value in every lane)
  const T d = rcp_nr(pn);
  const cpx<T> pinv = mk(pv.re * d, -pv.im * d);
  cpx<T> f[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) f[s] = mu[rg + 8 * s] * pinv;
#pragma unroll
  for (int t = t0; t < NT; ++t) {
    const cpx<T> pc = ex[cg + 8 * t];
#pragma unroll
    for (int s = 0; s < 2; ++s) x[s][t] = fms(x[s][t], f[s], pc);
  }
}

template <typename T, int NB, int... K>
__device__ __forceinline__ void wr_all(cpx<T> (&x)[2][WR<NB>::NT], int (&cs)[2], int (&kof)[2], int rg, int cg,
                                       cpx<T>* xs, bool& singular, std::integer_sequence<int, K...>) {
  (wr_step<T, NB, K>(x, cs, kof, rg, cg, xs, singular), ...);
}

template <typename T, int NB>
__global__ __launch_bounds__(64) void k_dyson_wr(const cpx<T>* __restrict__ vq, const cpx<T>* __restrict__ pnu,
                                                 cpx<T>* __restrict__ wc, int64_t nmat, int nk, int64_t ld,
                                                 int* __restrict__ cond) {
  using S = WR<NB>;
  constexpr int NT = S::NT, NN = S::NN, TA = S::TA;
  __shared__ cpx<T> sv[NN];  // V(q)
  __shared__ cpx<T> sp[NN];  // P; then the pivot exchange
  const int lane = threadIdx.x;
  const int rg = lane & 7, cg = lane >> 3;
  const int64_t mat = blockIdx.x;
  const int q = int(mat % nk);
  const cpx<T>* vm = vq + int64_t(q) * NN;
  const cpx<T>* pm = pnu + mat * NN;
  for (int e = lane; e < NN; e += 64) {
    sv[e] = vm[e];
    sp[e] = pm[e];
  }
  __syncthreads();
  // I - V P in the columns of slots t < TA, V in the right-hand-side columns
  cpx<T> acc[2][TA];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < TA; ++t) acc[s][t] = mk(T(0), T(0));
  const int r1 = min(rg + 8, NB - 1);  // row of slot 1 (clamped: rows past N_b are not kept)
#pragma unroll 4
  for (int j = 0; j < NB; ++j) {
    const cpx<T> v0 = sv[rg * NB + j], v1 = sv[r1 * NB + j];
#pragma unroll
    for (int t = 0; t < TA; ++t) {
      const cpx<T> pj = sp[j * NB + min(cg + 8 * t, NB - 1)];
      acc[0][t] = fma(acc[0][t], v0, pj);
      acc[1][t] = fma(acc[1][t], v1, pj);
    }
  }
  cpx<T> x[2][NT];
  int cs[2], kof[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int row = rg + 8 * s;
    const bool rv = row < NB;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int c = cg + 8 * t;
      cpx<T> val = mk(T(0), T(0));
      if (rv && c < NB)
        val = mk(T(row == c ? 1 : 0) - acc[s][t < TA ? t : 0].re, -acc[s][t < TA ? t : 0].im);
      else if (rv && c < 2 * NB)
        val = sv[row * NB + c - NB];
      x[s][t] = val;
    }
    cs[s] = rv ? 31 - row : int(0x80000000u);  // rows past N_b never pivot
    kof[s] = 0;
  }
  __syncthreads();  // every lane has read P: its area takes the pivot exchange
  bool singular = false;
  wr_all<T, NB>(x, cs, kof, rg, cg, sp, singular, std::make_integer_sequence<int, NB>{});
  if (singular && lane == 0) atomicOr(cond, kCondSingular);
  // row r of the right-hand side is row kof of the solution; W^C = W - V
  cpx<T>* wm = wc + mat * ld;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = kof[s];
    if (rg + 8 * s < NB) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int col = cg + 8 * t - NB;
        if (col >= 0 && col < NB) wm[k * NB + col] = x[s][t] - sv[k * NB + col];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// n_o x n_o inverse in registers, Gauss-Jordan with partial pivoting
// ---------------------------------------------------------------------------
template <int NO>
__device__ __forceinline__ void invert_inplace(cpx<double> (&a)[NO][NO]) {
  int perm[NO];
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    int p = k;
    double best = norm2(a[k][k]);
#pragma unroll
    for (int i = k + 1; i < NO; ++i) {
      const double v = norm2(a[i][k]);
      if (v > best) {
        best = v;
        p = i;
      }
    }
    perm[k] = p;
    // row swap k <-> p as exact 0/1-weighted blends (w x + (1 - w) y is exact
    // for w in {0, 1}); keeps the matrix in registers, unlike a select chain
#pragma unroll
    for (int i = k + 1; i < NO; ++i) {
      const double w = (p == i) ? 1.0 : 0.0, v = 1.0 - w;
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        const cpx<double> t = a[k][j], u = a[i][j];
        a[k][j] = mk(w * u.re + v * t.re, w * u.im + v * t.im);
        a[i][j] = mk(w * t.re + v * u.re, w * t.im + v * u.im);
      }
    }
    const cpx<double> pinv = inv(a[k][k]);
    a[k][k] = mk(1.0, 0.0);
#pragma unroll
    for (int j = 0; j < NO; ++j) a[k][j] = a[k][j] * pinv;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      if (i == k) continue;
      const cpx<double> f = a[i][k];
      a[i][k] = mk(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < NO; ++j) a[i][j] = fms(a[i][j], f, a[k][j]);
    }
  }
#pragma unroll
  for (int k = NO - 1; k >= 0; --k) {
#pragma unroll
    for (int c = k + 1; c < NO; ++c) {
      const double w = (perm[k] == c) ? 1.0 : 0.0, v = 1.0 - w;
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const cpx<double> t = a[i][k], u = a[i][c];
        a[i][k] = mk(w * u.re + v * t.re, w * u.im + v * t.im);
        a[i][c] = mk(w * t.re + v * u.re, w * t.im + v * u.im);
      }
    }
  }
}

struct DysonGArgs {
  const zd* hk;       // [no][no][nk]
  const zd* sig;      // [r][no][no][nk] or null
  const double* wn;   // [r]
  const zd* rho;      // [r]: G(beta^-) = sum_m rho_m G(i w_m)
  zd* g;              // [r][no][no][nk]
  double* scal;       // [0] mu (in: start / fixed; out), [1] n_target, [2] evaluations, [3] final N_e,
                      // [8] status (copy), [9] the value at ``extra`` (copy), so one read returns all
  double* partials;   // [2][4][max blocks]
  int* status;        // 0 ok, 2 not converged
  const double* extra;  // optional scalar copied to scal[9] by the final pass
  int* fail_word;       // optional: raised to the search's failing status by the final pass, never lowered here
  double* host = nullptr;  // optional pinned host words: the final pass leaves scal[0..9] there, and *fail_word in [10]
  int r, nk, mode, max_evals;
  double beta, tol_mu, tol_n;
  double ne_offset;   // added to -(2/N_k) sum Re rho_m Tr G_m (the uniform grid's 1/2 per spin-orbital)
};

template <int NO>
__device__ __forceinline__ void load_base(const DysonGArgs& A, int64_t gi, cpx<double> (&bm)[NO][NO]) {
  const int m = int(unsigned(gi) / unsigned(A.nk)), k = int(gi) - m * A.nk;  // r N_k < 2^31
  const double w = A.wn[m];
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      const zd h = A.hk[(int64_t(i) * NO + j) * A.nk + k];
      cpx<double> v = mk(-h.re, -h.im);
      if (A.sig) {
        const zd sg = A.sig[((int64_t(m) * NO + i) * NO + j) * A.nk + k];
        v = v - sg;
      }
      if (i == j) v.im += w;
      bm[i][j] = v;
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// block-level deterministic reductions (one wavefront per block); the xor butterfly (distances 32, 16, .. 1) leaves the
// same value in every lane.  The sum's exchanges stay in the vector unit: swaps of half and quarter waves, then
// rotations of a row of 16 by 8 and 4 (the sums so far repeat every 16 and 8 lanes, so these are the xor partners) and
// quad permutations.  Through LDS (__shfl_xor) its 24 dependent exchanges took longer than a 2 x 2 inverse.
__device__ __forceinline__ double wave_sum(double v) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x2 lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  u32x2 hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  v = __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
  lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  v = __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
  v += dpp_move<0x128>(v);  // row_ror:8
  v += dpp_move<0x124>(v);  // row_ror:4
  v += dpp_move<0x4e>(v);   // quad_perm 2 3 0 1
  v += dpp_move<0xb1>(v);   // quad_perm 1 0 3 2
  return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// ---------------------------------------------------------------------------
// The search as a chain of launches.  Its state lives in the scalar block:
//   [0] mu  [1] n_target  [2] evaluations  [3] last N_e  [4] lo  [5] hi
//   [6] step cap  [7] done flag
// Each k_dg_eval launch first takes the Newton step of the previous
// evaluation (every block takes the same step from the same partial sums),
// then evaluates; the final pass takes the last step.  Once the search has
// converged the remaining launches return at once, so a caller may queue a
// fixed number of steps (graph capture) or queue a few, read the done flag
// and continue.
// ---------------------------------------------------------------------------

// per-block partials of H(k): Gershgorin bounds (used when no starting point is given) and the sum of the
// diagonal (the mean level, whose change between two searches of a state shifts the start)
template <int NO>
__global__ __launch_bounds__(64) void k_dg_gersh(DysonGArgs A) {
  double glo = 1e300, ghi = -1e300, dsum = 0.0;
  for (int64_t k = int64_t(blockIdx.x) * 64 + threadIdx.x; k < A.nk; k += int64_t(gridDim.x) * 64) {
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      double rad = 0.0;
#pragma unroll
      for (int j = 0; j < NO; ++j)
        if (j != i) rad += sqrt(norm2(A.hk[(int64_t(i) * NO + j) * A.nk + k]));
      const double d = A.hk[(int64_t(i) * NO + i) * A.nk + k].re;
      glo = fmin(glo, d - rad);
      ghi = fmax(ghi, d + rad);
      dsum += d;
    }
  }
  glo = wave_min(glo);
  ghi = wave_max(ghi);
  dsum = wave_sum(dsum);
  if (threadIdx.x == 0) {
    A.partials[blockIdx.x] = glo;
    A.partials[gridDim.x + blockIdx.x] = ghi;
    A.partials[2 * gridDim.x + blockIdx.x] = dsum;
  }
}

// mu <- centre of the Gershgorin bounds if no finite start was given; otherwise, with ``track``, the start moves
// by the change of the mean diagonal of H since the previous search (scal[10]), the shift of a level by a change
// of Sigma_HF (so that a Hartree shift of many eV does not cost a chain of capped steps); resets the search
// set: the start point (mu0, n_target) comes as arguments instead of a copy into scal[0..1]
// diag_only: partials holds only nblk diagonal sums (a14's), no Gershgorin bounds
// bmax (optional): a14's nbmax block maxima of |Delta Sigma| (non-finite ones already +inf); their maximum goes to
// *dsig, so that a14 needs no reduction launch of its own (the maximum is exact, so the order does not matter)
constexpr int kMetWord = 2;  // of the status words: k_dg_search's count of blocks
struct DgBegin {
  const double* partials;
  int nblk;
  double inv_count;
  int track, set;
  double mu0, nt;
  int diag_only;
  const double* bmax;
  int nbmax;
  double* dsig;
};

// by the 64 lanes of one wavefront
__device__ __forceinline__ void dg_begin(double* __restrict__ scal, int* __restrict__ status, const DgBegin& B) {
  if (B.bmax) {
    double v = 0.0;
    for (int b = threadIdx.x; b < B.nbmax; b += 64) v = fmax(v, B.bmax[b]);
    v = wave_max(v);
    if (threadIdx.x == 0) *B.dsig = v;
  }
  double glo = 1e300, ghi = -1e300, dsum = 0.0;
  for (int b = threadIdx.x; b < B.nblk; b += 64) {
    if (B.diag_only) {
      dsum += B.partials[b];
    } else {
      glo = fmin(glo, B.partials[b]);
      ghi = fmax(ghi, B.partials[B.nblk + b]);
      dsum += B.partials[2 * B.nblk + b];
    }
  }
  if (B.diag_only) glo = ghi = NAN;  // no bounds: a start that is not finite stays so (status 1)
  glo = wave_min(glo);
  ghi = wave_max(ghi);
  const double mean = wave_sum(dsum) * B.inv_count;
  if (threadIdx.x != 0) return;
  if (B.set) {
    scal[0] = B.mu0;
    scal[1] = B.nt;
  }
  if (!isfinite(scal[0])) {
    scal[0] = 0.5 * (glo + ghi);
  } else if (B.track && isfinite(scal[10]) && isfinite(mean)) {
    scal[0] += mean - scal[10];
  }
  scal[10] = mean;
  const bool ok = isfinite(scal[0]);
  scal[2] = 0.0;
  scal[3] = 0.0;
  scal[4] = -INFINITY;
  scal[5] = INFINITY;
  scal[6] = 1.0;
  scal[7] = ok ? 0.0 : 1.0;
  status[0] = ok ? 0 : 1;
  status[kMetWord] = 0;
}

__global__ __launch_bounds__(64) void k_dg_begin(double* __restrict__ scal, int* __restrict__ status, DgBegin B) {
  dg_begin(scal, status, B);
}

// The search state after j Newton steps: mu, n_target, steps taken, N_e at the last evaluation, bracket lo / hi,
// step cap, done.  The host-visible words scal[0..7] hold it between rounds; inside a round the state after step
// j sits in slot j % 2 (scal[16 + 8 (j % 2) ..]) and the partial sums of evaluation j in half j % 2 of the
// partials, so that a launch reads the previous launch's slot and half while its block 0 writes the other ones.
constexpr int kDgSlot = 16;
constexpr int kDgMaxBlocks = 1024;  // of k_dg_eval

// one Newton step of the search from the summed partials (s: sum of rho Tr G, sd: of rho Tr G^2)
__device__ __forceinline__ void dg_newton_update(const DysonGArgs& A, double s, double sd, double (&st)[8]) {
  const double ne = -2.0 * s / double(A.nk) + A.ne_offset, dne = 2.0 * sd / double(A.nk);
  double mu = st[0], lo = st[4], hi = st[5], cap = st[6];
  const double nt = st[1];
  const double f = ne - nt;
  st[2] += 1.0;
  st[3] = ne;
  if (f < 0.0) lo = fmax(lo, mu);
  if (f > 0.0) hi = fmin(hi, mu);
  bool done = false;
  if (fabs(f) <= A.tol_n) {
    done = true;
  } else {
    double nxt = (dne > 0.0) ? mu - f / dne : NAN;
    const bool bracket = isfinite(lo) && isfinite(hi);
    if (bracket) {
      if (!(nxt > lo && nxt < hi)) nxt = 0.5 * (lo + hi);
    } else {
      if (!isfinite(nxt)) nxt = mu + (f < 0.0 ? cap : -cap);
      if (fabs(nxt - mu) > cap) {
        nxt = mu + (nxt > mu ? cap : -cap);
        cap *= 4.0;
      }
    }
    const double tol = A.tol_mu * fmax(1.0, fabs(mu));
    if (fabs(nxt - mu) <= tol || (bracket && hi - lo <= tol)) done = true;
    mu = nxt;
  }
  st[0] = mu;
  st[4] = lo;
  st[5] = hi;
  st[6] = cap;
  st[7] = done ? 1.0 : 0.0;
}

// the state after j steps of this round: step j (j >= 1) is taken from the state after j - 1 steps and the
// partial sums of evaluation j - 1.  Every lane of every block sums the partials in the same order (the
// butterfly reduction leaves the same bits in every lane), so all take the same step.
__device__ __forceinline__ void dg_state(const DysonGArgs& A, int j, int nblk, double (&st)[8]) {
  const double* src = (j == 0) ? A.scal : A.scal + kDgSlot + 8 * ((j - 1) & 1);
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = src[i];
  if (j >= 1 && st[7] == 0.0) {
    const double* part = A.partials + int64_t(2) * nblk * ((j - 1) & 1);
    double s = 0.0, sd = 0.0;
    for (int b = threadIdx.x & 63; b < nblk; b += 64) {
      s += part[b];
      sd += part[nblk + b];
    }
    s = wave_sum(s);
    sd = wave_sum(sd);
    dg_newton_update(A, s, sd, st);
  }
}

// one (node, k) point's share of rho Tr G and rho Tr G^2
template <int NO>
__device__ __forceinline__ void dg_point(const DysonGArgs& A, int64_t gi, double mu, double& acc, double& accd) {
  cpx<double> a[NO][NO];
  load_base<NO>(A, gi, a);
#pragma unroll
  for (int i = 0; i < NO; ++i) a[i][i].re += mu;
  invert_inplace<NO>(a);
  cpx<double> tr = mk(0.0, 0.0), tr2 = mk(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    tr = tr + a[i][i];
#pragma unroll
    for (int jj = 0; jj < NO; ++jj) tr2 = fma(tr2, a[i][jj], a[jj][i]);
  }
  const zd rh = A.rho[int(unsigned(gi) / unsigned(A.nk))];
  acc += rh.re * tr.re - rh.im * tr.im;
  accd += rh.re * tr2.re - rh.im * tr2.im;
}

// evaluation j of a round: N_e(mu) and dN_e/dmu at the state after j steps, as per-block partial sums
template <int NO>
__global__ __launch_bounds__(64) void k_dg_eval(DysonGArgs A, int j, int nblk) {
  double st[8];
  dg_state(A, j, nblk, st);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double* dst = A.scal + kDgSlot + 8 * (j & 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[i] = st[i];
  }
  if (st[7] != 0.0) return;
  const double mu = st[0];
  const int64_t total = int64_t(A.r) * A.nk;
  const int64_t stride = int64_t(gridDim.x) * 64;
  double acc = 0.0, accd = 0.0;
  for (int64_t gi = int64_t(blockIdx.x) * 64 + threadIdx.x; gi < total; gi += stride)
    dg_point<NO>(A, gi, mu, acc, accd);
  acc = wave_sum(acc);
  accd = wave_sum(accd);
  if (threadIdx.x == 0) {
    double* part = A.partials + int64_t(2) * nblk * (j & 1);
    part[blockIdx.x] = acc;
    part[nblk + blockIdx.x] = accd;
  }
}

// threads of the one-block search: as many as its registers allow
constexpr int dg_search_threads(int no) { return no <= 3 ? 1024 : no <= 5 ? 512 : 256; }

// The rest of a round's evaluations in one launch, which stops at convergence: with ``first`` = 0 all of them (and, with
// ``begin``, the start before them) in one block, else those after the ``first`` that k_dg_eval launches have taken.  An
// evaluation costs no launch, also not the ones that are queued beyond convergence; search_launches says where that
// pays.  A wavefront takes the points and the sum of one of k_dg_eval's blocks at a time, so the search is the same bit
// for bit.  The state ends in scal[0..7].
// Several blocks share an evaluation's points: each adds itself to the counter status[kMetWord] (which dg_begin clears)
// once its sums are in the partials, waits until all have, and takes the Newton step by itself.  A block writes the half
// of evaluation j + 2 only when all blocks have added themselves for j + 1, that is, have read the half of j.  The wait
// is bounded: a block that has looked kMeetLooks times goes on alone over all points (the same sums), adds itself no
// more, and so sends the others alone too; every block ends whether or not the others run beside it.
// An iteration of one three-orbital state in a batch (24 x 24, r = 52) takes 0.27 ms with 4 evaluations and 0.39 with 16,
// in 64 launches 0.44 and 0.50; a search that uses up all 64 (n_o = 5, 12 x 12) 1.29 against 1.18.  With the late ones
// in one block, 16 took 1.28 ms and 64 took 8.5: 33 us each at r N_k n_o^3 = 162,500 and 153 at 936,000.
constexpr int kMeetLooks = 4096, kMeetBlocks = 64;

__device__ __forceinline__ void store_agent(double* p, double v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_agent(const double* p) {
  return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p),
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

template <int NO>
__global__ __launch_bounds__(dg_search_threads(NO)) void k_dg_search(DysonGArgs A, DgBegin B, int begin, int first,
                                                                     int nblk, int steps) {
  constexpr int W = dg_search_threads(NO) / 64;
  __shared__ double part[2][kDgMaxBlocks];
  __shared__ int met;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (begin && wave == 0) dg_begin(A.scal, A.status, B);
  __syncthreads();
  double st[8];
  dg_state(A, first, nblk, st);
  const int total = A.r * A.nk;
  bool alone = gridDim.x == 1;
  for (int j = first; j < steps && st[7] == 0.0; ++j) {
    double* const shared = A.partials + int64_t(2) * nblk * (j & 1);
    for (;;) {
      const int nb = alone ? 1 : int(gridDim.x);
      for (int b = (alone ? 0 : int(blockIdx.x)) + nb * wave; b < nblk; b += nb * W) {
        double acc = 0.0, accd = 0.0;
        for (int gi = b * 64 + lane; gi < total; gi += nblk * 64) dg_point<NO>(A, gi, st[0], acc, accd);
        acc = wave_sum(acc);
        accd = wave_sum(accd);
        if (lane == 0 && alone) {
          part[0][b] = acc;
          part[1][b] = accd;
        } else if (lane == 0) {
          store_agent(shared + b, acc);
          store_agent(shared + nblk + b, accd);
        }
      }
      if (alone) break;
      __threadfence();
      __syncthreads();
      if (threadIdx.x == 0) {
        int* const count = A.status + kMetWord;
        const int target = (j - first + 1) * int(gridDim.x);
        int looks = 0;
        __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target && ++looks < kMeetLooks)
          __builtin_amdgcn_s_sleep(2);
        met = looks < kMeetLooks;
        __threadfence();
      }
      __syncthreads();
      if (met) {
        for (int b = threadIdx.x; b < nblk; b += W * 64) {
          part[0][b] = load_agent(shared + b);
          part[1][b] = load_agent(shared + nblk + b);
        }
        break;
      }
      alone = true;
    }
    __syncthreads();
    double s = 0.0, sd = 0.0;
    for (int b = lane; b < nblk; b += 64) {
      s += part[0][b];
      sd += part[1][b];
    }
    s = wave_sum(s);
    sd = wave_sum(sd);
    __syncthreads();
    dg_newton_update(A, s, sd, st);  // every wavefront takes the same step
  }
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) A.scal[i] = st[i];
  }
}

// n_o <= 2 and few points: the whole search in one block of 1024 threads, with the points' characteristic polynomials
// in registers.  With A the matrix at mu = c, m = Tr A / 2, s = ((A_00 - A_11) / 2)^2 + A_01 A_10 (the same at every mu),
// q = m + (mu - c) and D = q^2 - s the determinant at mu,
//   Tr G = 2 q / D,  Tr G^2 = (Tr G)^2 - 2 / D      (n_o = 1: 1 / q and its square),
// so an evaluation reads no memory and takes one complex reciprocal a point.  No term grows with the distance of mu from
// where the search began.  (An expansion of the determinant about that mu, det A + d Tr A + d^2, is 1.3 us a search faster
// but cancels: N_e was 4e-12 off after a start 300 eV away at beta = 100/eV, past the search's tolerance of 1e-13.)
// c = H_00 of the first point takes a common offset of the levels out of m.  N_e is then within 2e-14 of its value in
// extended precision for beta from 10 to 500/eV, offsets up to 1000 eV and bandwidths from 0.01 to 30 eV, as it is with
// the inverses of k_dg_eval.
constexpr int kPolyPoints = 16;  // complex pairs (n_o = 2) or values (1) a thread holds, divided by n_o
constexpr int kPolyNodes = 1024;
template <int NO>
__global__ __launch_bounds__(1024) void k_dg_search_poly(DysonGArgs A, DgBegin B, int begin, int steps) {
  constexpr int P = kPolyPoints / NO;
  __shared__ double red[32];
  __shared__ zd rho[kPolyNodes + 1];  // and a zero, for the threads' slots beyond the last point
  for (int m = threadIdx.x; m <= A.r; m += 1024) rho[m] = m < A.r ? A.rho[m] : mk(0.0, 0.0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (begin && wave == 0) dg_begin(A.scal, A.status, B);
  __syncthreads();
  double st[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = A.scal[i];
  const int total = A.r * A.nk;
  const double c = A.hk[0].re;
  cpx<double> hm[P], sq[P];  // m and s
  int node[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int gi = int(threadIdx.x) + 1024 * u;
    node[u] = A.r;
    hm[u] = mk(0.0, 1.0);  // regular at every mu
    sq[u] = mk(0.0, 0.0);
    if (gi < total) {
      cpx<double> a[NO][NO];
      load_base<NO>(A, gi, a);
      node[u] = int(unsigned(gi) / unsigned(A.nk));
      if constexpr (NO == 1) {
        hm[u] = mk(a[0][0].re + c, a[0][0].im);
      } else {
        a[0][0].re += c;
        a[1][1].re += c;
        hm[u] = scale(a[0][0] + a[1][1], 0.5);
        const cpx<double> h = scale(a[0][0] - a[1][1], 0.5);
        sq[u] = fma(h * h, a[0][1], a[1][0]);
      }
    }
  }
  for (int j = 0; j < steps && st[7] == 0.0; ++j) {
    const double d = st[0] - c;
    double acc = 0.0, accd = 0.0;
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const cpx<double> q = mk(hm[u].re + d, hm[u].im);
      cpx<double> t, t2;
      if constexpr (NO == 1) {
        t = scale(conj(q), rcp_nr(norm2(q)));
        t2 = t * t;
      } else {
        cpx<double> di = q * q - sq[u];
        di = scale(conj(di), 2.0 * rcp_nr(norm2(di)));  // 2 / D
        t = q * di;
        t2 = t * t - di;
      }
      const zd rh = rho[node[u]];
      acc += rh.re * t.re - rh.im * t.im;
      accd += rh.re * t2.re - rh.im * t2.im;
      if (u & 1) __builtin_amdgcn_sched_barrier(0);  // more points at once spill
    }
    acc = wave_sum(acc);
    accd = wave_sum(accd);
    if ((threadIdx.x & 63) == 0) {
      red[wave] = acc;
      red[16 + wave] = accd;
    }
    __syncthreads();
    acc = accd = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      acc += red[w];
      accd += red[16 + w];
    }
    __syncthreads();
    dg_newton_update(A, acc, accd, st);  // every thread takes the same step
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) A.scal[i] = st[i];
  }
}

// G at the search's result: with n >= 1 evaluations in this round the last step (from evaluation n - 1) is
// taken here, and block 0 writes the state back to the host-visible words
template <int NO>
__global__ __launch_bounds__(64) void k_dg_final(DysonGArgs A, int n, int nblk) {
  double st[8];
  if (A.mode == 1 && n >= 1) {
    dg_state(A, n, nblk, st);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) st[i] = A.scal[i];
  }
  const double mu = st[0];
  const int64_t total = int64_t(A.r) * A.nk;
  const int64_t stride = int64_t(gridDim.x) * 64;
  for (int64_t gi = int64_t(blockIdx.x) * 64 + threadIdx.x; gi < total; gi += stride) {
    cpx<double> a[NO][NO];
    load_base<NO>(A, gi, a);
#pragma unroll
    for (int i = 0; i < NO; ++i) a[i][i].re += mu;
    invert_inplace<NO>(a);
    const int m = int(unsigned(gi) / unsigned(A.nk)), k = int(gi) - m * A.nk;
#pragma unroll
    for (int i = 0; i < NO; ++i)
#pragma unroll
      for (int j = 0; j < NO; ++j) A.g[((int64_t(m) * NO + i) * NO + j) * A.nk + k] = a[i][j];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (A.mode == 1 && n >= 1) {
#pragma unroll
      for (int i = 0; i < 8; ++i) A.scal[i] = st[i];
    }
    if (A.mode == 1 && A.status[0] == 0) {
      const bool conv = st[7] != 0.0 || fabs(st[3] - st[1]) <= A.tol_n;
      if (!conv || !isfinite(mu)) A.status[0] = 2;
    }
    if (A.fail_word && A.status[0] > *A.fail_word) *A.fail_word = A.status[0];
    A.scal[8] = double(A.status[0]);
    if (A.extra) A.scal[9] = *A.extra;
    if (A.host) {  // the caller reads them once this launch has completed: no copy behind it
      for (int i = 0; i < 10; ++i) A.host[i] = A.scal[i];
      if (A.fail_word) A.host[10] = double(*A.fail_word);
      __threadfence_system();
    }
  }
}

// ---------------------------------------------------------------------------
// adjoint of Dyson W (FP64).  With A = I - V P and W = A^{-1} V, A^{-1} = I + W P and
// dW = A^{-1} dV (I + P W) + W dP W.  For a cotangent Wbar of W^C = W - V:
//   U = W^H Wbar,  Pbar = U W^H,  Y = Wbar W^H + P^H Pbar,
//   Vbar = A^{-H} Wbar (I + P W)^H - Wbar = P^H U + Y P^H,
// six products and no system to solve: W comes from the forward solve, through the folded basis where V allows it.
// (Solving A^H X = Wbar instead took two eliminations and a pass of X through memory.)  A small block per (q, chunk of
// nodes), so that few waves wait for each other; a lane owns a tile of R x C entries of every product, and two products
// that are ready together share a loop.  Each step loads R + C values from LDS for R C multiply-adds.  At 48 x 48,
// r = 59, N_b = 25 the vector unit issues 69% of the time, 93% of it multiply-adds, and a wavefront waits 27% of its time
// (11% for LDS); LDS lets 1.9 wavefronts on a SIMD.  At 25 x 25 the 2 x 3 tiles fill 117 lanes; 4 x 3 ones in a single
// wavefront load less, but LDS then holds one wavefront per SIMD and its latency shows.  The FP64 matrix rate equals the
// vector rate, so padding 25 to 32 on the matrix cores would only add work.  The whole adjoint, 39 nodes, V without the
// symmetry, before and now: N_b = 25 at 32 x 32 1960 -> 1700 us; at 24 x 24 N_b = 16 502 -> 411, 9 172 -> 95, 8 135 -> 71,
// 4 52 -> 32, 2 33 -> 20.
// V(q) is static, so Vbar(q) sums over the nodes: each block sums its chunk in a fixed order and writes a partial.
// ---------------------------------------------------------------------------
template <int NB>
struct BwdTile {
  static constexpr int TH = NB > 16 ? 128 : 64;
  static constexpr int R = NB > 9 ? 2 : 1, C = NB > 16 ? 3 : NB > 8 ? 2 : 1;
  static constexpr int RG = (NB + R - 1) / R, CG = (NB + C - 1) / C;
  static_assert(RG * CG <= TH, "one lane per tile");
};

template <int NB>
__global__ __launch_bounds__(BwdTile<NB>::TH) void k_dyson_w_bwd(const zd* __restrict__ vq, const zd* __restrict__ pnu,
                                                    const zd* __restrict__ wbar, const zd* __restrict__ wcm,
                                                    zd* __restrict__ pbar, zd* __restrict__ vpart, int r, int nk,
                                                    int chunks) {
  using S = BwdTile<NB>;
  constexpr int NN = NB * NB, R = S::R, C = S::C;
  __shared__ cpx<double> sP[NN], sW[NN], sB[NN], sU[NN];  // sB: Wbar, then Pbar; sU: U, then Y
  const int q = blockIdx.x, ch = blockIdx.y, lane = threadIdx.x;
  const int m0 = int(int64_t(r) * ch / chunks), m1 = int(int64_t(r) * (ch + 1) / chunks);
  // rows ti + RG a and columns tj + CG b: neighbouring lanes read neighbouring values; past N_b the last one, not kept
  const int ti = lane % S::RG, tj = min(lane / S::RG, S::CG - 1);
  int row[R], col[C];
  bool keep[R][C];
#pragma unroll
  for (int a = 0; a < R; ++a) row[a] = min(ti + S::RG * a, NB - 1);
#pragma unroll
  for (int b = 0; b < C; ++b) col[b] = min(tj + S::CG * b, NB - 1);
#pragma unroll
  for (int a = 0; a < R; ++a)
#pragma unroll
    for (int b = 0; b < C; ++b)
      keep[a][b] = lane < S::RG * S::CG && ti + S::RG * a < NB && tj + S::CG * b < NB;
  cpx<double> vacc[R][C];
#pragma unroll
  for (int a = 0; a < R; ++a)
#pragma unroll
    for (int b = 0; b < C; ++b) vacc[a][b] = mk(0.0, 0.0);
  for (int m = m0; m < m1; ++m) {
    const int64_t base = (int64_t(m) * nk + q) * NN;
    __syncthreads();  // the previous node's products are done with the LDS tiles
    for (int e = lane; e < NN; e += S::TH) {
      sP[e] = pnu[base + e];
      sB[e] = wbar[base + e];
      sW[e] = wcm[base + e] + vq[int64_t(q) * NN + e];  // W = W^C + V
    }
    __syncthreads();
    cpx<double> u[R][C], z[R][C];
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b) u[a][b] = z[a][b] = mk(0.0, 0.0);
    // U = W^H Wbar,  Z = Wbar W^H
#pragma unroll 5
    for (int k = 0; k < NB; ++k) {
      cpx<double> wr[R], bc[C], br[R], wc[C];
#pragma unroll
      for (int a = 0; a < R; ++a) wr[a] = conj(sW[k * NB + row[a]]), br[a] = sB[row[a] * NB + k];
#pragma unroll
      for (int b = 0; b < C; ++b) bc[b] = sB[k * NB + col[b]], wc[b] = conj(sW[col[b] * NB + k]);
#pragma unroll
      for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < C; ++b) {
          u[a][b] = fma(u[a][b], wr[a], bc[b]);
          z[a][b] = fma(z[a][b], br[a], wc[b]);
        }
    }
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b) {
        if (keep[a][b]) sU[row[a] * NB + col[b]] = u[a][b];
        u[a][b] = mk(0.0, 0.0);
      }
    __syncthreads();
    // Pbar = U W^H,  Vbar += P^H U
#pragma unroll 5
    for (int k = 0; k < NB; ++k) {
      cpx<double> ur[R], wc[C], pr[R], uc[C];
#pragma unroll
      for (int a = 0; a < R; ++a) ur[a] = sU[row[a] * NB + k], pr[a] = conj(sP[k * NB + row[a]]);
#pragma unroll
      for (int b = 0; b < C; ++b) wc[b] = conj(sW[col[b] * NB + k]), uc[b] = sU[k * NB + col[b]];
#pragma unroll
      for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < C; ++b) {
          u[a][b] = fma(u[a][b], ur[a], wc[b]);
          vacc[a][b] = fma(vacc[a][b], pr[a], uc[b]);
        }
    }
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b)
        if (keep[a][b]) {
          sB[row[a] * NB + col[b]] = u[a][b];
          pbar[base + row[a] * NB + col[b]] = u[a][b];
        }
    __syncthreads();
    // Y = Z + P^H Pbar
#pragma unroll 5
    for (int k = 0; k < NB; ++k) {
      cpx<double> pr[R], bc[C];
#pragma unroll
      for (int a = 0; a < R; ++a) pr[a] = conj(sP[k * NB + row[a]]);
#pragma unroll
      for (int b = 0; b < C; ++b) bc[b] = sB[k * NB + col[b]];
#pragma unroll
      for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < C; ++b) z[a][b] = fma(z[a][b], pr[a], bc[b]);
    }
#pragma unroll
    for (int a = 0; a < R; ++a)
#pragma unroll
      for (int b = 0; b < C; ++b)
        if (keep[a][b]) sU[row[a] * NB + col[b]] = z[a][b];
    __syncthreads();
    // Vbar += Y P^H
#pragma unroll 5
    for (int k = 0; k < NB; ++k) {
      cpx<double> yr[R], pc[C];
#pragma unroll
      for (int a = 0; a < R; ++a) yr[a] = sU[row[a] * NB + k];
#pragma unroll
      for (int b = 0; b < C; ++b) pc[b] = conj(sP[col[b] * NB + k]);
#pragma unroll
      for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < C; ++b) vacc[a][b] = fma(vacc[a][b], yr[a], pc[b]);
    }
  }
#pragma unroll
  for (int a = 0; a < R; ++a)
#pragma unroll
    for (int b = 0; b < C; ++b)
      if (keep[a][b]) vpart[(int64_t(ch) * nk + q) * NN + row[a] * NB + col[b]] = vacc[a][b];
}

// ---------------------------------------------------------------------------
// adjoint of Dyson G with the chemical potential.  G = [(i w + mu) - X]^{-1}
// with X = H + Sigma; dG = G (dX - dmu) G, so the direct cotangent of X is
// S = G^H Gbar G^H and dL/dmu = mubar - Re sum tr S.  With the filling held,
// N_e(mu, X) = N_target moves mu by -dN_X / N_mu, with
// N_mu = 2/N_k Re sum rho_m tr G^2 and the X-cotangent of N_e equal to
// -2/N_k conj(rho_m) (G^2)^H; the second pass adds that term.
// ---------------------------------------------------------------------------
template <int NO>
__global__ __launch_bounds__(64) void k_dyson_g_bwd1(DysonGArgs A, double mu, const zd* __restrict__ gbar,
                                                     zd* __restrict__ sbar, double* __restrict__ part) {
  const int64_t total = int64_t(A.r) * A.nk;
  const int64_t gi = int64_t(blockIdx.x) * 64 + threadIdx.x;
  double acc = 0.0, acc2 = 0.0;
  if (gi < total) {
    cpx<double> g[NO][NO];
    load_base<NO>(A, gi, g);
#pragma unroll
    for (int i = 0; i < NO; ++i) g[i][i].re += mu;
    invert_inplace<NO>(g);
    const int m = int(gi / A.nk), k = int(gi - int64_t(m) * A.nk);
    cpx<double> t1[NO][NO];
#pragma unroll
    for (int i = 0; i < NO; ++i)
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        cpx<double> s = mk(0.0, 0.0);
#pragma unroll
        for (int c = 0; c < NO; ++c) s = fma(s, conj(g[c][i]), gbar[((int64_t(m) * NO + c) * NO + j) * A.nk + k]);
        t1[i][j] = s;
      }
    cpx<double> tr2 = mk(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < NO; ++i)
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        cpx<double> s = mk(0.0, 0.0);
#pragma unroll
        for (int c = 0; c < NO; ++c) s = fma(s, t1[i][c], conj(g[j][c]));
        sbar[((int64_t(m) * NO + i) * NO + j) * A.nk + k] = s;
        if (i == j) acc += s.re;
        tr2 = fma(tr2, g[i][j], g[j][i]);
      }
    const zd rh = A.rho[m];
    acc2 = rh.re * tr2.re - rh.im * tr2.im;
  }
  acc = wave_sum(acc);
  acc2 = wave_sum(acc2);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = acc;
    part[gridDim.x + blockIdx.x] = acc2;
  }
}

template <int NO>
__global__ __launch_bounds__(64) void k_dyson_g_bwd2(DysonGArgs A, double mu, double mubar,
                                                     const double* __restrict__ part, int nblk,
                                                     zd* __restrict__ sbar) {
  double s = 0.0, s2 = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 64) {
    s += part[b];
    s2 += part[nblk + b];
  }
  s = wave_sum(s);
  s2 = wave_sum(s2);
  const double n_mu = 2.0 * s2 / double(A.nk);
  const double coef = (mubar - s) / n_mu * 2.0 / double(A.nk);
  const int64_t total = int64_t(A.r) * A.nk;
  const int64_t gi = int64_t(blockIdx.x) * 64 + threadIdx.x;
  if (gi >= total) return;
  cpx<double> g[NO][NO];
  load_base<NO>(A, gi, g);
#pragma unroll
  for (int i = 0; i < NO; ++i) g[i][i].re += mu;
  invert_inplace<NO>(g);
  const int m = int(gi / A.nk), k = int(gi - int64_t(m) * A.nk);
  const cpx<double> w = scale(conj(A.rho[m]), coef);
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      cpx<double> g2ji = mk(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < NO; ++c) g2ji = fma(g2ji, g[j][c], g[c][i]);
      const int64_t o = ((int64_t(m) * NO + i) * NO + j) * A.nk + k;
      sbar[o] = sbar[o] + w * conj(g2ji);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

template <typename T>
hipError_t dyson_w25(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, hipStream_t s, int64_t ld,
                     bool guarded) {
  const int64_t nmat = int64_t(p.r) * p.nk;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(unsigned(nmat)), dim3(64), 0, s, (const cpx<T>*)v_q, (const cpx<T>*)p_nu,
                       (cpx<T>*)wc_nu, nmat, p.nk, ld, p.d_status + kCondWord, guarded ? 1 : 0);
  };
  if (p.tune.w25_mfma == 1)
    go(k_dyson_w25<T, true>);
  else
    go(k_dyson_w25<T, false>);
  return hipGetLastError();
}

template <int NB, typename T>
hipError_t dyson_wr(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, hipStream_t s, int64_t ld) {
  const int64_t nmat = int64_t(p.r) * p.nk;
  hipLaunchKernelGGL((k_dyson_wr<T, NB>), dim3(unsigned(nmat)), dim3(64), 0, s, (const cpx<T>*)v_q,
                     (const cpx<T>*)p_nu, (cpx<T>*)wc_nu, nmat, p.nk, ld, p.d_status + kCondWord);
  return hipGetLastError();
}

template <int NB, typename T>
hipError_t dyson_w_small(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, hipStream_t s, int64_t ld) {
  constexpr int MPW = DysonWShape<NB>::MPW;
  const int64_t nmat = int64_t(p.r) * p.nk;
  hipLaunchKernelGGL((k_dyson_w<NB, T>), dim3(unsigned((nmat + MPW - 1) / MPW)), dim3(64), 0, s, (const cpx<T>*)v_q,
                     (const cpx<T>*)p_nu, (cpx<T>*)wc_nu, nmat, p.nk, ld, p.d_status + kCondWord);
  return hipGetLastError();
}

template <typename T>
hipError_t dyson_w_t(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, hipStream_t s, int64_t ld,
                     bool fold) {
  const int64_t nn = int64_t(p.nb) * p.nb, nmat = int64_t(p.r) * p.nk;
  if (ld == 0) ld = nn;
  if (ld < nn) return hipErrorInvalidValue;
  // FP32 calls on the caller's arrays keep the eliminations that follow, bit for bit: their rounding, amplified 19-56
  // times by the i nu -> tau map behind, shows at 1e-5 in W^C(tau), and a caller's results stay what they were.  That
  // is a choice and no limit: a state's FP32 phase solves its folded matrices in another order, and these sums in
  // another lane layout would keep their bits
  if constexpr (sizeof(T) == 4) {
    if (fold && p.nb == 8) return dyson_w_small<8, T>(p, v_q, p_nu, wc_nu, s, ld);
    if (fold && p.nb == 9) return dyson_wr<9, T>(p, v_q, p_nu, wc_nu, s, ld);
    if (fold && p.nb == 16) return dyson_wr<16, T>(p, v_q, p_nu, wc_nu, s, ld);
  }
  // FP64, N_b >= 9: matrices whose V(q) has the pair-exchange symmetry are solved per unordered pair; the others are
  // left marked for the general kernel behind.  24 x 24, r = 53: 234 instead of 447 us (N_b = 25), 67 instead of 163
  // (16), 28 instead of 71 (9).  A V without the symmetry pays for the look at it, up to 8% (N_b = 16, 12 x 12: 54
  // against 50 us); below 4,096 matrices, where the second launch costs as much as the smaller systems save (6 x 6: 23
  // against 18 us at N_b = 16), nothing is tried.  The mark sits in the output, so an output over the input P (or V)
  // takes the general kernel alone.
  const auto overlap = [&](const void* x, int64_t count) {
    const char *a = (const char*)x, *b = (const char*)wc_nu;
    return a < b + nmat * ld * int64_t(sizeof(cpx<T>)) && b < a + count * int64_t(sizeof(cpx<T>));
  };
  bool guarded = false;
  if (sizeof(T) == 8 && fold && !p.folded && fold_solver(p.nb, p.fold_nb) && nmat >= 4096 && !overlap(p_nu, nmat * nn) &&
      !overlap(v_q, p.nk * nn)) {
    const hipError_t e = launch_dyson_wq_fold(p, v_q, p_nu, wc_nu, ld, s);
    if (e != hipSuccess) return e;
    guarded = true;
  }
  if (p.nb == 25) return dyson_w25<T>(p, v_q, p_nu, wc_nu, s, ld, guarded);
  switch (p.nb) {  // up to five pairs the two-lanes-per-row form is as fast or faster
    case 1: return dyson_w_small<1, T>(p, v_q, p_nu, wc_nu, s, ld);
    case 2: return dyson_w_small<2, T>(p, v_q, p_nu, wc_nu, s, ld);
    case 3: return dyson_w_small<3, T>(p, v_q, p_nu, wc_nu, s, ld);
    case 4: return dyson_w_small<4, T>(p, v_q, p_nu, wc_nu, s, ld);
    case 5: return dyson_w_small<5, T>(p, v_q, p_nu, wc_nu, s, ld);
    default: break;
  }
  // the same at N_b = 9: FP64 212 matrices 6.0 against 8.4 us, 1,908 8.4 against 9.1, 2,400 9.9 against 9.5; FP32 640
  // matrices 8.9 against 12.1, 2,560 10.6 against 13.1, 5,760 the same
  if (p.nb == 9 && nmat < (sizeof(T) == 4 ? 6000 : 2200)) return dyson_wr<9, T>(p, v_q, p_nu, wc_nu, s, ld);
  // four matrices per wavefront; few larger ones (under six wavefronts of one matrix per SIMD) finish sooner one to a
  // wavefront: N_b = 16 with 1,908 matrices 10.6 against 18.4 us in FP32, with 7,632 the same
  if (p.nb >= 15 && nmat < 6000 && !guarded)
    return p.nb == 16 ? dyson_wr<16, T>(p, v_q, p_nu, wc_nu, s, ld) : dyson_wr<15, T>(p, v_q, p_nu, wc_nu, s, ld);
  return launch_dyson_wq(p, v_q, p_nu, wc_nu, ld, s, guarded);
}

template <int NO>
DysonGArgs dyson_g_args(const Plan& p, const void* h_k, const void* sig_iw, int mode, void* g_iw, double* scal,
                        double* partials, int* status) {
  DysonGArgs A;
  A.hk = (const zd*)h_k;
  A.sig = (const zd*)sig_iw;
  A.wn = p.d_wn;
  A.rho = (const zd*)p.dmaps64.m[5];
  A.g = (zd*)g_iw;
  A.scal = scal;
  A.partials = partials;
  A.status = status;
  A.r = p.r;
  A.nk = p.nk;
  A.mode = mode;
  A.max_evals = 200;
  A.beta = p.beta;
  A.tol_mu = 1e-13;
  A.tol_n = 1e-13;
  A.extra = nullptr;
  A.fail_word = nullptr;
  A.ne_offset = p.ne_offset;
  return A;
}

// grid of the search: one block per 64 (node, k) points, at most max_blocks (grid-stride beyond)
// one-wave blocks over the (node, k) points, at most 1024: every evaluation re-sums the previous one's per-block
// partials in each block, so that work grows with the square of the block count
static int dyson_g_blocks(const Plan& p) {
  const int64_t need = (int64_t(p.r) * p.nk + 63) / 64;
  const int64_t cap = p.max_blocks < kDgMaxBlocks ? p.max_blocks : kDgMaxBlocks;
  return int(need < cap ? need : cap);
}

}  // namespace

int dyson_g_partials_needed(const Plan& p) {
  const int64_t gb = (p.nk + 63) / 64 < 1024 ? (p.nk + 63) / 64 : 1024;  // start: three partials per block
  const int nb = dyson_g_blocks(p);                                      // evaluations: two halves of two
  return int(3 * gb > 4 * int64_t(nb) ? 3 * gb : 4 * int64_t(nb));
}

namespace {

// Where a search's evaluations run: the number of k_dg_eval launches, the rest in one k_dg_search.  By the work of an
// evaluation, r N_k n_o^3: up to 50,000 one block takes an evaluation in 10 us or less, a launch 12.
constexpr int64_t kSearchOneBlock = 50000, kSearchTail = 2000000;
constexpr int kSearchLaunches = 10;
bool search_poly(const Plan& p) { return p.no <= 2 && p.r <= kPolyNodes && int64_t(p.r) * p.nk <= 1024 * (kPolyPoints / p.no); }
int search_launches(const Plan& p, int steps, bool tail) {
  const int64_t work = int64_t(p.r) * p.nk * p.no * p.no * p.no;
  if (search_poly(p) || (p.no > 2 && work <= kSearchOneBlock)) return 0;
  return tail && work <= kSearchTail && steps > kSearchLaunches + 6 ? kSearchLaunches : steps;
}

template <int NO>
hipError_t dyson_g_search_no(const Plan& p, const void* h_k, const void* sig_iw, double* scal, double* partials,
                             int* status, int steps, const DysonGStart* start, int* pending, bool tail, hipStream_t s) {
  DysonGArgs A = dyson_g_args<NO>(p, h_k, sig_iw, 1, nullptr, scal, partials, status);
  const int launches = search_launches(p, steps, tail);
  DgBegin B = {};
  if (start) {
    const bool diag = start->dpart != nullptr;
    const int gb = int((p.nk + 63) / 64 < 1024 ? (p.nk + 63) / 64 : 1024);
    if (!diag) hipLaunchKernelGGL((k_dg_gersh<NO>), dim3(gb), dim3(64), 0, s, A);
    B = DgBegin{diag ? start->dpart : partials, diag ? start->dnblk : gb, 1.0 / (double(NO) * p.nk), start->track,
                start->set, start->mu0, start->nt, diag ? 1 : 0, start->bmax, start->nbmax, start->dsig};
    if (launches > 0) hipLaunchKernelGGL(k_dg_begin, dim3(1), dim3(64), 0, s, scal, status, B);
  }
  const int blocks = dyson_g_blocks(p);
  for (int i = 0; i < launches; ++i) hipLaunchKernelGGL((k_dg_eval<NO>), dim3(blocks), dim3(64), 0, s, A, i, blocks);
  if constexpr (NO <= 2) {
    if (search_poly(p)) {
      hipLaunchKernelGGL((k_dg_search_poly<NO>), dim3(1), dim3(1024), 0, s, A, B, start ? 1 : 0, steps);
      *pending = 0;
      return hipGetLastError();
    }
  }
  if (launches < steps || launches == 0) {
    const int per = dg_search_threads(NO) / 64, meet = std::min((blocks + per - 1) / per, kMeetBlocks);
    hipLaunchKernelGGL((k_dg_search<NO>), dim3(launches == 0 ? 1 : meet), dim3(dg_search_threads(NO)), 0, s, A, B,
                       start && launches == 0 ? 1 : 0, launches, blocks, steps);
  }
  *pending = launches == steps ? launches : 0;
  return hipGetLastError();
}

template <int NO>
hipError_t dyson_g_final_no(const Plan& p, const void* h_k, const void* sig_iw, int mode, void* g_iw,
                            double* scal, double* partials, int* status, const double* extra, int steps,
                            int* fail_word, double* host, hipStream_t s) {
  DysonGArgs A = dyson_g_args<NO>(p, h_k, sig_iw, mode, g_iw, scal, partials, status);
  A.extra = extra;
  A.fail_word = fail_word;
  A.host = host;
  const int blocks = dyson_g_blocks(p);
  hipLaunchKernelGGL((k_dg_final<NO>), dim3(blocks), dim3(64), 0, s, A, mode == 1 ? steps : 0, blocks);
  return hipGetLastError();
}

// workspace: W^C (pair matrix layout, dense), then the Vbar partials [chunks][N_k][N_b][N_b]
template <int NB>
hipError_t dyson_w_bwd_nb(const Plan& p, const void* v_q, const void* p_nu, const void* wbar, void* pbar,
                          void* ws, int chunks, hipStream_t s) {
  zd* wcm = (zd*)ws;
  zd* vpart = wcm + int64_t(p.r) * p.nk * NB * NB;
  const hipError_t e = dyson_w_t<double>(p, v_q, p_nu, wcm, s, 0, true);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_dyson_w_bwd<NB>), dim3(unsigned(p.nk), unsigned(chunks)), dim3(BwdTile<NB>::TH), 0, s, (const zd*)v_q,
                     (const zd*)p_nu, (const zd*)wbar, (const zd*)wcm, (zd*)pbar, vpart, p.r, p.nk, chunks);
  return hipGetLastError();
}

template <int NO>
hipError_t dyson_g_bwd_no(const Plan& p, const void* h_k, const void* sig_iw, double mu, double n_target,
                          double mubar, const void* gbar, void* sbar, hipStream_t s) {
  DysonGArgs A;
  A.hk = (const zd*)h_k;
  A.sig = (const zd*)sig_iw;
  A.wn = p.d_wn;
  A.rho = (const zd*)p.dmaps64.m[5];
  A.g = nullptr;
  A.scal = p.d_scalars;
  A.partials = p.d_partials;
  A.status = p.d_status;
  A.r = p.r;
  A.nk = p.nk;
  A.mode = 0;
  A.max_evals = 0;
  A.beta = p.beta;
  A.tol_mu = A.tol_n = 0.0;
  A.extra = nullptr;
  A.fail_word = nullptr;
  A.ne_offset = p.ne_offset;
  const int64_t total = int64_t(p.r) * p.nk;
  const int nblk = int((total + 63) / 64);
  if (2 * int64_t(nblk) > 8 * int64_t(p.max_blocks)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_dyson_g_bwd1<NO>), dim3(unsigned(nblk)), dim3(64), 0, s, A, mu, (const zd*)gbar, (zd*)sbar,
                     p.d_partials);
  if (std::isfinite(n_target))
    hipLaunchKernelGGL((k_dyson_g_bwd2<NO>), dim3(unsigned(nblk)), dim3(64), 0, s, A, mu, mubar,
                       (const double*)p.d_partials, nblk, (zd*)sbar);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dyson_w_bwd(const Plan& p, const void* v_q, const void* p_nu, const void* wbar, void* pbar,
                              void* vpart, int chunks, hipStream_t s) {
  switch (p.nb) {
#define QGW_CASE(NBV) \
  case NBV:           \
    return dyson_w_bwd_nb<NBV>(p, v_q, p_nu, wbar, pbar, vpart, chunks, s);
    QGW_FOR_EACH_NB(QGW_CASE)
#undef QGW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_dyson_g_bwd(const Plan& p, const void* h_k, const void* sig_iw, double mu, double n_target,
                              double mubar, const void* gbar, void* sbar, hipStream_t s) {
  switch (p.no) {
#define QGW_CASE(NOV) \
  case NOV:           \
    return dyson_g_bwd_no<NOV>(p, h_k, sig_iw, mu, n_target, mubar, gbar, sbar, s);
    QGW_FOR_EACH_NO(QGW_CASE)
#undef QGW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_dyson_w(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, hipStream_t s,
                          int64_t out_ld, bool fold) {
  return p.prec == 0 ? dyson_w_t<double>(p, v_q, p_nu, wc_nu, s, out_ld, fold)
                     : dyson_w_t<float>(p, v_q, p_nu, wc_nu, s, out_ld, fold);
}

#define QGW_NO_SWITCH(CALL)    \
  switch (p.no) {              \
    case 1: { constexpr int NOV = 1; return CALL; } \
    case 2: { constexpr int NOV = 2; return CALL; } \
    case 3: { constexpr int NOV = 3; return CALL; } \
    case 4: { constexpr int NOV = 4; return CALL; } \
    case 5: { constexpr int NOV = 5; return CALL; } \
    case 6: { constexpr int NOV = 6; return CALL; } \
    case 7: { constexpr int NOV = 7; return CALL; } \
    case 8: { constexpr int NOV = 8; return CALL; } \
    default: return hipErrorInvalidValue;          \
  }

bool dyson_g_one_block(const Plan& p) { return search_launches(p, 1, false) == 0; }

hipError_t launch_dyson_g_search(const Plan& p, const void* h_k, const void* sig_iw, double* scal, double* partials,
                                 int* status, int steps, const DysonGStart* start, int* pending, hipStream_t s,
                                 bool tail) {
  QGW_NO_SWITCH((dyson_g_search_no<NOV>(p, h_k, sig_iw, scal, partials, status, steps, start, pending, tail, s)))
}

hipError_t launch_dyson_g_final(const Plan& p, const void* h_k, const void* sig_iw, int mode, void* g_iw,
                                double* scal, double* partials, int* status, hipStream_t s, const double* extra,
                                int steps, int* fail_word, double* host) {
  QGW_NO_SWITCH((dyson_g_final_no<NOV>(p, h_k, sig_iw, mode, g_iw, scal, partials, status, extra, steps, fail_word,
                                       host, s)))
}

hipError_t launch_dyson_g_chain(const Plan& p, const void* h_k, const void* sig_iw, int mode, void* g_iw,
                                double* scal, double* partials, int* status, int steps, int* fail_word,
                                hipStream_t s, const DysonGStart& start, double* host) {
  hipError_t e = hipSuccess;
  int pending = 0;
  if (mode == 1)
    e = launch_dyson_g_search(p, h_k, sig_iw, scal, partials, status, steps, &start, &pending, s, true);
  if (e == hipSuccess) e = launch_dyson_g_final(p, h_k, sig_iw, mode, g_iw, scal, partials, status, s, start.dsig,
                                                pending, fail_word, host);
  return e;
}

#undef QGW_NO_SWITCH

}  // namespace qgw

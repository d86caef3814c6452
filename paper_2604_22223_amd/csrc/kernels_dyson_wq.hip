// Screened interaction W^C = (I - V P)^{-1} V - V (Eq. eq-screened-coulomb) for N_b <= 16: four matrices per wavefront.
//
// Sixteen lanes hold one matrix as a 4 x 4 grid of blocks: lane 4 rg + cg (a DPP row) holds rows rg + 4 s and columns
// cg + 4 t of the augmented system [I - V P | V], whose two halves are padded to whole slots.  The four matrices of a
// wavefront are four nodes of one q, so they share V(q).  Step K of the Gauss-Jordan elimination:
//  * the lanes of column K rank their unused rows by packed keys (|Re| + |Im| in FP32 bits, low bits 31 - row: ties go
//    to the lower row); two DPP row shifts and a row broadcast give the 16 lanes their matrix's pivot row;
//  * column K's entries reach the other columns by a DPP quad broadcast (registers only);
//  * the owners of the pivot row pass it through LDS (two buffers, alternating by step), and every lane subtracts
//    f_r (pivot row), f_r = m_r / a_pK, 1 - 1 / a_pK for the pivot row itself, which normalises it;
//  * column slots left of K drop out at compile time.
// In the layout with one matrix per wavefront (rows over 8 lanes, columns over 8) a lane reads 7 complex values from LDS
// for 8 multiply-adds in each step, and the pivot search and reciprocal serve one matrix.  Here a lane reads at most 9
// values for 32 multiply-adds and the search serves four matrices.  At N_b = 15, 24 x 24, r = 53 the vector unit is busy
// 48% of the time (FP32 73%) with 1.6 (2.2) wavefronts on a SIMD, 4-5% of their time waiting for LDS: the steps depend
// on each other, and the wavefronts that the LDS of a matrix lets in do not cover that.
#include "qgw_gj.h"
#include "qgw_internal.h"

#include <utility>

namespace qgw {

template <int NB>
struct WQ {
  static_assert(NB <= 16, "four row slots of four");
  static constexpr int RS = (NB + 3) / 4, CS = 2 * RS, NN = NB * NB;
  // LDS strides between the four matrices: 4 or 12 modulo 16 complex values, so that four matrices times four
  // columns fall into distinct banks
  static constexpr int PS = NN + (20 - NN % 16) % 16;
  static constexpr int EX = 4 * CS + 4;  // pivot row of one matrix and step
  static constexpr int SH = 4 * PS > 8 * EX ? 4 * PS : 8 * EX;  // P, then the pivot rows, then the result
};

// the owner lanes of a pivot row in slot S publish it from the slot of column K on and mark the row as used
template <typename T, int NB, int K, int S>
__device__ __forceinline__ void wq_publish(const cpx<T> (&x)[WQ<NB>::RS][WQ<NB>::CS], cpx<T>* ex, int cg, bool mine,
                                           int (&cs)[WQ<NB>::RS], int (&kof)[WQ<NB>::RS]) {
  if (mine) {
#pragma unroll
    for (int t = K / 4; t < WQ<NB>::CS; ++t) ex[cg + 4 * t] = x[S][t];
  }
  cs[S] |= mine ? int(0x80000000u) : 0;
  kof[S] = mine ? K : kof[S];
}

// cs[s] = 31 - row of a candidate row, with the sign bit set once it has pivoted (and for rows past N_b)
template <typename T, int NB, int K>
__device__ __forceinline__ void wq_step(cpx<T> (&x)[WQ<NB>::RS][WQ<NB>::CS], int (&cs)[WQ<NB>::RS],
                                        int (&kof)[WQ<NB>::RS], int rg, int cg, cpx<T>* xs, bool& singular) {
  constexpr int RS = WQ<NB>::RS, CS = WQ<NB>::CS, MIN = int(0x80000000u);
  constexpr int cgk = K % 4, tk = K / 4, t0 = (K + 1) / 4;
  int key = MIN;
#pragma unroll
  for (int s = 0; s < RS; ++s) key = max(key, (mag_bits(x[s][tk]) & ~31) | cs[s]);
  key = cg == cgk ? key : MIN;
  key = max(key, dpp_shl_i<0x108>(key));
  key = max(key, dpp_shl_i<0x104>(key));
  key = __builtin_amdgcn_update_dpp(key, key, 0x150 + cgk, 0xF, 0xF, false);  // from lane cgk of the matrix
  const int p = 31 - (key & 31);
  cpx<T>* ex = xs + (K & 1) * 4 * WQ<NB>::EX;
  wq_publish<T, NB, K, 0>(x, ex, cg, p == rg, cs, kof);
  if constexpr (RS > 1) wq_publish<T, NB, K, 1>(x, ex, cg, p == rg + 4, cs, kof);
  if constexpr (RS > 2) wq_publish<T, NB, K, 2>(x, ex, cg, p == rg + 8, cs, kof);
  if constexpr (RS > 3) wq_publish<T, NB, K, 3>(x, ex, cg, p == rg + 12, cs, kof);
  cpx<T> m[RS];
#pragma unroll
  for (int s = 0; s < RS; ++s) m[s] = dpp_move<0x55 * cgk>(x[s][tk]);
  __syncthreads();
  const cpx<T> pv = ex[K];
  const T pn = norm2(pv);
  singular |= !(pn > T(0)) || !isfinite(pn);  // exact zero, NaN or overflow (the same value in the matrix's lanes)
  const T d = rcp_nr(pn);
  const cpx<T> pinv = mk(pv.re * d, -pv.im * d);
  // the pivot row's own factor 1 - 1 / a_pK makes it (pivot row) / a_pK; formed from the reciprocal, one rounding
#pragma unroll
  for (int s = 0; s < RS; ++s) {
    m[s] = m[s] * pinv;
    if (rg + 4 * s == p) m[s] = mk(T(1) - pinv.re, -pinv.im);
  }
#pragma unroll
  for (int t = t0; t < CS; ++t) {
    const cpx<T> pc = ex[cg + 4 * t];
#pragma unroll
    for (int s = 0; s < RS; ++s) x[s][t] = fms(x[s][t], m[s], pc);
  }
}

template <typename T, int NB, int... K>
__device__ __forceinline__ void wq_all(cpx<T> (&x)[WQ<NB>::RS][WQ<NB>::CS], int (&cs)[WQ<NB>::RS],
                                       int (&kof)[WQ<NB>::RS], int rg, int cg, cpx<T>* xs, bool& singular,
                                       std::integer_sequence<int, K...>) {
  (wq_step<T, NB, K>(x, cs, kof, rg, cg, xs, singular), ...);
}

// On entry su holds V(q) and sp, at stride PS, the four matrices P; on return sp holds W^C = (I - V P)^{-1} V - V of
// each.  True for a lane of a matrix that met a zero or non-finite pivot.
template <typename T, int NB>
__device__ __forceinline__ bool wq_solve(const cpx<T>* su, cpx<T>* sp, int lane) {
  using S = WQ<NB>;
  constexpr int RS = S::RS, CS = S::CS, PS = S::PS;
  const int mw = lane >> 4, rg = (lane >> 2) & 3, cg = lane & 3;
  cpx<T> x[RS][CS];
  int cs[RS], kof[RS], row[RS];
#pragma unroll
  for (int s = 0; s < RS; ++s) {
    const int rr = rg + 4 * s;
    row[s] = min(rr, NB - 1);
    cs[s] = rr < NB ? 31 - rr : int(0x80000000u);
    kof[s] = 0;
#pragma unroll
    for (int t = 0; t < RS; ++t) x[s][t] = mk(T(0), T(0));
  }
  const cpx<T>* pm = sp + mw * PS;
#pragma unroll 3
  for (int j = 0; j < NB; ++j) {
    cpx<T> u[RS], pj[RS];
#pragma unroll
    for (int s = 0; s < RS; ++s) u[s] = su[row[s] * NB + j];
#pragma unroll
    for (int t = 0; t < RS; ++t) pj[t] = pm[j * NB + min(cg + 4 * t, NB - 1)];
#pragma unroll
    for (int s = 0; s < RS; ++s)
#pragma unroll
      for (int t = 0; t < RS; ++t) x[s][t] = fma(x[s][t], u[s], pj[t]);
  }
#pragma unroll
  for (int s = 0; s < RS; ++s)
#pragma unroll
    for (int t = 0; t < RS; ++t) {
      const bool in = rg + 4 * s < NB && cg + 4 * t < NB;
      x[s][t] = in ? mk(T(rg + 4 * s == cg + 4 * t ? 1 : 0) - x[s][t].re, -x[s][t].im) : mk(T(0), T(0));
      x[s][RS + t] = in ? su[row[s] * NB + cg + 4 * t] : mk(T(0), T(0));
    }
  __syncthreads();  // P has been read: its area takes the pivot rows
  bool singular = false;
  wq_all<T, NB>(x, cs, kof, rg, cg, sp + mw * S::EX, singular, std::make_integer_sequence<int, NB>{});
  __syncthreads();  // the pivot rows have been read: the area takes W^C
#pragma unroll
  for (int s = 0; s < RS; ++s)
#pragma unroll
    for (int t = 0; t < RS; ++t) {
      const int col = cg + 4 * t, k = kof[s];  // row r of the right-hand side is row kof of the solution
      if (rg + 4 * s < NB && col < NB) sp[mw * PS + k * NB + col] = x[s][RS + t] - su[k * NB + col];
    }
  __syncthreads();
  return singular;
}

// block (q, group of four nodes); guarded: only a q whose first matrix of the group carries the folded kernel's mark
// (that kernel takes or leaves all nodes of a q alike)
template <typename T, int NB>
__global__ __launch_bounds__(64) void k_dyson_wq(const cpx<T>* __restrict__ vq, const cpx<T>* __restrict__ pnu,
                                                 cpx<T>* __restrict__ wc, int r, int nk, int64_t ld,
                                                 int* __restrict__ cond, int guarded) {
  using S = WQ<NB>;
  constexpr int NN = S::NN, PS = S::PS;
  __shared__ cpx<T> su[NN];
  __shared__ cpx<T> sp[S::SH];
  const int lane = threadIdx.x;
  const int q = int(blockIdx.x % unsigned(nk)), m0 = 4 * int(blockIdx.x / unsigned(nk));
  const int nv = min(4, r - m0);
  if constexpr (sizeof(T) == 8) {
    if (guarded && !is_left_mark(wc[(int64_t(m0) * nk + q) * ld])) return;
  }
  for (int e = lane; e < NN; e += 64) su[e] = vq[int64_t(q) * NN + e];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const cpx<T>* src = pnu + (int64_t(min(m0 + i, r - 1)) * nk + q) * NN;  // nodes past r repeat the last one
    for (int e = lane; e < NN; e += 64) sp[i * PS + e] = src[e];
  }
  __syncthreads();
  const bool singular = wq_solve<T, NB>(su, sp, lane);
  if (singular && (lane >> 4) < nv && (lane & 15) == 0) atomicOr(cond, kCondSingular);
  for (int i = 0; i < nv; ++i) {
    cpx<T>* dst = wc + (int64_t(m0 + i) * nk + q) * ld;
    for (int e = lane; e < NN; e += 64) dst[e] = sp[i * PS + e];
  }
}

// The same solve on full NF x NF pair matrices through the folded basis (NB classes): where V(q) is unchanged under
// i <-> l of both indices, P is summed over the members of its classes as it is read and W^C written to every member;
// elsewhere the group's matrices are marked and left to the general kernel.  FP64 (FP32 calls keep their kernels).
template <int NB, int NF>
__global__ __launch_bounds__(64) void k_dyson_wq_fold(const zd* __restrict__ vq, const zd* __restrict__ pnu,
                                                      zd* __restrict__ wc, int r, int nk, int64_t ld,
                                                      int* __restrict__ cond, const int* __restrict__ fold) {
  using T = double;
  using S = WQ<NB>;
  constexpr int NN = S::NN, PS = S::PS, FF = NF * NF;
  __shared__ cpx<T> su[NN];
  __shared__ cpx<T> sp[S::SH];
  const int lane = threadIdx.x;
  const int q = int(blockIdx.x % unsigned(nk)), m0 = 4 * int(blockIdx.x / unsigned(nk));
  const int nv = min(4, r - m0);
  const int *cls = fold + 2 * NB, *partner = cls + NF, *rep = partner + NF;
  const cpx<T>* vm = vq + int64_t(q) * FF;
  // V(q) against its exchanged partners; a V without the symmetry mostly shows it in the first 64 entries
  auto differs = [&](int e) {
    const int a = e / NF, b = e - a * NF;
    const cpx<T> v = vm[e], x = vm[partner[a] * NF + b], y = vm[a * NF + partner[b]];
    return !(v.re == x.re && v.im == x.im && v.re == y.re && v.im == y.im);
  };
  bool bad = differs(lane);
  if (!__any(bad))
    for (int e = lane + 64; e < FF; e += 64) bad |= differs(e);
  if (__any(bad)) {
    if (lane < nv) wc[(int64_t(m0 + lane) * nk + q) * ld] = left_mark();
    return;
  }
  for (int e = lane; e < NN; e += 64) {
    const int u = e / NB, v = e - u * NB;
    const int ra = rep[u], rb = partner[ra], ca = rep[v], cb = partner[ca];
    su[e] = vm[ra * NF + ca];
    const int o0 = ra * NF + ca, o1 = rb * NF + ca, o2 = ra * NF + cb, o3 = rb * NF + cb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const cpx<T>* src = pnu + (int64_t(min(m0 + i, r - 1)) * nk + q) * FF;
      const cpx<T> p0 = src[o0], p1 = src[o1], p2 = src[o2], p3 = src[o3];
      cpx<T> s = p0;
      if (rb != ra) s = s + p1;
      if (cb != ca) s = s + (rb != ra ? p2 + p3 : p2);
      sp[i * PS + e] = s;
    }
  }
  __syncthreads();
  const bool singular = wq_solve<T, NB>(su, sp, lane);
  if (singular && (lane >> 4) < nv && (lane & 15) == 0) atomicOr(cond, kCondSingular);
  for (int e = lane; e < FF; e += 64) {
    const int a = e / NF, b = e - a * NF, o = cls[a] * NB + cls[b];
    for (int i = 0; i < nv; ++i) wc[(int64_t(m0 + i) * nk + q) * ld + e] = sp[i * PS + o];
  }
}

namespace {

unsigned wq_blocks(const Plan& p) { return unsigned(int64_t((p.r + 3) / 4) * p.nk); }

template <typename T, int NB>
hipError_t wq_nb(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, int64_t ld, hipStream_t s, int guarded) {
  hipLaunchKernelGGL((k_dyson_wq<T, NB>), dim3(wq_blocks(p)), dim3(64), 0, s, (const cpx<T>*)v_q, (const cpx<T>*)p_nu,
                     (cpx<T>*)wc_nu, p.r, p.nk, ld, p.d_status + kCondWord, guarded);
  return hipGetLastError();
}

template <int NB, int NF>
hipError_t wq_fold(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, int64_t ld, hipStream_t s) {
  hipLaunchKernelGGL((k_dyson_wq_fold<NB, NF>), dim3(wq_blocks(p)), dim3(64), 0, s, (const zd*)v_q, (const zd*)p_nu,
                     (zd*)wc_nu, p.r, p.nk, ld, p.d_status + kCondWord, p.d_fold_pairs);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_dyson_wq(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, int64_t ld, hipStream_t s,
                           int guarded) {
  switch (p.nb) {
#define QGW_CASE(NBV)                                                                         \
  case NBV:                                                                                   \
    return p.prec == 0 ? wq_nb<double, NBV>(p, v_q, p_nu, wc_nu, ld, s, guarded)              \
                       : wq_nb<float, NBV>(p, v_q, p_nu, wc_nu, ld, s, guarded);
    QGW_FOR_EACH_NB_WQ(QGW_CASE)
#undef QGW_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_dyson_wq_fold(const Plan& p, const void* v_q, const void* p_nu, void* wc_nu, int64_t ld,
                                hipStream_t s) {
  if (p.prec != 0) return hipErrorInvalidValue;
#define QGW_CASE(NFV, NBV) \
  if (p.nb == NFV && p.fold_nb == NBV) return wq_fold<NBV, NFV>(p, v_q, p_nu, wc_nu, ld, s);
  QGW_FOR_EACH_FOLD(QGW_CASE)
#undef QGW_CASE
  return hipErrorInvalidValue;
}

}  // namespace qgw

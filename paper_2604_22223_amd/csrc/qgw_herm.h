// Per-thread eigen-decomposition of small Hermitian matrices held in
// registers (n_o <= 8), for the static problems per k: the quasiparticle
// Hamiltonian and the Hartree-Fock density.  Cyclic complex Jacobi (round-robin order): each
// rotation first turns a_pq real with a phase on column q, then zeroes it
// with a real plane rotation; sweeps stop at an off-diagonal norm below
// 1e-30 of the total (at most 30 sweeps).
#pragma once

#include "qgw_gj.h"
#include "qgw_internal.h"

namespace qgw {

template <int NO>
struct HermEig {
  cpx<double> a[NO][NO];  // in: Hermitian matrix; out: diagonal holds the eigenvalues
  cpx<double> v[NO][NO];  // eigenvectors (columns)
};

template <int NO>
__device__ __forceinline__ double offdiag2(const cpx<double> (&a)[NO][NO], double& total) {
  double off = 0.0, all = 0.0;
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      const double v = norm2(a[i][j]);
      all += v;
      if (i != j) off += v;
    }
  total = all;
  return off;
}

// One thread per matrix leaves few wavefronts in flight, so the serial chain of a rotation bounds the solve.  No branch
// on a vanishing a_pq (the angle is then zero), so that the disjoint rotations of a round (see jacobi_round) can
// overlap; reciprocals and square roots by rsqrt and Newton steps.  n_o = 5, 576 matrices: 34 -> 31 us; a whole
// density call 126 -> 94 us at n_o = 5, 166 -> 119 us at 6 (with the search's change in kernels_hf.hip).
template <int NO, int P, int Q>
__device__ __forceinline__ void jacobi_rotate(HermEig<NO>& h) {
  const cpx<double> apq = h.a[P][Q];
  const double n2 = norm2(apq);
  const bool zero = n2 < 1e-300;
  const double rg = rsqrt(zero ? 1.0 : n2);  // 1 / |a_pq|
  const cpx<double> e = zero ? mk(1.0, 0.0) : scale(apq, rg);  // a_pq = |a_pq| e
  const double app = h.a[P][P].re, aqq = h.a[Q][Q].re;
  const double tau = fmin(fmax(0.5 * (aqq - app) * rg, -1e140), 1e140);
  const double w = 1.0 + tau * tau;
  const double t = zero ? 0.0 : (tau >= 0.0 ? 1.0 : -1.0) * rcp_nr(fabs(tau) + w * rsqrt(w));
  const double c = rsqrt(1.0 + t * t), s = t * c;
  // W on the (P, Q) plane: W_PP = c, W_PQ = s, W_QP = -s conj(e), W_QQ = c conj(e)
  const cpx<double> ce = conj(e);
  // columns: A <- A W, V <- V W
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const cpx<double> ap = h.a[i][P], aq = h.a[i][Q];
    h.a[i][P] = scale(ap, c) - scale(aq * ce, s);
    h.a[i][Q] = scale(ap, s) + scale(aq * ce, c);
    const cpx<double> vp = h.v[i][P], vq = h.v[i][Q];
    h.v[i][P] = scale(vp, c) - scale(vq * ce, s);
    h.v[i][Q] = scale(vp, s) + scale(vq * ce, c);
  }
  // rows: A <- W^H A (W^H_PP = c, W^H_PQ = -s e, W^H_QP = s, W^H_QQ = c e)
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    const cpx<double> ap = h.a[P][j], aq = h.a[Q][j];
    h.a[P][j] = scale(ap, c) - scale(e * aq, s);
    h.a[Q][j] = scale(ap, s) + scale(e * aq, c);
  }
  h.a[P][Q] = mk(0.0, 0.0);
  h.a[Q][P] = mk(0.0, 0.0);
  h.a[P][P].im = 0.0;
  h.a[Q][Q].im = 0.0;
}

// a sweep in the order of a round robin: round R rotates the disjoint planes {i, j} with i + j = 2 R (mod M - 1), M = n_o
// rounded up to even, and {R, M - 1}; with n_o odd the index M - 1 does not exist and R rests
template <int NO, int R, int I>
__device__ __forceinline__ void jacobi_round(HermEig<NO>& h) {
  constexpr int M = NO + (NO & 1);
  if constexpr (I < M / 2) {
    constexpr int A = I == 0 ? R : (R + I) % (M - 1), B = I == 0 ? M - 1 : (R - I + M - 1) % (M - 1);
    constexpr int P = A < B ? A : B, Q = A < B ? B : A;
    if constexpr (Q < NO) {
      if constexpr (NO < 7)
        jacobi_rotate<NO, P, Q>(h);
      else if (norm2(h.a[P][Q]) >= 1e-300)  // one at a time: overlapped ones spill (n_o = 8: 422 -> 475 us)
        jacobi_rotate<NO, P, Q>(h);
    }
    jacobi_round<NO, R, I + 1>(h);
  }
}

template <int NO, int R>
__device__ __forceinline__ void jacobi_sweep(HermEig<NO>& h) {
  if constexpr (R < NO + (NO & 1) - 1) {
    jacobi_round<NO, R, 0>(h);
    jacobi_sweep<NO, R + 1>(h);
  }
}

template <int NO>
__device__ __forceinline__ void herm_eig(HermEig<NO>& h) {
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = 0; j < NO; ++j) h.v[i][j] = mk(i == j ? 1.0 : 0.0, 0.0);
  for (int sweep = 0; sweep < 30; ++sweep) {
    double total = 0.0;
    const double off = offdiag2<NO>(h.a, total);
    if (!(off > 1e-30 * total)) break;
    jacobi_sweep<NO, 0>(h);
  }
}

// out = V diag(f) V^H, Hermitian by construction
template <int NO>
__device__ __forceinline__ void spectral(const cpx<double> (&v)[NO][NO], const double (&f)[NO],
                                         cpx<double> (&out)[NO][NO]) {
#pragma unroll
  for (int i = 0; i < NO; ++i)
#pragma unroll
    for (int j = 0; j < NO; ++j) {
      cpx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int n = 0; n < NO; ++n) acc = acc + scale(v[i][n] * conj(v[j][n]), f[n]);
      out[i][j] = acc;
    }
}

}  // namespace qgw

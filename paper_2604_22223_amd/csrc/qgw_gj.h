// Helpers of the register Gauss-Jordan solvers (pivot keys, cross-lane moves, reciprocal).
#pragma once
#include "qgw_complex.h"

namespace qgw {

// The mark that the folded Dyson-W kernel leaves in the first entry of a matrix it has not solved (a NaN pair that no
// arithmetic makes).  A solved matrix that held it all the same would be solved once more by the general kernel.
__device__ __forceinline__ cpx<double> left_mark() {
  return mk(__longlong_as_double(0x7ff85157475f5701ll), __longlong_as_double(0x7ff85157475f5702ll));
}
__device__ __forceinline__ bool is_left_mark(cpx<double> v) {
  return __double_as_longlong(v.re) == 0x7ff85157475f5701ll && __double_as_longlong(v.im) == 0x7ff85157475f5702ll;
}

// row shift by DPP; a lane whose source lies outside its row gets INT_MIN, the identity of the max it feeds, so the
// shift folds into the max instruction (no copy of the value first)
template <int CTRL>
__device__ __forceinline__ int dpp_shl_i(int v) {
  return __builtin_amdgcn_update_dpp(int(0x80000000u), v, CTRL, 0xF, 0xF, false);
}

// 1 / d by the hardware estimate and Newton-Raphson steps r <- r (2 - d r)
__device__ __forceinline__ double rcp_nr(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = __builtin_fma(-d, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float rcp_nr(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(r, __builtin_fmaf(-d, r, 1.0f), r);
}

// |Re| + |Im| rounded to FP32, as bits; a larger value compares larger
template <typename T>
__device__ __forceinline__ int mag_bits(cpx<T> a) {
  return __float_as_int(float(fabs(a.re) + fabs(a.im)));
}

// a value of any 32-bit-multiple size through one DPP control (every source lane exists)
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_move(T v) {
  static_assert(sizeof(T) % 4 == 0, "32-bit words");
  int w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < int(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_update_dpp(w[i], w[i], CTRL, 0xF, 0xF, false);
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

}  // namespace qgw

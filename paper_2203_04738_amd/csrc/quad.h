// Contraction of four rows with sixteen weight columns per gate, weights in registers.
//
// v_mfma_f32_4x4x1_16b_f32 holds 16 blocks of 4 rows x 4 columns, one k each.  With CBSZ = 2 the A
// block `abid` of each group of four is broadcast to the group, so a group (16 lanes) contracts
// 4 rows x 16 columns over its own k and the four groups split K:
//   A: lane l holds rows l % 4 at k = 4 (l / 4) + e (one 16-byte load per 64 k);
//   B: lane l holds column l % 16 at k = 16 (l / 16) + 4 abid + e;
//   D: register v of lane l is row v, column l % 16, summed over the k of group l / 16.
#pragma once
#include "gemm_core.h"

namespace mg {

// Sum of the four k-groups of a 4-row x 16-column block: in, register v of lane l is row v, column
// l % 16 of group l / 16; out, lane l holds row quad_row(l), column l % 16 of the sum.
__device__ inline float quad_fold(const floatx4& a) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  auto add = [](u2 s) { return __uint_as_float(s[0]) + __uint_as_float(s[1]); };
  auto u = [](float f) { return __float_as_uint(f); };
  const float x01 = add(__builtin_amdgcn_permlane32_swap(u(a[0]), u(a[1]), false, false));
  const float x23 = add(__builtin_amdgcn_permlane32_swap(u(a[2]), u(a[3]), false, false));
  return add(__builtin_amdgcn_permlane16_swap(u(x01), u(x23), false, false));
}
__device__ inline int quad_row(int lane) { return ((lane >> 5) & 1) + 2 * ((lane >> 4) & 1); }

// acc[r][g] += A_rg (64 k of four rows, see above) * the sixteen weights of gate g at those k; the
// sums of the gates and row groups alternate, so that consecutive MFMAs do not wait for each other
// (a lone sum is kept as two).
template <int RB, int NG, int NP, class GetA, class GetW>
__device__ inline void quad_mma(floatx4 (&acc)[RB][NG][NP], GetA getA, GetW getW) {
#define MG_QUAD_STEP(E, A)                                                                       \
  _Pragma("unroll") for (int r = 0; r < RB; ++r) _Pragma("unroll") for (int g = 0; g < NG; ++g)  \
      acc[r][g][A % NP] = __builtin_amdgcn_mfma_f32_4x4x1f32(                                    \
          getA(r, g)[E], getW(g)[4 * A + E], acc[r][g][A % NP], 2, A, 0);
#define MG_QUAD_E(E) MG_QUAD_STEP(E, 0) MG_QUAD_STEP(E, 1) MG_QUAD_STEP(E, 2) MG_QUAD_STEP(E, 3)
  MG_QUAD_E(0) MG_QUAD_E(1) MG_QUAD_E(2) MG_QUAD_E(3)
#undef MG_QUAD_E
#undef MG_QUAD_STEP
}

}  // namespace mg

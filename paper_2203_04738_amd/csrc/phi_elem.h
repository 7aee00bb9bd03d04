// One element of the GRU level step: its operands, gates, update and the outputs of the epilogue
// modes.  Shared by the forward kernels.
#pragma once
#include "common.h"
#include "gates.h"

namespace mg {

// Operands of one output element that do not depend on the contraction: they are
// loaded separately so that the few-row kernel can fetch them before its dot
// products instead of after.
struct PhiEpiIn {
  float pr, pz, pn, h, gval, cur;
  float pr2, pz2, pn2, cur2;     // STEP_RELAX_RHS: projection and current value of the coarse step
  float prep;                    // STEP_RESID with resid_adds: the prepared half of the right-hand side
};
// Element offsets (column 0) of one row (level point, batch element) of a launch into
// the arrays the epilogue touches: input state, projection, out/cur/g, and the coarse
// (or coefficient) array.  Computed once per tile row and kept in LDS: the index
// arithmetic (a division by B and 64-bit products) is not repeated per element.
struct PhiRow {
  long long in, p, o, a;
};
__device__ inline PhiRow phi_row(const PhiArgs& a, long long r, int aux_width) {
  const long long pt = (unsigned)r / (unsigned)a.B;   // rows < 2^31: 32-bit division
  const int b = (int)(r - pt * a.B);
  PhiRow ro;
  ro.in = (a.in.at(pt) * a.B + b) * a.H;
  ro.p = (a.p.at(pt) * a.B + b) * (3LL * a.H);
  ro.o = (a.o.at(pt) * a.B + b) * a.H;
  ro.a = ((aux_width == a.H ? a.a.at(pt) : a.o.at(pt)) * a.B + b) * (long long)aux_width;
  // (row offsets are multiples of four elements: bit 0 marks the coarse points of ff_cf / ff_rem)
  if (a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem) ro.a |= 1;
  return ro;
}
// STEP_RELAX_KAPPA2: element offset of the row's coarse output point (index a) in the coarse
// level's coefficient array (4H wide).
__device__ inline long long phi_row_coarse_kappa(const PhiArgs& a, long long r) {
  const long long pt = (unsigned)r / (unsigned)a.B;
  const int b = (int)(r - pt * a.B);
  return (a.a.at(pt) * a.B + b) * (4LL * a.H);
}
struct PhiBias {          // recurrent biases of one hidden column
  float r, z, n;
};
__device__ inline PhiBias phi_bias_load(const PhiArgs& a, int j) {
  return PhiBias{a.b_h[j], a.b_h[a.H + j], a.b_h[2 * a.H + j]};
}

template <int MODE>
__device__ inline PhiEpiIn phi_epi_load(const PhiArgs& a, const PhiRow& ro, int j) {
  const int H = a.H;
  PhiEpiIn e;
  const float* pp = a.P + ro.p;
  e.pr = pp[j];
  e.pz = pp[H + j];
  e.pn = pp[2 * H + j];
  e.h = a.u_in[ro.in + j];
  const long long oi = ro.o + j;
  e.gval = (MODE != STEP_KAPPA && a.g) ? a.g[oi] : 0.f;
  e.cur = (MODE == STEP_RESID || MODE == STEP_RHS) ? a.u[oi] : 0.f;
  e.pr2 = e.pz2 = e.pn2 = e.cur2 = e.prep = 0.f;
  if (MODE == STEP_RELAX_RHS || MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK) {
    const float* p2 = pp + a.dp2;
    e.pr2 = p2[j];
    e.pz2 = p2[H + j];
    e.pn2 = p2[2 * H + j];
    if (MODE == STEP_RELAX_RHS) e.cur2 = a.u[oi + a.do2];
  }
  if (MODE == STEP_RESID && a.resid_adds) e.prep = a.gc[(ro.a & ~1LL) + j];
  return e;
}

// Gates of Eq. 1, the update of Eq. 16 / Eq. 3 and the mode-specific outputs of one
// element, given the three recurrent contractions (U_r h)_j, (U_z h)_j, (U_n h)_j.
//   RELAX: v0 = new state (+ g)          RESID: v0 = -r (coarse right-hand side), v1 = cur
//   RHS:   v0 = cur - step + g           KAPPA: v0..v4 = k_r, k_z, k_q, k_d, k_n
struct PhiOut {
  float v0, v1, v2, v3, v4, v5;       // v5: new state (+ g) of STEP_RELAX_KAPPA
  float c0, c1, c2, c3;               // STEP_RELAX_KAPPA2: k_r, k_z, k_q, k_d of the coarse step
};
// Coefficient vectors of the transposed Jacobian of one step (Appendix A.2), from its gates.
struct PhiKappa {
  float kr, kz, kq, kd, kn;
};
__device__ inline PhiKappa phi_kappa(float gamma, bool implicit, float h, float rg, float zg,
                                     float q, float n, float c, float rd, float hn) {
  float kd, dn, dz;
  if (implicit) {
    kd = rd;
    dn = gamma * c * rd;
    dz = -gamma * (n - hn) * rd;
  } else {
    kd = 1.0f - gamma * c;
    dn = gamma * c;
    dz = -gamma * (n - h);
  }
  const float kn = dn * (1.0f - n * n);
  return PhiKappa{kn * q * rg * (1.0f - rg), dz * zg * (1.0f - zg), kn * rg, kd, kn};
}
template <int MODE>
__device__ inline PhiOut phi_elem(float gamma, bool implicit, float sr, float sz, float sn,
                                  const PhiEpiIn& e, const PhiBias& bh, float gamma2 = 0.f) {
  const float h = e.h;
  const float rg = sigmoidf_(e.pr + sr + bh.r);
  const float zg = sigmoidf_(e.pz + sz + bh.z);
  const float q = sn + bh.n;
  const float n = tanhf_(e.pn + rg * q);
  const float c = 1.0f - zg;
  const float d = 1.0f + gamma * c;
  const float rd = fast_rcp(d);
  const float hn = implicit ? (h + gamma * c * n) * rd : h + gamma * c * (n - h);
  PhiOut o{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2) o.v5 = hn + e.gval;
  if (MODE == STEP_RELAX) {
    o.v0 = hn + e.gval;
  } else if (MODE == STEP_RELAX_RHS) {
    o.v0 = hn + e.gval;
    // the coarse level's step from the same state: same sums, its own projection and step size
    const float rg2 = sigmoidf_(e.pr2 + sr + bh.r);
    const float zg2 = sigmoidf_(e.pz2 + sz + bh.z);
    const float n2 = tanhf_(e.pn2 + rg2 * q);
    const float c2 = 1.0f - zg2;
    const float hn2 = implicit ? (h + gamma2 * c2 * n2) * fast_rcp(1.0f + gamma2 * c2)
                               : h + gamma2 * c2 * (n2 - h);
    o.v1 = e.cur2 - hn2;
  } else if (MODE == STEP_RELAX_CK) {
    o.v0 = hn + e.gval;
    // coefficient vectors of the coarser level's step from the same state
    const float rg2 = sigmoidf_(e.pr2 + sr + bh.r);
    const float zg2 = sigmoidf_(e.pz2 + sz + bh.z);
    const float n2 = tanhf_(e.pn2 + rg2 * q);
    const float c2 = 1.0f - zg2;
    const float rd2 = fast_rcp(1.0f + gamma2 * c2);
    const float hn2 = implicit ? (h + gamma2 * c2 * n2) * rd2 : h + gamma2 * c2 * (n2 - h);
    const PhiKappa k2 = phi_kappa(gamma2, implicit, h, rg2, zg2, q, n2, c2, rd2, hn2);
    o.c0 = k2.kr;
    o.c1 = k2.kz;
    o.c2 = k2.kq;
    o.c3 = k2.kd;
  } else if (MODE == STEP_RESID) {
    o.v0 = -(e.cur - hn - e.gval);
    o.v1 = e.cur;
  } else if (MODE == STEP_RHS) {
    o.v0 = (e.cur - hn) + e.gval;
  } else {  // STEP_KAPPA (and the relaxation modes that keep them): coefficients of this step
    const PhiKappa k = phi_kappa(gamma, implicit, h, rg, zg, q, n, c, rd, hn);
    o.v0 = k.kr;
    o.v1 = k.kz;
    o.v2 = k.kq;
    o.v3 = k.kd;
    o.v4 = k.kn;
    if (MODE == STEP_RELAX_KAPPA2) {
      // the coarse level's step from the same state: same sums, its own projection and step size
      const float rg2 = sigmoidf_(e.pr2 + sr + bh.r);
      const float zg2 = sigmoidf_(e.pz2 + sz + bh.z);
      const float n2 = tanhf_(e.pn2 + rg2 * q);
      const float c2 = 1.0f - zg2;
      const float rd2 = fast_rcp(1.0f + gamma2 * c2);
      const float hn2 = implicit ? (h + gamma2 * c2 * n2) * rd2 : h + gamma2 * c2 * (n2 - h);
      const PhiKappa k2 = phi_kappa(gamma2, implicit, h, rg2, zg2, q, n2, c2, rd2, hn2);
      o.c0 = k2.kr;
      o.c1 = k2.kz;
      o.c2 = k2.kq;
      o.c3 = k2.kd;
    }
  }
  return o;
}

}  // namespace mg

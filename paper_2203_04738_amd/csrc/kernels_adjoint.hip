// Adjoint kernels: the fused transposed-Jacobian level step
//   w_out = k_d*w + U_r^T(k_r*w) + U_z^T(k_z*w) + U_n^T(k_q*w)
// (discrete adjoint of Eq. 16 / Eq. 3, Appendix A.2) with the same MGRIT
// epilogues as the forward step, the transposition of U it contracts with, and
// the parameter-gradient reductions of Alg. 3's gradient line.
#include "common.h"
#include "gemm_core.h"
#include "gemm_core_bf16.h"
#include "gemm_terms.h"
#include "skinny.h"

namespace mg {

// ---------------------------------------------------------------------------
// Adjoint level step: out[R,H] = (kap[:, 0:3H] * (w,w,w))[R,3H] . UT[H,3H]^T + k_d*w
// ---------------------------------------------------------------------------
// Operands of one output element that do not depend on the contraction.
struct AdjEpiIn {
  float kd, wv, gval, cur;
};
// Element offsets (column 0) of one row of a launch: input adjoint, coefficient row,
// out/cur/g, coarse array.  Computed once per tile row and kept in LDS.
struct AdjRow {
  long long in, k, o, a;
};
__device__ inline AdjRow adj_row(const AdjArgs& a, long long r) {
  const long long pt = (unsigned)r / (unsigned)a.B;   // rows < 2^31: 32-bit division
  const int b = (int)(r - pt * a.B);
  AdjRow ro;
  ro.in = (a.in.at(pt) * a.B + b) * a.H;
  ro.k = (a.k.at(pt) * a.B + b) * (long long)a.kw;
  ro.o = (a.o.at(pt) * a.B + b) * a.H;
  ro.a = (a.a.at(pt) * a.B + b) * a.H;
  // (row offsets are multiples of four elements: bit 0 marks the coarse points of ff_cf / ff_rem)
  if (a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem) ro.a |= 1;
  return ro;
}

template <int MODE>
__device__ inline AdjEpiIn adj_epi_load(const AdjArgs& a, const AdjRow& ro, int j) {
  AdjEpiIn e;
  e.kd = a.kap[ro.k + 3 * a.H + j];
  e.wv = a.w_in[ro.in + j];
  const long long oi = ro.o + j;
  e.gval = a.g ? a.g[oi] : 0.f;
  e.cur = MODE == STEP_RESID ? a.w[oi] : 0.f;
  return e;
}

// Output of one element of the adjoint step: row (point pt, batch b), column j, given
// the contraction  sum_g (U_g^T (k_g * w))_j.
template <int MODE>
__device__ inline void adj_epi_finish(const AdjArgs& a, const AdjRow& ro, int j, float dot,
                                      const AdjEpiIn& e, double& nrm) {
  const float wn = e.kd * e.wv + dot;
  const long long oi = ro.o + j;
  if (MODE == STEP_RELAX) {
    a.w[oi] = wn + e.gval;
  } else {  // STEP_RESID
    const float res = e.cur - wn - e.gval;
    const long long ai = (ro.a & ~1LL) + j;
    a.gc[ai] = -res;
    a.wc[ai] = (ro.a & 1) ? -res : 0.f;                // zero guess; -r at the marked points
    nrm += (double)res * (double)res;
  }
}

// Epilogue of one MFMA tile over the staged sums (see EpiStage).
struct AdjEpiIn4 {
  floatx4 kd, wv, gval, cur;
};
template <class C, int MODE>
__device__ inline void adj_tile_epilogue(const AdjArgs& a, const typename TileSums<C>::type& acc, const AdjRow* rowtab,
                                         float* stage, long long m0, int n0, long long R,
                                         double& nrm) {
  typedef EpiStage<C> E;
  const int H = a.H;
  const int c4 = E::col4();
  const int j = n0 + c4 * 4;
  const bool colok = E::active() && j < H;
  const int jc = colok ? j : H - 4;                     // clamped columns are never stored
#pragma unroll
  for (int ba = 0; ba < C::BM; ++ba) {
    __syncthreads();                                    // staging area no longer read
    stage_write<C>(acc, ba, stage);
    AdjEpiIn4 in[E::ITEMS];
    long long oo[E::ITEMS], oa[E::ITEMS];
    int trow[E::ITEMS];
#pragma unroll
    for (int it = 0; it < E::ITEMS; ++it) {
      trow[it] = E::tile_row(E::staged_row(it), ba);
      const AdjRow ro = rowtab[trow[it]];               // rows beyond the launch hold its last row
      oo[it] = ro.o;
      oa[it] = ro.a;
      in[it].kd = ldg4(a.kap + ro.k + 3 * H + jc);
      in[it].wv = ldg4(a.w_in + ro.in + jc);
      in[it].gval = a.g ? ldg4(a.g + ro.o + jc) : zero4();
      in[it].cur = MODE == STEP_RESID ? ldg4(a.w + ro.o + jc) : zero4();
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < E::ITEMS; ++it) {
      const floatx4 dot = E::read(stage, 0, E::staged_row(it), c4);
      if (!colok || m0 + trow[it] >= R) continue;
      const floatx4 wn = in[it].kd * in[it].wv + dot;
      const long long oi = oo[it] + j;
      if (MODE == STEP_RELAX) {
        *reinterpret_cast<floatx4*>(a.w + oi) = wn + in[it].gval;
      } else {  // STEP_RESID
        const floatx4 res = in[it].cur - wn - in[it].gval;
        const long long ai = (oa[it] & ~1LL) + j;
        *reinterpret_cast<floatx4*>(a.gc + ai) = -res;
        // zero guess of the coarse error equation; -r at the marked points
        *reinterpret_cast<floatx4*>(a.wc + ai) = (oa[it] & 1) ? -res : zero4();
#pragma unroll
        for (int i = 0; i < 4; ++i) nrm += (double)res[i] * (double)res[i];
      }
    }
  }
}

struct KapW {
  floatx4 kap, w;
};

template <class C, int MODE>
__global__ __launch_bounds__(C::NT, C::MINWG) void adj_step_kernel(AdjArgs a) {
  constexpr int LDSF =
      C::LDS_FLOATS > EpiStage<C>::FLOATS ? C::LDS_FLOATS : EpiStage<C>::FLOATS;
  __shared__ __attribute__((aligned(16))) float lds[LDSF];
  const int H = a.H, B = a.B, K = 3 * a.H;
  const long long R = (long long)a.nk * B;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (H + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const int tid = threadIdx.x;
  __shared__ AdjRow rowtab[C::TM];
  if (tid < C::TM) {
    long long r = m0 + tid;
    if (r >= R) r = R - 1;
    rowtab[tid] = adj_row(a, r);
  }
  // (visible to all waves after the barriers inside the contraction)

  const float* krow[C::A_CHUNKS];
  const float* wrow[C::A_CHUNKS];
  const float* brow[C::B_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row<C>(s);
    if (r >= R) r = R - 1;     // clamped rows are never stored
    const long long pt = (unsigned)r / (unsigned)B;   // rows < 2^31: 32-bit division
    const int b = (int)(r - pt * B);
    krow[s] = a.kap + (a.k.at(pt) * B + b) * (long long)a.kw;
    wrow[s] = a.w_in + (a.in.at(pt) * B + b) * H;
  }
#pragma unroll
  for (int s = 0; s < C::B_CHUNKS; ++s) {
    int j = n0 + chunk_row<C>(s);
    if (j >= H) j = H - 1;
    brow[s] = (const float*)a.UT + (long long)j * K;
  }
  Acc<C> acc;
  acc.zero();
  // A operand: kappa and w stay raw in registers during the MFMAs of the current
  // slice and are multiplied when the slice is written to LDS
  auto la = [&](int s, int k) {
    const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
    return KapW{ldg4(krow[s] + k), ldg4(wrow[s] + kk)};
  };
  auto lb = [&](int s, int k) { return ldg4(brow[s] + k); };
  auto fa = [](const KapW& r) { return r.kap * r.w; };
  if (K % C::TK == 0 && C::KS == 1 && C::BM * C::BN >= 4) {
    // Whole slices per gate (H is a multiple of the slice width): the sum over k may run
    // in any slice order, so slice i takes gate i % 3 and the columns of slice i / 3 of
    // that gate.  The three slices that multiply the same columns of w then follow each
    // other, and w is loaded for the first of them only.
    floatx4 wkeep[C::A_CHUNKS];
    auto col = [&](int k, int& kk) {
      const int i = k / C::TK;
      const int g = i % 3;
      kk = (i / 3) * C::TK + (k - i * C::TK);
      return g;
    };
    auto lag = [&](int s, int k) {
      int kk;
      const int g = col(k, kk);
      if (g == 0) wkeep[s] = ldg4(wrow[s] + kk);
      return KapW{ldg4(krow[s] + g * H + kk), wkeep[s]};
    };
    auto lbg = [&](int s, int k) {
      int kk;
      const int g = col(k, kk);
      return ldg4(brow[s] + g * H + kk);
    };
    gemm_nt_tile<C, false>(acc, K, lag, lbg, fa, Identity4(), lds);
  } else if (K % C::TK == 0) {
    gemm_nt_tile<C, false>(acc, K, la, lb, fa, Identity4(), lds);
  } else {
    gemm_nt_tile<C, true>(acc, K, la, lb, fa, Identity4(), lds);
  }

  double nrm = 0.0;
  adj_tile_epilogue<C, MODE>(a, acc, rowtab, lds, m0, n0, R, nrm);
  if (MODE == STEP_RESID && a.norm) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if ((tid & 63) == 0) atomicAdd(a.norm, nrm);
  }
}

// bf16 weights: the fp32 products kappa*w go to LDS as one bf16 tile or as hi + lo tiles
// (the configuration's A2, see gemm_core_bf16.h).
struct KapW8 {
  floatx4 k0, k1, w0, w1;
};

template <class C, int MODE>
__global__ __launch_bounds__(C::NT, C::MINWAVES) void adj_step_kernel_bf16(AdjArgs a) {
  constexpr int LDSF = C::LDS_ELEMS / 2 + 1 > EpiStage<C>::FLOATS ? C::LDS_ELEMS / 2 + 1
                                                                  : EpiStage<C>::FLOATS;
  __shared__ __attribute__((aligned(16))) float ldsf[LDSF];
  bf16_t* lds = reinterpret_cast<bf16_t*>(ldsf);
  const int H = a.H, B = a.B, K = 3 * a.H;
  const long long R = (long long)a.nk * B;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (H + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const int tid = threadIdx.x;
  __shared__ AdjRow rowtab[C::TM];
  if (tid < C::TM) {
    long long r = m0 + tid;
    if (r >= R) r = R - 1;
    rowtab[tid] = adj_row(a, r);
  }
  // (visible to all waves after the barriers inside the contraction)

  const float* krow[C::A_CHUNKS];
  const float* wrow[C::A_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row_b<C>(s);
    if (r >= R) r = R - 1;
    const long long pt = (unsigned)r / (unsigned)B;   // rows < 2^31: 32-bit division
    const int b = (int)(r - pt * B);
    krow[s] = a.kap + (a.k.at(pt) * B + b) * (long long)a.kw;
    wrow[s] = a.w_in + (a.in.at(pt) * B + b) * H;
  }
  typename TileSums<C>::type acc;
  auto la = [&](int s, int k) {
    const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
    return KapW8{ldg4(krow[s] + k), ldg4(krow[s] + k + 4), ldg4(wrow[s] + kk),
                 ldg4(wrow[s] + kk + 4)};
  };
  auto fa = [](const KapW8& r) { return F32x8{r.k0 * r.w0, r.k1 * r.w1}; };
  if constexpr (C::NP == 3) {
    auto urow = [&](int, int c) { return (long long)min(n0 + c, H - 1); };
    // Where gates are whole slices: the sum over k may run in any slice order, so slice i takes gate i % 3
    // and the columns of slice i / 3 of that gate; the three slices that multiply the same columns
    // of w follow each other, and w is loaded for the first of them only (see adj_step_kernel).
    const bool whole = H % C::TK == 0;
    F32x8 wkeep[C::A_CHUNKS];
    auto ordered = [&](int s, int k) {
      if (!whole || __builtin_amdgcn_readfirstlane(k) < H) {
        const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
        wkeep[s] = F32x8{ldg4(wrow[s] + kk), ldg4(wrow[s] + kk + 4)};
      }
      return KapW8{ldg4(krow[s] + k), ldg4(krow[s] + k + 4), wkeep[s].lo4, wkeep[s].hi4};
    };
    contract_terms<C>(
        acc, K, ordered,
        [&](int s) { return row_top<C>(s, K, [&](int k) { return fa(la(s, k)); }); }, fa, a.UT3, H, urow, lds,
        [&](int tr, int k) {
          const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
          return ldg4(a.kap + rowtab[tr].k + k) * ldg4(a.w_in + rowtab[tr].in + kk);
        },
        [&](int g, int c) { return (const float*)a.UT + urow(g, c) * K; },
        [&](int i) { return whole ? i % 3 * H + i / 3 * C::TK : i * C::TK; });
  } else {
    acc.zero();
    const bf16_t* brow[C::B_CHUNKS];
#pragma unroll
    for (int s = 0; s < C::B_CHUNKS; ++s) {
      int j = n0 + chunk_row_b<C>(s);
      if (j >= H) j = H - 1;
      brow[s] = (const bf16_t*)a.UT + (long long)j * K;
    }
    auto lb = [&](int s, int k) { return ldg8h(brow[s] + k); };
    if (K % C::TK == 0)
      gemm_nt_tile_bf16<C, false>(acc, K, la, lb, fa, lds);
    else
      gemm_nt_tile_bf16<C, true>(acc, K, la, lb, fa, lds);
  }

  double nrm = 0.0;
  adj_tile_epilogue<C, MODE>(a, acc, rowtab, ldsf, m0, n0, R, nrm);
  if (MODE == STEP_RESID && a.norm) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if ((tid & 63) == 0) atomicAdd(a.norm, nrm);
  }
}

// ---------------------------------------------------------------------------
// Input gradients: dx[R, D] = S_x[R, 3H] . WT[D, 3H]^T,  S_x = (k_r w, k_z w, k_n w)
// of step t in row (t-1)*B + b  (input-side counterpart of Alg. 3's gradient line)
// ---------------------------------------------------------------------------
typedef TileCfg<2, 2, 2, 2, 1> DxCfg;            // 128 x 128 tile
typedef TileCfgB<2, 2, 2, 2, 1, true> DxCfgB;
typedef TileCfgB<2, 2, 2, 2, 1, true, 1, 1, 2, 1, 64, false> DxCfgF;   // kappa * w as one bf16 term
typedef TileCfgB<4, 2, 1, 2, 1, true, 1, 1, 2, 3, 32> DxCfgS;     // 8 waves of 32 x 64

// Stores one accumulator tile of a plain GEMM: out[m, n], leading dimension N.
template <class C>
__device__ inline void store_tile(const Acc<C>& acc, float* out, long long m0, int n0,
                                  long long M, int N) {
#pragma unroll
  for (int a = 0; a < C::BM; ++a)
#pragma unroll
    for (int b = 0; b < C::BN; ++b) {
      int row, col;
      acc_coord<C>(a, b, 0, row, col);
      const int n = n0 + col;
      if (n >= N) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc_coord<C>(a, b, e, row, col);
        const long long m = m0 + row;
        if (m < M) out[m * N + n] = acc.v[0][a][b][e];
      }
    }
}

__global__ __launch_bounds__(DxCfg::NT) void input_grad_kernel(
    const float* __restrict__ kap0, const float* __restrict__ w, const float* __restrict__ WT,
    float* __restrict__ dx, long long R, int B, int H, int D) {
  typedef DxCfg C;
  __shared__ __attribute__((aligned(16))) float lds[C::LDS_FLOATS];
  const int K = 3 * H;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  // coefficient and adjoint rows are one time point ahead of the dx row
  const float* krow[C::A_CHUNKS];
  const float* wrow[C::A_CHUNKS];
  const float* brow[C::B_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row<C>(s);
    if (r >= R) r = R - 1;     // clamped rows are never stored
    krow[s] = kap0 + (r + B) * (5LL * H);
    wrow[s] = w + (r + B) * H;
  }
#pragma unroll
  for (int s = 0; s < C::B_CHUNKS; ++s) {
    int n = n0 + chunk_row<C>(s);
    if (n >= D) n = D - 1;
    brow[s] = WT + (long long)n * K;
  }
  Acc<C> acc;
  acc.zero();
  auto la = [&](int s, int k) {
    // third gate: k_n is the fifth coefficient block
    const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
    const int ks = k >= 2 * H ? k + 2 * H : k;
    return KapW{ldg4(krow[s] + ks), ldg4(wrow[s] + kk)};
  };
  auto lb = [&](int s, int k) { return ldg4(brow[s] + k); };
  auto fa = [](const KapW& r) { return r.kap * r.w; };
  if (K % C::TK == 0)
    gemm_nt_tile<C, false>(acc, K, la, lb, fa, Identity4(), lds);
  else
    gemm_nt_tile<C, true>(acc, K, la, lb, fa, Identity4(), lds);
  store_tile<C>(acc, dx, m0, n0, R, D);
}

template <class C>
__global__ __launch_bounds__(C::NT, InTerms<C>::value ? C::MINWAVES : 1) void input_grad_kernel_bf16(
    const float* __restrict__ kap0, const float* __restrict__ w, const bf16_t* __restrict__ WT,
    const float* __restrict__ WTf, float* __restrict__ dx, long long R, int B, int H, int D) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[C::LDS_ELEMS];
  const int K = 3 * H;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const float* krow[C::A_CHUNKS];
  const float* wrow[C::A_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row_b<C>(s);
    if (r >= R) r = R - 1;
    krow[s] = kap0 + (r + B) * (5LL * H);
    wrow[s] = w + (r + B) * H;
  }
  typename TileSums<C>::type acc;
  auto la = [&](int s, int k) {
    const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
    const int ks = k >= 2 * H ? k + 2 * H : k;
    return KapW8{ldg4(krow[s] + ks), ldg4(krow[s] + ks + 4), ldg4(wrow[s] + kk),
                 ldg4(wrow[s] + kk + 4)};
  };
  auto fa = [](const KapW8& r) { return F32x8{r.k0 * r.w0, r.k1 * r.w1}; };
  if constexpr (C::NP == 3) {
    auto wrow_of = [&](int, int c) { return (long long)min(n0 + c, D - 1); };
    contract_terms<C>(
        acc, K, la, [&](int s) { return row_top<C>(s, K, [&](int k) { return fa(la(s, k)); }); }, fa,
        WT, D, wrow_of, lds,
        [&](int tr, int k) {
          const long long r = m0 + tr < R ? m0 + tr : R - 1;
          const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
          const int ks = k >= 2 * H ? k + 2 * H : k;
          return ldg4(kap0 + (r + B) * (5LL * H) + ks) * ldg4(w + (r + B) * H + kk);
        },
        [&](int g, int c) { return WTf + wrow_of(g, c) * K; });
  } else {
    acc.zero();
    const bf16_t* brow[C::B_CHUNKS];
#pragma unroll
    for (int s = 0; s < C::B_CHUNKS; ++s) {
      int n = n0 + chunk_row_b<C>(s);
      if (n >= D) n = D - 1;
      brow[s] = WT + (long long)n * K;
    }
    auto lb = [&](int s, int k) { return ldg8h(brow[s] + k); };
    if (K % C::TK == 0)
      gemm_nt_tile_bf16<C, false>(acc, K, la, lb, fa, lds);
    else
      gemm_nt_tile_bf16<C, true>(acc, K, la, lb, fa, lds);
  }
  if constexpr (InTerms<C>::value)
    store_tile_terms<C>(acc, dx, nullptr, m0, n0, R, D);
  else
    store_tile<C>(acc, dx, m0, n0, R, D);
}

hipError_t launch_input_grads(const float* kap0, const float* w, const void* WT, const void* WT3,
                              float* dx, int T, int B, int D, int H, int bf16, int one_term,
                              hipStream_t s) {
  const long long R = (long long)T * B;
  prof_begin(6, s);
  if (bf16 == 2) {
    typedef DxCfgS C;
    dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(input_grad_kernel_bf16<C>, grid, dim3(C::NT), 0, s, kap0, w,
                       (const bf16_t*)WT3, (const float*)WT, dx, R, B, H, D);
  } else if (bf16 && one_term) {
    typedef DxCfgF C;
    dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(input_grad_kernel_bf16<C>, grid, dim3(C::NT), 0, s, kap0, w,
                       (const bf16_t*)WT, (const float*)nullptr, dx, R, B, H, D);
  } else if (bf16) {
    typedef DxCfgB C;
    dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(input_grad_kernel_bf16<C>, grid, dim3(C::NT), 0, s, kap0, w,
                       (const bf16_t*)WT, (const float*)nullptr, dx, R, B, H, D);
  } else {
    typedef DxCfg C;
    dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (D + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(input_grad_kernel, grid, dim3(C::NT), 0, s, kap0, w, (const float*)WT, dx,
                       R, B, H, D);
  }
  prof_end(6, 2.0 * (double)R * 3 * H * D,
           4.0 * (double)R * (4.0 * H + D) + (bf16 == 1 ? 2.0 : 4.0) * 3.0 * H * D, s);
  return hipGetLastError();
}

// Few-row variant (coarsest-level solve, serial BPTT): see skinny.h
template <int CT>
struct AdjSkMaxNT {
  static constexpr int value = CT >= 8 ? 512 : SK_MAXNT;
};

template <int CT, int MODE, class WT>
__global__ __launch_bounds__(AdjSkMaxNT<CT>::value) void adj_skinny_kernel(AdjArgs a,
                                                                           int rows_block) {
  constexpr int VP = sk_pow2_ceil(SK_RR * CT);
  __shared__ float red[(SK_MAXNT / 64) * VP];
  const int H = a.H, K = 3 * a.H;
  const int R = a.nk * a.B;
  const int r0 = blockIdx.y * rows_block;
  const int rows_here = min(rows_block, R - r0);
  const SkGeom geo = sk_geom(rows_block, K);
  const int ksl = geo.ksl;
  const int tid = threadIdx.x;
  const int ks = tid & (ksl - 1), rg = tid / ksl;
  const int j0 = blockIdx.x * CT;

  const int n_out = rows_here * CT;
  const bool epi = tid < n_out && j0 + tid % CT < H;
  int e_j = 0;
  AdjRow ero = {};
  AdjEpiIn ein = {};
  if (epi) {
    ero = adj_row(a, r0 + tid / CT);
    e_j = j0 + tid % CT;
    ein = adj_epi_load<MODE>(a, ero, e_j);
  }

  // rows beyond the block are clamped to its last row (their sums are never used)
  const float* krow[SK_RR];
  const float* wrow[SK_RR];
#pragma unroll
  for (int i = 0; i < SK_RR; ++i) {
    const AdjRow ro = adj_row(a, r0 + min(rg * SK_RR + i, rows_here - 1));
    krow[i] = a.kap + ro.k;
    wrow[i] = a.w_in + ro.in;
  }
  const WT* urow[CT];
#pragma unroll
  for (int u = 0; u < CT; ++u) urow[u] = (const WT*)a.UT + (long long)min(j0 + u, H - 1) * K;
  float acc[SK_RR][CT];
  skinny_dot<CT, WT>(acc, K, ks, ksl, urow, [&](int i, int k) {
    const int kk = k >= 2 * H ? k - 2 * H : (k >= H ? k - H : k);
    return ldg4(krow[i] + k) * ldg4(wrow[i] + kk);
  });
  float v[VP];
#pragma unroll
  for (int q = 0; q < VP; ++q) v[q] = q < SK_RR * CT ? acc[q / CT][q % CT] : 0.f;
  skinny_reduce<VP>(v, red, rg, ks, ksl);
  __syncthreads();

  double nrm = 0.0;
  for (int e = tid; e < n_out; e += geo.nt) {
    const int row = e / CT, c = e % CT;
    const int j = j0 + c;
    if (j >= H) continue;
    const float dot = skinny_sum<VP>(red, row / SK_RR, (row % SK_RR) * CT + c, ksl);
    if (e == tid && epi) {
      adj_epi_finish<MODE>(a, ero, e_j, dot, ein, nrm);
    } else {   // more outputs than threads (tiny K only)
      const AdjRow ro = adj_row(a, r0 + row);
      adj_epi_finish<MODE>(a, ro, j, dot, adj_epi_load<MODE>(a, ro, j), nrm);
    }
  }
  if (MODE == STEP_RESID && a.norm && nrm != 0.0) atomicAdd(a.norm, nrm);
}

typedef TileCfg<2, 2, 2, 2, 1> AdjBig;    // 128 x 128, 256 threads
typedef TileCfg<2, 2, 1, 1, 1> AdjMid;    //  64 x 64, 256 threads
typedef TileCfg<1, 1, 1, 1, 1, 128, 1, 4> AdjSmall;  //  32 x 32, 4 waves splitting K
// fp32 operands in terms (K-slices of 32)
typedef TileCfgB<2, 2, 2, 2, 1, true, 1, 1, 2, 3, 32> AdjBigS;
// the same tile with 8 waves of 64 x 32 each
typedef TileCfgB<4, 2, 1, 2, 1, true, 1, 1, 2, 3, 32> AdjBigS8;
// 128 x 256 as eight waves of 128 x 32, one workgroup per CU: see launch_adj_step
typedef TileCfgB<2, 4, 2, 2, 1, true, 1, 1, 1, 3, 32> AdjHugeS;
// 64 x 128 as eight waves, two groups splitting K, one workgroup per CU
typedef TileCfgB<2, 2, 1, 2, 1, true, 2, 1, 1, 3, 32> AdjWideKS;
// mid-size launches: 64 x 128 as four waves of 32 x 64, and 64 x 64 with two groups of four waves
// splitting K (the adjoint's K is 3H: with one group the 64 x 64 tile waits on its slices)
typedef TileCfgB<2, 2, 1, 2, 1, true, 1, 1, 2, 3, 32> AdjWideS;
typedef TileCfgB<2, 2, 1, 1, 1, true, 2, 1, 2, 3, 32> AdjMidS;

template <class C>
static void launch_adj_f32(const AdjArgs& a, hipStream_t s) {
  const long long R = (long long)a.nk * a.B;
  dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (a.H + C::TN - 1) / C::TN));
  if (a.mode == STEP_RELAX)
    hipLaunchKernelGGL((adj_step_kernel<C, STEP_RELAX>), grid, dim3(C::NT), 0, s, a);
  else
    hipLaunchKernelGGL((adj_step_kernel<C, STEP_RESID>), grid, dim3(C::NT), 0, s, a);
}

template <class C>
static void launch_adj_terms(const AdjArgs& a, hipStream_t s) {
  const long long R = (long long)a.nk * a.B;
  dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (a.H + C::TN - 1) / C::TN));
  if (a.mode == STEP_RELAX)
    hipLaunchKernelGGL((adj_step_kernel_bf16<C, STEP_RELAX>), grid, dim3(C::NT), 0, s, a);
  else
    hipLaunchKernelGGL((adj_step_kernel_bf16<C, STEP_RESID>), grid, dim3(C::NT), 0, s, a);
}

// bf16 weights, kappa * w as one bf16 term (A2: two).  Every column tile forms the products again (8 bytes
// of coefficients and state per element against 2 of a weight), so tiles are as wide as they can be with
// a workgroup for each CU; where even small tiles leave CUs idle, groups of waves split K.  The tile with
// the smallest number of rounds over the 256 CUs of a whole GPU times its time for one: us of a launch of
// exactly one round at K = 3072, one term.  Only their ratios count; those of two terms and of other K were not
// measured, the rule as a whole was (K = 600 to 3072), us with 128 x 128, 64 x 64 and 32 x 32 tiles only :
// these, one term: 512 rows x 1024 31.3 : 23.7, 1024 x 1024 48 : 35.5, 2048 x 1024 61 : 52, 4096 x
// 1024 90 : 71, 8192 x 1024 174 : 115, 2048 x 512 25.9 : 19.3, 16384 x 512 103 : 74, 4096 x 256 15.6 : 12.7, 1500 x
// 200 10.8 : 9.3, 32768 x 296 114 : 99; two terms: 512 x 1024 32 : 27, 2048 x 1024 63 : 57, 8192 x 1024 198 : 144,
// 16384 x 512 112 : 85, 1500 x 200 11.9 : 10.1.
template <bool A2>
static void launch_adj_half(const AdjArgs& a, hipStream_t s) {
  const long long R = (long long)a.nk * a.B;
  static const struct {
    int tm, tn, us;
  } tile[] = {{32, 32, 22}, {32, 64, 25}, {32, 128, 34}, {64, 64, 38}, {64, 128, 51}, {64, 256, 72},
              {128, 128, 90}, {128, 256, 115}};
  int best = 0;
  long long cost = 0;
  for (int i = 0; i < 8; ++i) {
    const long long n = ((R + tile[i].tm - 1) / tile[i].tm) * ((a.H + tile[i].tn - 1) / tile[i].tn);
    const long long c = (n + 255) / 256 * tile[i].us;
    if (i == 0 || c < cost) {
      best = i;
      cost = c;
    }
  }
  switch (best) {
    case 0: return launch_adj_terms<TileCfgB<1, 1, 1, 1, 1, true, 4, 1, 2, 1, 64, A2>>(a, s);
    case 1: return launch_adj_terms<TileCfgB<1, 2, 1, 1, 1, true, 4, 1, 2, 1, 64, A2>>(a, s);
    case 2: return launch_adj_terms<TileCfgB<1, 4, 1, 1, 1, true, 2, 1, 2, 1, 64, A2>>(a, s);
    case 3:   // (up to three K-slices of 64: nothing to split; 25600 rows x 64, two terms, 15.0 split : 12.3)
      if (a.H <= 64) return launch_adj_terms<TileCfgB<2, 2, 1, 1, 1, true, 1, 1, 2, 1, 64, A2>>(a, s);
      return launch_adj_terms<TileCfgB<2, 2, 1, 1, 1, true, 2, 1, 2, 1, 64, A2>>(a, s);
    case 4: return launch_adj_terms<TileCfgB<2, 2, 1, 2, 1, true, 2, 1, 2, 1, 64, A2>>(a, s);
    case 5: return launch_adj_terms<TileCfgB<2, 4, 1, 2, 1, true, 1, 1, 2, 1, 128, A2>>(a, s);
    case 6: return launch_adj_terms<TileCfgB<4, 2, 1, 2, 1, true, 1, 1, 2, 1, 64, A2>>(a, s);
    default: return launch_adj_terms<TileCfgB<2, 4, 2, 2, 1, true, 1, 1, 2, 1, 64, A2>>(a, s);
  }
}

// Rows per workgroup of the few-row adjoint step: every workgroup streams the
// coefficient and adjoint rows of its row block (24H bytes per row), so the block is
// kept small and the workgroup takes more columns instead.
constexpr int ADJ_SK_ROWS = 8;

static int adj_sk_rows(long long R) { return R < ADJ_SK_ROWS ? (int)R : ADJ_SK_ROWS; }

template <int CT, int MODE>
static void launch_adj_skinny_mode(const AdjArgs& a, dim3 grid, hipStream_t s) {
  const int rb = adj_sk_rows((long long)a.nk * a.B);
  const dim3 block(sk_geom(rb, 3 * a.H).nt);
  if (a.bf16 == 1)
    hipLaunchKernelGGL((adj_skinny_kernel<CT, MODE, bf16_t>), grid, block, 0, s, a, rb);
  else
    hipLaunchKernelGGL((adj_skinny_kernel<CT, MODE, float>), grid, block, 0, s, a, rb);
}

template <int CT>
static void launch_adj_skinny(const AdjArgs& a, dim3 grid, hipStream_t s) {
  if (a.mode == STEP_RELAX)
    launch_adj_skinny_mode<CT, STEP_RELAX>(a, grid, s);
  else
    launch_adj_skinny_mode<CT, STEP_RESID>(a, grid, s);
}

// modes STEP_RELAX and STEP_RESID (the adjoint cycle solves its coarse equations for the
// error and needs no right-hand-side launch)
hipError_t launch_adj_step(const AdjArgs& a, hipStream_t s) {
  if (a.nk <= 0) return hipSuccess;
  if (a.mode != STEP_RELAX && a.mode != STEP_RESID) return hipErrorInvalidValue;
  const long long R = (long long)a.nk * a.B;
  auto tiles = [&](int tm, int tn) { return ((R + tm - 1) / tm) * ((a.H + tn - 1) / tn); };
  const int kind = R <= 2 * SK_MAXROWS ? 5 : 1;
  prof_begin(kind, s, R, a.mode);
  if (R <= 2 * SK_MAXROWS) {
    // up to four columns per workgroup (eight measured 1.8 us slower per step at 32 rows x 512)
    const int rb = adj_sk_rows(R);
    const int nrb = (int)((R + rb - 1) / rb);
    const long long hw = (long long)a.H * nrb;
    const int ct = hw >= 1024 ? 4 : (hw >= 512 ? 2 : 1);
    dim3 grid((unsigned)((a.H + ct - 1) / ct), (unsigned)nrb);
    if (ct == 4)
      launch_adj_skinny<4>(a, grid, s);
    else if (ct == 2)
      launch_adj_skinny<2>(a, grid, s);
    else
      launch_adj_skinny<1>(a, grid, s);
  } else if (a.bf16 == 1) {
    if (a.one_term) launch_adj_half<false>(a, s);
    else launch_adj_half<true>(a, s);
  }
  // terms, large launches: the products kappa * w are formed, scaled and split once per column tile, so
  // the widest tile that fills the CUs, one workgroup each (us at 16384 rows x 512, x 1024: 128 x 128
  // 92, 322; 64 x 256 88, 296; 128 x 256 86, 291).  Two column tiles from 384 on: below that it would be
  // mostly padding
  else if (a.bf16 == 2 && a.H >= 384 && tiles(AdjHugeS::TM, AdjHugeS::TN) >= 192) {
    launch_adj_terms<AdjHugeS>(a, s);
  } else if (tiles(AdjBig::TM, AdjBig::TN) >= 384) {
    if (a.bf16 == 2 && a.mode == STEP_RELAX)
      launch_adj_terms<AdjBigS8>(a, s);
    else if (a.bf16 == 2)
      launch_adj_terms<AdjBigS>(a, s);
    else
      launch_adj_f32<AdjBig>(a, s);
  }
  // terms, by what fills the chip (us, 64 x 128 : the same with K split : 64 x 64 with K split):
  // 4096 rows x 1024 (512 wide tiles) 101 : 103 : 137, 3200 x 1000 (400) 113 : 108 : 153, 2048 x 512 (128;
  // 256 of 64 x 64) 34 : 24 : 23, 1024 x 1024 (128; 256) 62 : 41 : 40.  The lines of 384 and 192 tiles
  // were drawn on three bf16 terms, where such steps took twice as long; below them fp32 tiles are the
  // slower ones now (1024 x 520, 144 tiles of 64 x 64: 22, with the 32 x 32 fp32 tiles it takes 42)
  else if (a.bf16 == 2 && tiles(AdjWideS::TM, AdjWideS::TN) >= 384)
    launch_adj_terms<AdjWideS>(a, s);
  // one round of 64 x 128 tiles, one per CU: eight waves splitting K (4096 rows x 512, 256 tiles: 43 us with
  // two 64 x 64 tiles per CU, which form and split every product twice as often, 30 this way)
  else if (a.bf16 == 2 && tiles(AdjWideS::TM, AdjWideS::TN) >= 192 &&
           tiles(AdjWideS::TM, AdjWideS::TN) <= 256)
    launch_adj_terms<AdjWideKS>(a, s);
  else if (a.bf16 == 2 && R > 32 && tiles(AdjMidS::TM, AdjMidS::TN) >= 192)
    launch_adj_terms<AdjMidS>(a, s);
  else if (R > 32 && tiles(AdjMid::TM, AdjMid::TN) >= 256)
    launch_adj_f32<AdjMid>(a, s);
  else   // (operands in terms included: 32 x 32 tiles are faster in fp32, see launch_phi_cfg, and no less
         // accurate, see gemm_nt_tile)
    launch_adj_f32<AdjSmall>(a, s);
  prof_end(kind, 6.0 * (double)R * a.H * a.H, 28.0 * (double)R * a.H, s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// UT[cols, rows] = U[rows, cols]^T
// ---------------------------------------------------------------------------
template <class T>
__global__ void transpose_kernel(const T* __restrict__ U, T* __restrict__ UT, int rows, int cols) {
  __shared__ T t[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
  for (int i = ty; i < 32; i += 8) {
    int r = r0 + i, c = c0 + tx;
    t[i][tx] = (r < rows && c < cols) ? U[(long long)r * cols + c] : T(0);
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    int c = c0 + i, r = r0 + tx;
    if (r < rows && c < cols) UT[(long long)c * rows + r] = t[tx][i];
  }
}

hipError_t launch_transpose(const void* U, void* UT, int rows, int cols, int bf16, hipStream_t s) {
  dim3 grid((cols + 31) / 32, (rows + 31) / 32);
  if (bf16)
    hipLaunchKernelGGL(transpose_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)U,
                       (bf16_t*)UT, rows, cols);
  else
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, s, (const float*)U,
                       (float*)UT, rows, cols);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Parameter gradients: dU = S^T Hprev, dW = Sx^T X, db_h = colsum S, db_i = colsum Sx
// with S[k, g*H+j] = kap0[k][g*H+j] * w[k][j] (gates r, z, q) and Sx the same
// except that its third block uses k_n (stored at 4H..5H) instead of k_q.
// Row k = (t-1)*B + b for step t = 1..T: kap0 and w rows are offset by one time
// point, Hprev = h[t-1] and X = x[t-1] are not.
// ---------------------------------------------------------------------------
constexpr int GTK = 32;            // K-slice (rows of the sum) per iteration
constexpr int GT = 128;            // output tile is GT x GT
constexpr int GLD = GT;            // LDS row stride in floats; odd rows swap their 32-column
                                   // halves pairwise (column ^ 32), which keeps the two
                                   // half-waves of an operand read on different banks

struct GradArgs {
  const float* kap0;   // [(T+1),B,5H]
  const float* w;      // [(T+1),B,H]
  const void* Bm;      // h[(T+1),B,H] (float) or x[T,B,D] (float or bf16); row k as is
  float* part;         // [splits][3H][N]
  float* bpart;        // [splits][3H] column sums of S (bias gradients), written by the first column tile
  long long Ktot;      // T*B
  long long Kper;      // rows per split (multiple of GTK)
  int B, H, N;         // N = H (dU) or D (dW)
  int third_off;       // 2H (k_q, dU) or 4H (k_n, dW)
  int mtiles, ntiles;  // output tiles along 3H and N
  int splits;          // row splits
};

// Both gradients in one launch of the fp32 kernel: workgroups from `first` on belong to dW.
struct GradPair {
  GradArgs g[2];
  unsigned first;
  float *db_i, *db_h;  // one split: the sums are the gradients (g[].part = dU, dW), biases go here; else null
};

// acc += sum over the rows k in [kbeg, kend) of S[k, m] Bm[k, n], m = m0.., n = n0..; colsum: this
// thread's share of the column sums of S.  Both operands are read with the contracted index k
// slowest, so an LDS slice is stored [k][m] and a lane reads its MFMA operand as one float per
// k-pair.  As, Bs: GTK * GLD floats each.
template <class BT, bool SKIP>
__device__ inline void grad_contract_f32(const GradArgs& a, int m0, int n0, long long kbeg,
                                         long long kend, float* As, float* Bs,
                                         floatx16 (&acc)[2][2], floatx4& colsum) {
  const int H = a.H, N = a.N, M = 3 * a.H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;
  const long long rowoff = a.B;   // kap0 / w rows are one time point ahead
  // each thread stages NCH float4 of A and of B per slice: slice row = q/32, col4 = q%32.
  // The column part is fixed per thread; out-of-range columns and rows are clamped
  // for the load and zeroed when the slice is written to LDS.
  constexpr int NCH = GTK * (GT / 4) / 256;
  const int c4 = tid & 31;
  const int m = m0 + c4 * 4, n = n0 + c4 * 4;
  const bool m_ok = m < M, n_ok = n < N;
  const int mc = m_ok ? m : 0, nc = n_ok ? n : 0;
  const int gate = mc / H, jcol = mc - gate * H;
  const int src = gate == 2 ? a.third_off + jcol : mc;
  floatx4 rk[NCH], rw[NCH], rb[NCH];
  auto fetch = [&](long long k0) {
#pragma unroll
    for (int s = 0; s < NCH; ++s) {
      long long k = k0 + (tid >> 5) + s * 8;
      if (k >= kend) k = kend - 1;
      rk[s] = ldg4(a.kap0 + (k + rowoff) * (5LL * H) + src);
      rw[s] = ldg4(a.w + (k + rowoff) * H + jcol);
      rb[s] = ldg4w((const BT*)a.Bm + k * N + nc);
    }
  };
  const int wcol = (c4 * 4) ^ (((tid >> 5) & 1) << 5);     // slice rows kr and tid >> 5: same parity
  auto stash = [&](long long k0) {
#pragma unroll
    for (int s = 0; s < NCH; ++s) {
      const int kr = (tid >> 5) + s * 8;
      const bool k_ok = k0 + kr < kend;
      const floatx4 p = (k_ok && m_ok) ? rk[s] * rw[s] : zero4();
      colsum += p;
      *reinterpret_cast<floatx4*>(&As[kr * GLD + wcol]) = p;
      *reinterpret_cast<floatx4*>(&Bs[kr * GLD + wcol]) = (k_ok && n_ok) ? rb[s] : zero4();
    }
  };
  auto frags = [&](int p, float (&av)[2], float (&bv)[2]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      av[i] = As[(2 * p + lh) * GLD + wm * 64 + ((i ^ lh) << 5) + li];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      bv[j] = Bs[(2 * p + lh) * GLD + wn * 64 + ((j ^ lh) << 5) + li];
  };

  // SKIP: 32 x 32 blocks of this wave that hold no outputs are left out (a layer of 32 columns fills one
  // of two)
  const int mi = M - m0 - wm * 64, nj = N - n0 - wn * 64;
  const bool full = !SKIP || (mi > 32 && nj > 32);
  if (kbeg < kend) {
    fetch(kbeg);
    stash(kbeg);
    __syncthreads();
    for (long long k0 = kbeg; k0 < kend; k0 += GTK) {
      const bool more = k0 + GTK < kend;
      if (more) fetch(k0 + GTK);
      __builtin_amdgcn_sched_barrier(0);
      float av[2][2], bv[2][2];
      __builtin_amdgcn_s_setprio(2);      // MFMA phase first at issue (see gemm_core.h)
      if (full) {
        frags(0, av[0], bv[0]);
#pragma unroll
        for (int p = 0; p < GTK / 2; ++p) {
          if (p + 1 < GTK / 2) frags(p + 1, av[(p + 1) & 1], bv[(p + 1) & 1]);
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[p & 1][i], bv[p & 1][j],
                                                               acc[i][j], 0, 0, 0);
          if (p + 1 < GTK / 2) {
            // one LDS read of the next k-pair, one MFMA of this pair, four times
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else if (mi > 0 && nj > 0) {
#pragma unroll 4
        for (int p = 0; p < GTK / 2; ++p) {
          frags(p, av[0], bv[0]);
          acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[0][0], bv[0][0], acc[0][0], 0, 0, 0);
          if (mi > 32)
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[0][1], bv[0][0], acc[1][0], 0, 0, 0);
          if (nj > 32)
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[0][0], bv[0][1], acc[0][1], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      if (more) {
        stash(k0 + GTK);
        __syncthreads();
      }
    }
  }
}

// C[m, n] = sum_k S[k, m] Bm[k, n] over this split's rows k.
// 1-D grid: workgroups go round-robin over the 8 XCDs, so split z is given to XCD
// z % 8 and all output tiles of a split run on that XCD: its rows of S and Bm are
// fetched into one L2 only.
// SKIP: for small problems, see grad_contract_f32 (its branches spill four registers).
template <class BT, bool SKIP>
__global__ __launch_bounds__(256, 3) void grad_gemm_kernel(GradPair pair) {
  __shared__ __attribute__((aligned(16))) float As[GTK * GLD];
  __shared__ __attribute__((aligned(16))) float Bs[GTK * GLD];
  const int which = blockIdx.x >= pair.first ? 1 : 0;
  const GradArgs& a = pair.g[which];
  const int bid = (int)(blockIdx.x - (which ? pair.first : 0));
  const int N = a.N, M = 3 * a.H;
  const int tiles = a.mtiles * a.ntiles;
  if (bid >= tiles * a.splits) return;      // (`first` is a multiple of the XCDs)
  int tile, z;
  if (a.splits % NXCD == 0) {
    const int j = bid / NXCD;
    tile = j % tiles;
    z = (j / tiles) * NXCD + bid % NXCD;
  } else {
    tile = bid % tiles;
    z = bid / tiles;
  }
  const int m0 = (tile % a.mtiles) * GT, n0 = (tile / a.mtiles) * GT;
  const long long kbeg = (long long)z * a.Kper;
  long long kend = kbeg + a.Kper;
  if (kend > a.Ktot) kend = a.Ktot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;
  const int c4 = tid & 31;

  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // Bias gradients are the column sums of S: every thread adds up the products it stages
  // (its four columns, its rows of every slice); the eight row groups meet in LDS at the end.
  floatx4 colsum = zero4();
  grad_contract_f32<BT, SKIP>(a, m0, n0, kbeg, kend, As, Bs, acc, colsum);
  const int nt = tile / a.mtiles;
  {
    float* red = As;                    // [8][GT] floats (the slices are no longer read)
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) red[(tid >> 5) * GT + c4 * 4 + e] = colsum[e];
    __syncthreads();
    if (tid < GT && m0 + tid < M) {
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) sum += red[q * GT + tid];
      // every column tile holds the same sums: the first one reports them
      if (nt == 0) {
        const int c = m0 + tid, H = a.H;
        if (!pair.db_h) {
          a.bpart[(long long)z * M + c] = sum;
        } else {                          // as in bias_reduce
          if (which == 0) pair.db_h[c] = sum;
          if ((which == 0) == (c < 2 * H)) pair.db_i[c] = sum;
        }
      }
    }
  }
  float* out = a.part + (long long)z * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int mm = m0 + wm * 64 + i * 32 + 8 * (e / 4) + 4 * lh + (e & 3);
        const int nn = n0 + wn * 64 + j * 32 + li;
        if (mm < M && nn < N) out[(long long)mm * N + nn] = acc[i][j][e];
      }
}

// The same contraction for the bf16-input variant on the bf16 MFMA
// (v_mfma_f32_32x32x16_bf16).  The instruction wants eight consecutive k per lane,
// the operands have k as the slow index, so the transposition happens in registers on
// the way to LDS: a thread loads an 8 (k) x 4 (m) block of kappa and w, forms the
// products and writes, for each of its four m, the eight k as one 16-byte row segment
// of a [m][k] tile - after which fragments are read exactly as in the NT kernels.
// fp32 operands (S = kappa*w, and h for dU) go to LDS as hi + lo bf16 tiles:
//   dW: S_hi x + S_lo x (x is bf16 already);  dU: S_hi h_hi + S_lo h_hi + S_hi h_lo.
// Bias gradients: column sums of the fp32 products, accumulated by the staging threads.
constexpr int HB_TK = 64;                 // k rows per slice
constexpr int HB_LD = HB_TK + 8;          // LDS row stride in bf16 elements
template <bool B_BF16>
__global__ __launch_bounds__(256, 2) void grad_gemm_bf16_kernel(GradArgs a) {
  constexpr int NBT = B_BF16 ? 1 : 2;     // B tiles in LDS (hi, lo)
  __shared__ __attribute__((aligned(16))) bf16_t As[2][GT * HB_LD];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[NBT][GT * HB_LD];
  const int H = a.H, N = a.N, M = 3 * a.H;
  const int tiles = a.mtiles * a.ntiles;
  int tile, z;
  if (a.splits % NXCD == 0) {
    const int j = blockIdx.x / NXCD;
    tile = j % tiles;
    z = (j / tiles) * NXCD + blockIdx.x % NXCD;
  } else {
    tile = blockIdx.x % tiles;
    z = blockIdx.x / tiles;
  }
  const int nt = tile / a.mtiles;
  const int m0 = (tile % a.mtiles) * GT, n0 = nt * GT;
  const long long kbeg = (long long)z * a.Kper;
  long long kend = kbeg + a.Kper;
  if (kend > a.Ktot) kend = a.Ktot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;
  const long long rowoff = a.B;           // kap0 / w rows are one time point ahead

  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // staging block of this thread: A: columns m4*4..+3, rows k8*8..+7 of the slice
  const int m4 = tid & 31, k8 = tid >> 5;
  const int m = m0 + m4 * 4;
  const bool m_ok = m < M;
  const int mc = m_ok ? m : 0;
  const int gate = mc / H, jcol = mc - gate * H;
  const int src = gate == 2 ? a.third_off + jcol : mc;
  // B (bf16): columns n8*8..+7, rows kb*8..+7, threads 0..127;  B (fp32): as A
  const int n8 = tid & 15, kb = B_BF16 ? (tid >> 4) : k8;
  const bool b_thread = !B_BF16 || tid < 128;
  const int n = n0 + (B_BF16 ? n8 * 8 : m4 * 4);
  const bool n_ok = n < N;
  const int nc = n_ok ? n : 0;

  // LDS chunk positions.  A thread's rows are four (fp32 operands) or eight (bf16 second
  // operand) apart, 64 or 128 bytes modulo the 256 the banks span, so the 16-byte chunk it
  // writes is exchanged with another chunk of the row, chosen by the column block (bits 4-5,
  // or 4-6, of the row; the readers apply the same exchange): sixteen neighbouring lanes
  // then cover all banks once.
  const int ka = (k8 ^ ((m4 >> 2) & 3)) * 8;              // k8 == kb for fp32 operands
  const int kbs = (kb ^ ((n8 >> 1) & 7)) * 8;
  floatx4 rk[8], rw[8];
  floatx4 rbf[B_BF16 ? 1 : 8];
  bf16x8 rbh[B_BF16 ? 8 : 1];
  float colsum[4] = {0.f, 0.f, 0.f, 0.f};
  auto fetch = [&](long long k0) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      long long k = k0 + k8 * 8 + r;
      if (k >= kend) k = kend - 1;
      rk[r] = ldg4(a.kap0 + (k + rowoff) * (5LL * H) + src);
      rw[r] = ldg4(a.w + (k + rowoff) * H + jcol);
    }
    if (b_thread) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        long long k = k0 + kb * 8 + r;
        if (k >= kend) k = kend - 1;
        if constexpr (B_BF16)
          rbh[r] = ldg8h((const bf16_t*)a.Bm + k * N + nc);
        else
          rbf[r] = ldg4((const float*)a.Bm + k * N + nc);
      }
    }
  };
  auto stash = [&](long long k0) {
    floatx4 p[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const bool k_ok = k0 + k8 * 8 + r < kend;
      p[r] = (k_ok && m_ok) ? rk[r] * rw[r] : zero4();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      F32x8 v;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v.lo4[r] = p[r][e];
        v.hi4[r] = p[4 + r][e];
        colsum[e] += p[r][e] + p[4 + r][e];
      }
      bf16x8 hi, lo;
      split_bf16(v, hi, lo);
      *reinterpret_cast<bf16x8*>(&As[0][(m4 * 4 + e) * HB_LD + ka]) = hi;
      *reinterpret_cast<bf16x8*>(&As[1][(m4 * 4 + e) * HB_LD + ka]) = lo;
    }
    if (b_thread) {
      if constexpr (B_BF16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          bf16x8 o;
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const bool k_ok = k0 + kb * 8 + r < kend;
            o[r] = (k_ok && n_ok) ? rbh[r][e] : (__bf16)0.f;
          }
          *reinterpret_cast<bf16x8*>(&Bs[0][(n8 * 8 + e) * HB_LD + kbs]) = o;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          F32x8 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v.lo4[r] = (k0 + kb * 8 + r < kend && n_ok) ? rbf[r][e] : 0.f;
            v.hi4[r] = (k0 + kb * 8 + 4 + r < kend && n_ok) ? rbf[4 + r][e] : 0.f;
          }
          bf16x8 hi, lo;
          split_bf16(v, hi, lo);
          *reinterpret_cast<bf16x8*>(&Bs[0][(m4 * 4 + e) * HB_LD + ka]) = hi;
          *reinterpret_cast<bf16x8*>(&Bs[NBT - 1][(m4 * 4 + e) * HB_LD + ka]) = lo;
        }
      }
    }
  };

  if (kbeg < kend) {
    fetch(kbeg);
    stash(kbeg);
    __syncthreads();
    for (long long k0 = kbeg; k0 < kend; k0 += HB_TK) {
      const bool more = k0 + HB_TK < kend;
      if (more) fetch(k0 + HB_TK);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < HB_TK / 16; ++c) {
        bf16x8 fa[2][2], fb[NBT][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            fa[t][i] = *reinterpret_cast<const bf16x8*>(
                &As[t][(wm * 64 + i * 32 + li) * HB_LD + ((2 * c + lh) ^ ((2 * i + (li >> 4)) & 3)) * 8]);
#pragma unroll
        for (int t = 0; t < NBT; ++t)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int sw = B_BF16 ? (4 * wn + 2 * j + (li >> 4)) & 7 : (2 * j + (li >> 4)) & 3;
            fb[t][j] = *reinterpret_cast<const bf16x8*>(
                &Bs[t][(wn * 64 + j * 32 + li) * HB_LD + ((2 * c + lh) ^ sw) * 8]);
          }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[0][j], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[1][i], fb[0][j], acc[i][j], 0, 0, 0);
            if constexpr (!B_BF16)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[NBT - 1][j], acc[i][j], 0, 0, 0);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
      if (more) {
        stash(k0 + HB_TK);
        __syncthreads();
      }
    }
  }
  // column sums: the eight row groups of a column meet in LDS (the A tiles are free now)
  float* red = reinterpret_cast<float*>(&As[0][0]);      // [8][GT] floats = 4 KB
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) red[k8 * GT + m4 * 4 + e] = colsum[e];
  __syncthreads();
  if (tid < GT && m0 + tid < M) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) sum += red[q * GT + tid];
    // every column tile holds the same sums: the first one reports them
    if (nt == 0) a.bpart[(long long)z * M + m0 + tid] = sum;
  }
  float* out = a.part + (long long)z * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int mm = m0 + wm * 64 + i * 32 + 8 * (e / 4) + 4 * lh + (e & 3);
        const int nn = n0 + wn * 64 + j * 32 + li;
        if (mm < M && nn < N) out[(long long)mm * N + nn] = acc[i][j][e];
      }
}

// Wide-tile form of the bf16 contraction above (128 x 256 outputs per workgroup, each wave 64 x 128),
// used when the second operand has more than 128 columns.  The kernel above is bound by the bytes
// it pulls through the vector-memory path (8 bytes of kappa and w per S element, re-read by every
// column tile); twice the columns per tile take 40 % off those.  Both operands are written to LDS
// in the order they have in memory, [k][column] (S after the product and the hi/lo split, eight
// bytes per thread and row; the second operand as loaded), and the k-major MFMA fragments are
// formed by the LDS transpose read (ds_read_b64_tr_b16): within 16 lanes, lane i receives element
// i % 4 of what lanes 4e + i / 4 (e = 0..3) point at.  With lanes 4r..4r+3 of a block pointing at
// sixteen consecutive columns of row k + r, lane i therefore gets column i of rows k..k+3; two
// reads give the eight k of a 32x32x16 operand.  Row strides are 64 bytes modulo 256, so the four
// rows of a read fall on different banks; the writes are contiguous.
constexpr int TR_TK = 32;                  // k rows per slice
constexpr int TR_GN = 256;                 // tile columns (second operand)
constexpr int TR_LDA = GT + 32;            // row strides in elements: 320 and 576 bytes
constexpr int TR_LDB = TR_GN + 32;
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// eight k (rows p .. p + 7 of the LDS tile, in the lane's own order) of this lane's column
__device__ inline bf16x8 lds_tr8(const bf16_t* p, int ld) {
  typedef __attribute__((address_space(3))) short4v* lptr;
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)p);
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr)(p + 4 * ld));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ inline void split_bf16_4(const floatx4& v, bf16x4& hi, bf16x4& lo) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    hi[i] = (__bf16)v[i];
    lo[i] = (__bf16)(v[i] - (float)hi[i]);
  }
}

// ONE: S and an fp32 second operand enter as one bf16 term each (dtype MGRIT_BF16); otherwise as
// hi + lo, with the products S_hi B_hi + S_lo B_hi (+ S_hi B_lo for an fp32 second operand).
template <bool B_BF16, bool ONE>
__global__ __launch_bounds__(256, 2) void grad_gemm_tr_kernel(GradArgs a) {
  constexpr int NBT = (B_BF16 || ONE) ? 1 : 2;     // tiles of the second operand in LDS (hi, lo)
  constexpr int NAT = ONE ? 1 : 2;                 // tiles of S
  __shared__ __attribute__((aligned(16))) bf16_t As[NAT][TR_TK * TR_LDA];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[NBT][TR_TK * TR_LDB];
  const int H = a.H, N = a.N, M = 3 * a.H;
  const int tiles = a.mtiles * a.ntiles;
  int tile, z;
  if (a.splits % NXCD == 0) {
    const int j = blockIdx.x / NXCD;
    tile = j % tiles;
    z = (j / tiles) * NXCD + blockIdx.x % NXCD;
  } else {
    tile = blockIdx.x % tiles;
    z = blockIdx.x / tiles;
  }
  const int nt = tile / a.mtiles;
  const int m0 = (tile % a.mtiles) * GT, n0 = nt * TR_GN;
  const long long kbeg = (long long)z * a.Kper;
  long long kend = kbeg + a.Kper;
  if (kend > a.Ktot) kend = a.Ktot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;
  const long long rowoff = a.B;           // kap0 / w rows are one time point ahead

  floatx16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // staging of S: columns m4*4..+3, slice rows k8 + 8r (r = 0..3)
  const int m4 = tid & 31, k8 = tid >> 5;
  const int m = m0 + m4 * 4;
  const bool m_ok = m < M;
  const int mc = m_ok ? m : 0;
  const int gate = mc / H, jcol = mc - gate * H;
  const int src = gate == 2 ? a.third_off + jcol : mc;
  // second operand: bf16: columns m4*8..+7, rows k8 + 8r (r = 0..3);
  //                 fp32: columns c4*4..+3, rows kf + 4r (r = 0..7)
  const int c4 = tid & 63, kf = tid >> 6;
  const int n = n0 + (B_BF16 ? m4 * 8 : c4 * 4);
  const bool n_ok = n < N;
  const int nc = n_ok ? n : 0;
  floatx4 rk[4], rw[4];
  floatx4 rbf[B_BF16 ? 1 : 8];
  bf16x8 rbh[B_BF16 ? 4 : 1];
  floatx4 colsum = zero4();
  auto fetch = [&](long long k0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      long long k = k0 + k8 + 8 * r;
      if (k >= kend) k = kend - 1;
      rk[r] = ldg4(a.kap0 + (k + rowoff) * (5LL * H) + src);
      rw[r] = ldg4(a.w + (k + rowoff) * H + jcol);
      if constexpr (B_BF16) rbh[r] = ldg8h((const bf16_t*)a.Bm + k * N + nc);
    }
    if constexpr (!B_BF16) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        long long k = k0 + kf + 4 * r;
        if (k >= kend) k = kend - 1;
        rbf[r] = ldg4((const float*)a.Bm + k * N + nc);
      }
    }
  };
  auto stash = [&](long long k0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = k8 + 8 * r;
      const bool k_ok = k0 + row < kend;
      const floatx4 p = (k_ok && m_ok) ? rk[r] * rw[r] : zero4();
      colsum += p;
      bf16x4 hi, lo;
      split_bf16_4(p, hi, lo);
      *reinterpret_cast<bf16x4*>(&As[0][row * TR_LDA + m4 * 4]) = hi;
      if constexpr (!ONE) *reinterpret_cast<bf16x4*>(&As[NAT - 1][row * TR_LDA + m4 * 4]) = lo;
      if constexpr (B_BF16) {
        bf16x8 zv;
#pragma unroll
        for (int i = 0; i < 8; ++i) zv[i] = (__bf16)0.f;
        *reinterpret_cast<bf16x8*>(&Bs[0][row * TR_LDB + m4 * 8]) = (k_ok && n_ok) ? rbh[r] : zv;
      }
    }
    if constexpr (!B_BF16) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int row = kf + 4 * r;
        const floatx4 v = (k0 + row < kend && n_ok) ? rbf[r] : zero4();
        bf16x4 hi, lo;
        split_bf16_4(v, hi, lo);
        *reinterpret_cast<bf16x4*>(&Bs[0][row * TR_LDB + c4 * 4]) = hi;
        if constexpr (!ONE) *reinterpret_cast<bf16x4*>(&Bs[NBT - 1][row * TR_LDB + c4 * 4]) = lo;
      }
    }
  };
  // transpose reads: lane (block b = lane / 16, i = lane % 16) points at row 8 * (b / 2) + i / 4,
  // columns 16 * (b % 2) + 4 * (i % 4) .. + 3 of a 32-column block and receives column
  // 16 * (b % 2) + i = lane % 32 of rows 8 * (lane / 32) .. + 3
  const int i16 = lane & 15, half = (lane >> 4) & 1;
  const int a_off = (lh * 8 + (i16 >> 2)) * TR_LDA + wm * 64 + half * 16 + 4 * (i16 & 3);
  const int b_off = (lh * 8 + (i16 >> 2)) * TR_LDB + wn * 128 + half * 16 + 4 * (i16 & 3);

  if (kbeg < kend) {
    fetch(kbeg);
    stash(kbeg);
    __syncthreads();
    for (long long k0 = kbeg; k0 < kend; k0 += TR_TK) {
      const bool more = k0 + TR_TK < kend;
      if (more) fetch(k0 + TR_TK);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(2);
#pragma unroll
      for (int c = 0; c < TR_TK / 16; ++c) {
        bf16x8 fa[NAT][2], fb[NBT][4];
#pragma unroll
        for (int t = 0; t < NAT; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            fa[t][i] = lds_tr8(&As[t][a_off + c * 16 * TR_LDA + i * 32], TR_LDA);
#pragma unroll
        for (int t = 0; t < NBT; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            fb[t][j] = lds_tr8(&Bs[t][b_off + c * 16 * TR_LDB + j * 32], TR_LDB);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[0][j], acc[i][j], 0, 0, 0);
            if constexpr (!ONE)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[NAT - 1][i], fb[0][j], acc[i][j], 0, 0, 0);
            if constexpr (!B_BF16 && !ONE)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][i], fb[NBT - 1][j], acc[i][j], 0, 0, 0);
          }
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      if (more) {
        stash(k0 + TR_TK);
        __syncthreads();
      }
    }
  }
  // column sums: the eight row groups of a column meet in LDS (the A tiles are free now)
  float* red = reinterpret_cast<float*>(&As[0][0]);      // [8][GT] floats = 4 KB
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) red[k8 * GT + m4 * 4 + e] = colsum[e];
  __syncthreads();
  if (tid < GT && m0 + tid < M) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) sum += red[q * GT + tid];
    // every column tile holds the same sums: the first one reports them
    if (nt == 0) a.bpart[(long long)z * M + m0 + tid] = sum;
  }
  float* out = a.part + (long long)z * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int mm = m0 + wm * 64 + i * 32 + 8 * (e / 4) + 4 * lh + (e & 3);
        const int nn = n0 + wn * 128 + j * 32 + li;
        if (mm < M && nn < N) out[(long long)mm * N + nn] = acc[i][j][e];
      }
}

// The same partial products for fp32 operands carried as two fp16 terms each (see gemm_terms.h): S and the
// second operand (h or x) are split on their way to LDS, three products.  Staging as in
// grad_gemm_tr_kernel: LDS rows in memory order, fragments from the transpose read.
// NB: 32-column blocks of a wave; 4: tiles of 128 x 256, 2: of 128 x 128.  Every operand element is loaded,
// multiplied and split once per tile that uses it; the wide tile does that a quarter less often per MFMA.
// Columns are exchanged by bits 0-1 of the row, so that the four rows of a read fall on different banks.
// The sums run over time, so it is the columns of both operands that are scaled, and since an adjoint decays backwards
// (2^-0.3 to 2^-1 a step) while inputs begin and end anywhere, the scales move along: a slice whose values leave
// the range of a scale renews the scales from its own largest values, and the sums follow by the same powers of
// two, exactly.  (Scales of a whole split, 128 to 6500 rows: gradients of inputs that end 32 steps before the
// sequence does were 3e-3 off, 64 steps 1.)  In a slice that no scales fit, because rows of it (batch rows, steps) lie
// further apart than fp16 reaches, and in the GRAD_THREES - 1 after it, the operands are three bf16 terms, six
// products.  What two terms leave out of a value is thus at most 2^-20 of the largest of its row and of its
// column in the slice (2^-22 of the value where it is within 2^10 of the column's largest); values that
// are denormal beside normal ones count as zeros.  (The sum runs forwards: backwards it ends up 1.7-3
// times further from 64 bits.)
// What bounds it is issue: per slice and wave 48 MFMAs (1536 clocks of 3700), 230 VALU instructions of staging and 100
// that look whether the scales fit; renewing them takes 3 us.  65536 rows, 1536 x 1024 0.79 ms (261 TFLOP/s; six
// products of three bf16 terms 1.07, two terms with scales of a whole split 0.69), 1536 x 512 0.45 (0.55,
// 0.37), 3072 x 1024 1.53 (2.09, 1.25), 12800 rows, 3000 x 1000 0.31 (0.42, 0.30).  By the data, 65536 rows x
// 1536 x (1024 + 512): dense 1.31, inputs that end early 1.29, one-hot 1.37, 2 % dense 1.51, rectified 1.48, a loss
// that differs by 10^3 between batch rows 1.52, by 10^6 3.3 (three terms throughout; with fp32 slices 6.2),
// columns of the inputs by 10^6 3.5; six products throughout without a look at scales 1.6.
// Branches that are rarely taken are marked as such: without that the compiler spills sums around the products.
constexpr int HS_TK = 32;
// A column's largest value of a slice is brought into [2^GRAD_TOP, 2^(GRAD_TOP + 1)) when the scales are renewed, and
// they stay as long as it and the rows' largest values are within [2^GRAD_LOW, 2^GRAD_HIGH).  (GRAD_TOP 6 to
// 10: the same time.)  A scale rises by up to 2^GRAD_RISE above the least one of its column: no sum overflows.
constexpr int GRAD_TOP = 8, GRAD_LOW = -5, GRAD_HIGH = 15, GRAD_RISE = 30, GRAD_THREES = 8;
constexpr int EXP2_MAX = 127;              // of a column that has held nothing but zeros

__device__ inline int exponent_of(float x) { return (int)(__float_as_uint(x) >> 23) - 127; }
__device__ inline void top4(floatx4& m, floatx4 v) {
#pragma unroll
  for (int e = 0; e < 4; ++e) m[e] = fmaxf(m[e], fabsf(v[e]));
}
template <int CTRL>
__device__ inline unsigned dpp(unsigned x) {
  return __builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, false);
}
constexpr int DPP_XOR1 = 0xb1, DPP_XOR2 = 0x4e, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128;
// Largest of the lanes' values of each of four columns that Q neighbouring lanes take of a row, the other lanes of the
// wave of other rows: lane i receives it for column i / 16 of its four.
template <int Q>
__device__ inline float column_top(const floatx4& m) {
  auto top2 = [](auto x) { return fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])); };
  const float a = top2(__builtin_amdgcn_permlane32_swap(__float_as_uint(m[0]), __float_as_uint(m[2]), false, false));
  const float b = top2(__builtin_amdgcn_permlane32_swap(__float_as_uint(m[1]), __float_as_uint(m[3]), false, false));
  const float c = top2(__builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false));
  return Q == 16 ? c : fmaxf(c, __uint_as_float(dpp<DPP_ROR8>(__float_as_uint(c))));
}
// The lanes' bits of a row that Q neighbouring lanes take.
template <int Q>
__device__ inline unsigned row_or(unsigned x) {
  x |= dpp<DPP_XOR1>(x);
  x |= dpp<DPP_XOR2>(x);
  x |= dpp<DPP_HALF_MIRROR>(x);
  return Q == 16 ? x | dpp<DPP_ROR8>(x) : x;
}
// Whether two fp16 terms plainly carry a slice's values in the scales of their columns: every column and every row has
// a value of at least 2, and none is 2^GRAD_HIGH or more.  From the terms as a wave stages them, row after row (Q
// neighbouring lanes to a row, R rows to a lane): "at least 2" is one bit of a first term, so that
// bits are collected instead of largest values.  Zeros do not fit here (all zeros of S do: an adjoint that
// has decayed to nothing).
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
template <int R, int Q>
struct GradFit {
  static constexpr unsigned TWO = 0x40004000u;
  unsigned c0 = 0, c1 = 0, rows = 0;
  float top = 0.f;
  // v: the lane's values of row r, t: their first terms
  __device__ inline void add(int r, const floatx4& v, uintx2 t) {
    c0 |= t[0];
    c1 |= t[1];
    rows |= ((t[0] | t[1]) >> r) & (TWO >> r);
    top = fmaxf(fmaxf(fmaxf(top, fabsf(v[0])), fmaxf(fabsf(v[1]), fabsf(v[2]))), fabsf(v[3]));
  }
  // f: the scales of the lane's columns
  __device__ inline unsigned long long off(const floatx4& f) const {
    const auto h = __builtin_amdgcn_permlane32_swap(c0, c1, false, false);
    const unsigned x = h[0] | h[1];
    const auto q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    unsigned c = q[0] | q[1];
    if (Q == 8) c |= dpp<DPP_ROR8>(c);
    unsigned g = row_or<Q>(rows);
    g |= g >> 16;
    constexpr unsigned FULL = 0x7fffu & (0x7fffu << (15 - R));
    const bool low = ((c & TWO) != TWO) | ((g & FULL) != FULL);
    const unsigned long long b = __ballot(low | (top >= (float)(1 << GRAD_HIGH)));
    const float least = fminf(fminf(f[0], f[1]), fminf(f[2], f[3])) * 0x1p-126f;
    return Q == 8 && __ballot(top > least) == 0 ? 0 : b;
  }
};
// Whether they do not: a value of 2^GRAD_LOW is enough, zeros fit, and what was denormal before it was scaled.
// value(r): row r, scaled by f; scale: that of the lane's column after column_top.
template <int R, int Q, class Value>
__device__ inline bool grad_misfit(const floatx4& f, float scale, Value value) {
  constexpr float low = 1.f / (1 << -GRAD_LOW), high = 1 << GRAD_HIGH;
  floatx4 cm = zero4();
  unsigned in = 0, any = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const floatx4 v = value(r);
    top4(cm, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      in |= fabsf(v[e]) >= low ? 1u << r : 0;
      any |= fabsf(v[e]) > f[e] * 0x1p-126f ? 1u << r : 0;
    }
    __builtin_amdgcn_sched_barrier(0);     // (rows one by one: registers are short)
  }
  const float m = column_top<Q>(cm);
  return (m >= high) | ((m < low) & (m > scale * 0x1p-126f)) | ((row_or<Q>(any) & ~row_or<Q>(in)) != 0);
}
// Renews the scale f of a column whose largest value in the slice is m (all: of the wave's columns), returns by how
// much its exponent changes.  least: the least exponent it has been scaled by.
__device__ inline int grad_renew(float& f, float m, float all, int& least) {
  auto usable = [](float x) { return x >= 0x1p-126f && x <= 3.4028235e38f; };
  const int old = exponent_of(f), t = exponent_of(m) + old;
  int e = old;
  if (usable(m)) {
    if (t > GRAD_TOP || t < 0) e = GRAD_TOP - exponent_of(m);
  } else if (old == EXP2_MAX && usable(all)) {
    e = GRAD_TOP - exponent_of(all);       // (what it will hold is most likely of that size)
  }
  e = max(min(min(e, EXP2_MAX), least + GRAD_RISE), -100);
  f = exp2_int(e);
  least = min(least, e);
  return e - old;
}

template <int NB>
__global__ __launch_bounds__(256, 2) void grad_gemm_x3_kernel(GradArgs a) {
  constexpr int GN = 64 * NB;
  constexpr int APL = HS_TK * GT, BPL = HS_TK * GN;        // elements of a term
  __shared__ __attribute__((aligned(16))) bf16_t tiles_lds[3 * (APL + BPL)];
  __shared__ __attribute__((aligned(16))) float mscale[GT], nscale[GN];
  __shared__ __attribute__((aligned(16))) int change[GT + GN];
  __shared__ int mleast[GT], nleast[GN], refused, renewed;
  bf16_t *const As = tiles_lds, *const Bs = tiles_lds + 3 * APL;
  const int H = a.H, N = a.N, M = 3 * a.H;
  const int tiles = a.mtiles * a.ntiles;
  // an XCD gets consecutive items, split by split: its rows of S and Bm enter one L2 only
  const int item = (blockIdx.x % NXCD) * (gridDim.x / NXCD) + blockIdx.x / NXCD;
  if (item >= tiles * a.splits) return;
  const int tile = item % tiles, z = item / tiles;
  const int nt = tile / a.mtiles;
  const int m0 = (tile % a.mtiles) * GT, n0 = nt * GN;
  const long long kbeg = (long long)z * a.Kper;
  long long kend = kbeg + a.Kper;
  if (kend > a.Ktot) kend = a.Ktot;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, li = lane & 31, lh = lane >> 5;

  // wave: rows wm * 64 .., columns (j / 2) * 128 + wn * 64 + (j % 2) * 32 .. of block j
  floatx16 acc[2][NB];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  // Staging: a wave takes 32 columns of S and GN / 4 of the second operand, all rows of the slice, so that it finds
  // its columns' largest values by itself.  A thread takes four columns of rows srow(r) and xrow(r), whose
  // bits 0-1 (the exchange of columns) do not depend on r; those of half a wave fall on different banks.
  constexpr unsigned XQ = GN / 16;
  constexpr int XG = 64 / XQ, NR = HS_TK / XG;       // lanes to a row, rows at a time
  auto srow = [](unsigned lane, int r) { return (int)(lane / 8) + 8 * r; };
  auto xrow = [](unsigned lane, int r) {
    const int g = lane / XQ;
    return XG * r + (XG == 4 ? (g & 1) * 2 + (g >> 1) : g);
  };
  auto scol = [&](unsigned lane) { return wave * 32 + (int)(lane % 8 * 4); };
  auto xcol = [&](unsigned lane) { return wave * (GN / 4) + (int)(lane % XQ * 4); };
  const int m = m0 + scol(lane), n = n0 + xcol(lane);
  const bool m_ok = m < M, n_ok = n < N;
  const int mc = m_ok ? m : 0, nc = n_ok ? n : 0;
  const int gate = mc / H, jcol = mc - gate * H;
  const int src = gate == 2 ? a.third_off + jcol : mc;
  floatx4 rk[4], rw[4], rb[NR];
  float colsum[2] = {0.f, 0.f};           // of columns scol + 2 lh, + 1: rows of both halves of the wave
  // Slice k0 into registers (rows beyond the split: its last one).  Uniform bases and 32-bit offsets.  (What follows
  // from the thread's position is formed anew for each slice: kept, it would spill, and a reload in front of
  // the products waits for every load in flight.)
  const unsigned koff = 4 * src, woff = 4 * jcol, noff = 4 * nc;
  auto at = [](const float* base, unsigned offset) {
    return ldg4(reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + offset));
  };
  auto fetch = [&](long long k0) {
    if (k0 >= kend) k0 = kend - 1;
    const int last = (int)min(kend - k0, (long long)HS_TK) - 1;
    unsigned t = lane;
    asm volatile("" : "+v"(t));
    const float* const kbase = a.kap0 + (k0 + a.B) * (5LL * H);
    const float* const wbase = a.w + (k0 + a.B) * H;       // kap0 / w rows are one time point ahead
    const float* const bbase = (const float*)a.Bm + k0 * N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const unsigned k = min(srow(t, r), last);
      rk[r] = at(kbase, __umul24(k, 20 * H) + koff);
      rw[r] = at(wbase, __umul24(k, 4 * H) + woff);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
      rb[r] = at(bbase, min(xrow(t, r), last) * (4u * N) + noff);
  };
  // (the scales stay in LDS: registers are short)
  if (tid < GT) {
    mscale[tid] = exp2_int(EXP2_MAX);
    mleast[tid] = EXP2_MAX;
  }
  if (tid < GN) {
    nscale[tid] = exp2_int(EXP2_MAX);
    nleast[tid] = EXP2_MAX;
  }
  if (tid == 0) refused = renewed = 0;
  __syncthreads();
  auto scale4 = [](const float* p) { return *reinterpret_cast<const floatx4*>(p); };
  auto put = [](bf16_t* dst, int plane, floatx4 v) {
    const uintx2 w0 = uintx2{round2_f16(v[0], v[1]), round2_f16(v[2], v[3])};
    float rest[4];                         // (v[e] minus its half of w0: as minus2_f16, v is used again)
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(rest[0]) : "v"(w0[0]), "v"(v[0]));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rest[1]) : "v"(w0[0]), "v"(v[1]));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(rest[2]) : "v"(w0[1]), "v"(v[2]));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rest[3]) : "v"(w0[1]), "v"(v[3]));
    const uintx2 w1 = uintx2{round2_f16(rest[0], rest[1]), round2_f16(rest[2], rest[3])};
    *reinterpret_cast<uintx2*>(dst) = w0;
    *reinterpret_cast<uintx2*>(dst + plane) = w1;
    return w0;
  };
  // the rows in registers to LDS, in terms; whether they do not fit
  auto stash = [&]() {
    unsigned t = lane;
    asm volatile("" : "+v"(t));
    const floatx4 fm = scale4(&mscale[scol(t)]), fn = scale4(&nscale[xcol(t)]);
    GradFit<4, 8> fit;
    bf16_t* const ad = &As[srow(t, 0) * GT + (scol(t) ^ ((srow(t, 0) & 3) << 5))];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const floatx4 v = rk[r] * rw[r] * fm;
      fit.add(r, v, put(ad + 8 * r * GT, APL, v));
      if (r & 1) __builtin_amdgcn_sched_barrier(0);        // (more rows at a time: sums spill)
    }
    GradFit<NR, XQ> fitb;
    bf16_t* const bd = &Bs[xrow(t, 0) * GN + (xcol(t) ^ ((xrow(t, 0) & 3) << 5))];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const floatx4 v = rb[r] * fn;
      fitb.add(r, v, put(bd + XG * r * GN, BPL, v));
      if (r & 1) __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_expect((fit.off(fm) | fitb.off(fn)) == 0, 1)) return false;
    asm volatile("" : "+v"(t));            // (the scaled values are formed anew, and in a branch)
    const floatx4 gm = scale4(&mscale[scol(t)]), gn = scale4(&nscale[xcol(t)]);
    const bool bad = grad_misfit<4, 8>(gm, mscale[scol(t) + t / 16], [&](int r) { return rk[r] * rw[r] * gm; });
    return __ballot(bad | grad_misfit<NR, XQ>(gn, nscale[xcol(t) + t / 16],
                                              [&](int r) { return rb[r] * gn; })) != 0;
  };
  // (columns beyond the matrix are copies of others and not stored; rows beyond the split count as zeros)
  auto clear = [&](long long k0) {
    if (__builtin_expect(k0 + HS_TK > kend, 0)) {
      const int rows = (int)(kend - k0);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (srow(lane, r) >= rows) rk[r] = rw[r] = zero4();
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if (xrow(lane, r) >= rows) rb[r] = zero4();
    }
  };
  // sums times 2^(sign (exps[row] + exps[GT + column]))
  auto add_exponents = [&](const int* exps, int sign) {
    typedef int intx4_ __attribute__((ext_vector_type(4)));
    unsigned t = tid;
    asm volatile("" : "+v"(t));            // (addresses are formed here, not kept through the loop)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      intx4_ me[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        me[q] = *reinterpret_cast<const intx4_*>(&exps[t / 128 * 64 + i * 32 + 8 * q + (t / 32 & 1) * 4]);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int ne = exps[GT + (j >> 1) * 128 + (t / 64 & 1) * 64 + (j & 1) * 32 + t % 32];
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = ldexpf(acc[i][j][e], sign * (me[e / 4][e % 4] + ne));
      }
    }
  };
  // new scales from the rows in registers, the sums are brought to them; whether there are any
  auto rescale = [&](int turn) {
    unsigned t = lane;
    asm volatile("" : "+v"(t));
    floatx4 tm = zero4(), tn = zero4();
#pragma unroll
    for (int r = 0; r < 4; ++r) top4(tm, rk[r] * rw[r]);
#pragma unroll
    for (int r = 0; r < NR; ++r) top4(tn, rb[r]);
    const float m = column_top<8>(tm), n = column_top<XQ>(tn);
    float allm = m, alln = n;              // (of the wave's columns)
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      allm = fmaxf(allm, __shfl_xor(allm, o, 64));
      alln = fmaxf(alln, __shfl_xor(alln, o, 64));
    }
    const int cm = scol(t) + t / 16, cn = xcol(t) + t / 16;
    int d = 0;
    if (t % 16 < 8) d |= change[cm] = grad_renew(mscale[cm], m, allm, mleast[cm]);
    if (t % 16 < XQ) d |= change[GT + cn] = grad_renew(nscale[cn], n, alln, nleast[cn]);
    if (d != 0) renewed = turn;
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(renewed) != turn) return false;
    add_exponents(change, 1);
    return true;
  };
  // the rows in registers to LDS, in three bf16 terms (scaled too: the sums are)
  auto stash3 = [&]() {
    unsigned t = lane;
    asm volatile("" : "+v"(t));
    const floatx4 fm = scale4(&mscale[scol(t)]), fn = scale4(&nscale[xcol(t)]);
    auto put3 = [](bf16_t* dst, int plane, floatx4 v) {
      float x[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const uintx2 w = {round2_bf16(x[0], x[1]), round2_bf16(x[2], x[3])};
        *reinterpret_cast<uintx2*>(dst + i * plane) = w;
        if (i < 2) {
          minus2_bf16(x[0], x[1], w[0]);
          minus2_bf16(x[2], x[3], w[1]);
        }
      }
    };
    bf16_t* const ad = &As[srow(t, 0) * GT + (scol(t) ^ ((srow(t, 0) & 3) << 5))];
    bf16_t* const bd = &Bs[xrow(t, 0) * GN + (xcol(t) ^ ((xrow(t, 0) & 3) << 5))];
#pragma unroll
    for (int r = 0; r < 4; ++r) put3(ad + 8 * r * GT, APL, rk[r] * rw[r] * fm);
#pragma unroll
    for (int r = 0; r < NR; ++r) put3(bd + XG * r * GN, BPL, rb[r] * fn);
  };
  // transpose reads: see grad_gemm_tr_kernel
  const int i16 = lane & 15, half = (lane >> 4) & 1, rr = i16 >> 2;
  int aoff[2], boff[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    aoff[i] = (lh * 8 + rr) * GT + ((wm * 64 + i * 32 + half * 16 + 4 * (i16 & 3)) ^ (rr << 5));
    boff[i] = (lh * 8 + rr) * GN + ((wn * 64 + i * 32 + half * 16 + 4 * (i16 & 3)) ^ (rr << 5));
  }
  auto multiply = [&]() {
#pragma unroll
    for (int c = 0; c < HS_TK / 16; ++c) {
      f16x8 fa[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
          fa[t][i] = __builtin_bit_cast(
              f16x8, lds_tr8(&As[t * APL + aoff[i] + c * 16 * GT], GT));
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        f16x8 fb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          fb[u] = __builtin_bit_cast(
              f16x8, lds_tr8(&Bs[u * BPL + boff[j & 1] + c * 16 * GN + (j >> 1) * 128], GN));
#pragma unroll
        for (int u = 0; u < 3; ++u)              // a0 b0, a1 b0, a0 b1
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[u == 1][i], fb[u == 2], acc[i][j], 0, 0, 0);
      }
    }
  };
  // Six products of three terms.  (Sums of their own, added to the others: accumulating where they are, the compiler
  // keeps two sets of them.)
  auto multiply3 = [&]() {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      floatx16 sum[2];
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[0][e] = sum[1][e] = 0.f;
#pragma unroll 1
      for (int c = 0; c < HS_TK / 16; ++c) {
        bf16x8 fa[3][2], fb[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          fb[t] = lds_tr8(&Bs[t * BPL + boff[j & 1] + c * 16 * GN + (j >> 1) * 128], GN);
#pragma unroll
          for (int i = 0; i < 2; ++i) fa[t][i] = lds_tr8(&As[t * APL + aoff[i] + c * 16 * GT], GT);
        }
#pragma unroll
        for (int s = 2; s >= 0; --s)
#pragma unroll
          for (int t = s; t >= 0; --t)
#pragma unroll
            for (int i = 0; i < 2; ++i)
              sum[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[t][i], fb[s - t], sum[i], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i][j] += sum[i];
    }
  };

  if (kbeg < kend) fetch(kbeg);
  // refused: 2 t if slice t (1, 2, ..) does not fit the scales as they are, 2 t + 1 if no renewed ones either
  int turn = 2, threes = 0;                // slices that three terms take from here on
  for (long long k0 = kbeg; k0 < kend; k0 += HS_TK, turn += 2) {
    clear(k0);
    // a tree of eight rows: one addition per slice into the long sum (four rows: bias gradients 2-15 %
    // further from 64 bits).  The halves of the wave exchange two columns each.  Only the first column
    // tile reports it.
    if (nt == 0) {
      const floatx4 t = (rk[0] * rw[0] + rk[1] * rw[1]) + (rk[2] * rw[2] + rk[3] * rw[3]);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[e]), __float_as_uint(t[2 + e]),
                                                        false, false);
        colsum[e] += __uint_as_float(x[0]) + __uint_as_float(x[1]);
      }
    }
    if (__builtin_expect(threes == 0, 1)) {
      if (stash()) refused = turn;
      __syncthreads();
      if (__builtin_expect(__builtin_amdgcn_readfirstlane(refused) == turn, 0)) {
        bool plain = rescale(turn);
        if (plain) {
          if (stash()) refused = turn + 1;
          __syncthreads();
          plain = __builtin_amdgcn_readfirstlane(refused) != turn + 1;
        }
        if (!plain) threes = GRAD_THREES;
      }
    }
    const bool three = threes > 0;
    if (__builtin_expect(three, 0)) {
      --threes;
      stash3();
      __syncthreads();
      multiply3();
    }
    fetch(k0 + HS_TK);                     // (beyond the split: its last row, not used)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(2);
    if (__builtin_expect(!three, 1)) multiply();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  }
  // the sums as they are
  if (tid < GT) change[tid] = exponent_of(mscale[tid]);
  if (tid < GN) change[GT + tid] = exponent_of(nscale[tid]);
  __syncthreads();
  add_exponents(change, -1);
  {
    // sums that are not finite: with fp32 operands (terms of an infinity make sums of infinities not a number)
    floatx4 s = zero4();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e & 3] = fmaf(acc[i][j][e], 0.f, s[e & 3]);
    const float u = (s[0] + s[1]) + (s[2] + s[3]);
    if (__builtin_expect(__syncthreads_or(u != u), 0)) {
      static_assert(sizeof(tiles_lds) >= 2 * GTK * GLD * sizeof(float), "fp32 slices must fit");
#pragma unroll
      for (int hb = 0; hb < NB / 2; ++hb) {
        if (n0 + hb * 128 >= N) break;               // (uniform)
        floatx16 full[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) full[i][j][e] = 0.f;
        floatx4 unused = zero4();
        grad_contract_f32<float, false>(a, m0, n0 + hb * 128, kbeg, kend, (float*)tiles_lds,
                                        (float*)tiles_lds + GTK * GLD, full, unused);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][2 * hb + j] = full[i][j];
      }
    }
  }
  // column sums of S: those of the rows of a wave meet in LDS (the A tiles are free now)
  float* red = reinterpret_cast<float*>(As);      // [4][GT] floats
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) red[(lane / 8 & 3) * GT + scol(lane) + 2 * lh + e] = colsum[e];
  __syncthreads();
  if (nt == 0 && tid < GT && m0 + tid < M) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) sum += red[q * GT + tid];
    a.bpart[(long long)z * M + m0 + tid] = sum;
  }
  float* out = a.part + (long long)z * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int mm = m0 + wm * 64 + i * 32 + 8 * (e / 4) + 4 * lh + (e & 3);
        const int nn = n0 + (j >> 1) * 128 + wn * 64 + (j & 1) * 32 + li;
        if (mm < M && nn < N) out[(long long)mm * N + nn] = acc[i][j][e];
      }
}

// out[i] = sum over the row splits of part[z][i], four elements per thread.  Few outputs leave most
// of the chip idle and a thread's additions wait for one load after the other, so G thread rows of a
// workgroup share the splits (eight loads in flight each) and meet in LDS, in a fixed order.
template <int G>
__device__ inline void reduce_partials(const floatx4* __restrict__ part, floatx4* __restrict__ out,
                                       long long n4, int splits, unsigned block) {
  constexpr int CW = 256 / G;
  __shared__ floatx4 red[G > 1 ? G : 1][CW];
  const int c = threadIdx.x % CW, grp = threadIdx.x / CW;
  const long long i = (long long)block * CW + c;
  floatx4 s = zero4();
  if (i < n4) {
    int z = grp;
    for (; z + 7 * G < splits; z += 8 * G) {
      floatx4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(z + u * G) * n4 + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; z < splits; z += G) s += part[z * n4 + i];
  }
  if (G > 1) {
    red[grp][c] = s;
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int q = 1; q < G; ++q) s += red[q][c];
  }
  if (i < n4) out[i] = s;
}
template <int G>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const floatx4* __restrict__ part,
                                                              floatx4* __restrict__ out,
                                                              long long n4, int splits) {
  reduce_partials<G>(part, out, n4, splits, blockIdx.x);
}

// Bias gradients from the column sums the two gradient GEMMs leave behind, one row per
// row split: pu[nu][3H] (columns k_r w, k_z w, k_q w) and pw[nw][3H] (k_r w, k_z w, k_n w).
// A workgroup covers 32 columns; its eight thread rows share the splits and meet in LDS.
__device__ inline void bias_reduce(const float* __restrict__ pu, int nu, const float* __restrict__ pw,
                                   int nw, float* __restrict__ db_i, float* __restrict__ db_h, int H,
                                   unsigned block) {
  __shared__ float red[2][8][32];
  const int lane = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int c = block * 32 + lane;
  float su = 0.f, sw = 0.f;
  if (c < 3 * H) {
    for (int z = grp; z < nu; z += 8) su += pu[(long long)z * 3 * H + c];
    if (c >= 2 * H)
      for (int z = grp; z < nw; z += 8) sw += pw[(long long)z * 3 * H + c];
  }
  red[0][grp][lane] = su;
  red[1][grp][lane] = sw;
  __syncthreads();
  if (grp == 0 && c < 3 * H) {
    su = 0.f;
    sw = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      su += red[0][q][lane];
      sw += red[1][q][lane];
    }
    db_h[c] = su;
    db_i[c] = c < 2 * H ? su : sw;
  }
}
__global__ void __launch_bounds__(256)
bias_reduce_kernel(const float* pu, int nu, const float* pw, int nw, float* db_i, float* db_h, int H) {
  bias_reduce(pu, nu, pw, nw, db_i, db_h, H, blockIdx.x);
}
// The three together, where both GEMMs ran in one launch: bu and bw workgroups for dU and dW.
template <int G>
__global__ __launch_bounds__(256) void reduce_pair_kernel(GradPair pair, floatx4* dU, floatx4* dW,
                                                          float* db_i, float* db_h, unsigned bu,
                                                          unsigned bw) {
  const GradArgs &u = pair.g[0], &w = pair.g[1];
  const unsigned b = blockIdx.x;
  if (b < bu)
    reduce_partials<G>((const floatx4*)u.part, dU, 3LL * u.H * u.N / 4, u.splits, b);
  else if (b < bu + bw)
    reduce_partials<G>((const floatx4*)w.part, dW, 3LL * w.H * w.N / 4, w.splits, b - bu);
  else
    bias_reduce(u.bpart, u.splits, w.bpart, w.splits, db_i, db_h, u.H, b - bu - bw);
}

// Row splits of a gradient GEMM.  Enough workgroups for at least two per slot (256 CUs x
// the kernel's resident workgroups: three for the fp32 kernel, two for the others); a
// multiple of 8 (whole splits per XCD) unless fewer than 8 fill the slots as well, chosen
// so that the grid is close to a whole number of rounds over the slots: a partly filled
// last round costs as much time as a full one.
// Tile columns of a gradient GEMM: the bf16 contraction takes 256 where the second operand is
// wider than one 128-column tile.
static int grad_tile_n(int N, int bf16) { return bf16 == 1 && N > GT ? TR_GN : GT; }

static int grad_splits(long long Ktot, int M, int N, int bf16) {
  const int gn = grad_tile_n(N, bf16);
  const long long tiles = (long long)((M + GT - 1) / GT) * ((N + gn - 1) / gn);
  const long long slots = bf16 == 0 ? 768 : 512;
  long long maxs = (Ktot + 4 * GTK - 1) / (4 * GTK);   // at least 4 slices per split
  if (maxs > 256) maxs = 256;
  if (maxs < 1) maxs = 1;
  long long want = (2 * slots + tiles - 1) / tiles;
  if (want > maxs) want = maxs;
  auto efficiency = [&](long long sp) {
    const double rounds = (double)(tiles * sp) / (double)slots;
    return rounds / (double)(long long)(rounds + 0.999999);
  };
  long long best = want < NXCD ? want : want / NXCD * NXCD;
  double best_eff = want < NXCD ? efficiency(want) : 0.0;
  if (best_eff >= 0.97) return (int)best;
  for (long long sp = (want + NXCD - 1) / NXCD * NXCD; sp <= maxs && sp <= 4 * want; sp += NXCD) {
    const double eff = efficiency(sp);
    if (eff > best_eff + 0.02) {
      best_eff = eff;
      best = sp;
    }
    if (eff >= 0.97) break;
  }
  return (int)best;
}

// Tile columns and row splits of the kernel on terms, at most `cap` splits (what the partials have room
// for): the least of rounds over the 512 workgroup slots x (slices x us per slice + 10) + what the partials
// cost.  us per slice of 32 rows, measured: a workgroup alone on its CU 1.9 (128 columns) and 2.9 (256), two
// of them 2.3 and 3.8; partials are written and read at 6 TB/s.  Predicted : measured us of one gradient of
// 65536 rows, 128 / 256 columns at their best splits: 1536 x 1024 963 : 947 / 810 : 793; 1536 x 512 789 : 822 (5
// splits) / 404 : 459; 3072 x 1024 in 256 columns 1589 : 1536.
struct GradX3 {
  int cols, splits;
};
static GradX3 grad_x3_shape(long long Ktot, int M, int N, int cap) {
  constexpr double LONE[2] = {1.9, 2.9}, TWO[2] = {2.3, 3.8};
  GradX3 best = {0, 1};
  double least = 0;
  for (int wide = 0; wide < (N > GT ? 2 : 1); ++wide) {
    const int gn = GT << wide;
    const long long tiles = (long long)((M + GT - 1) / GT) * ((N + gn - 1) / gn);
    for (int sp = 1; sp <= cap; ++sp) {
      const long long n = tiles * sp, rest = n % 512;
      const double slices = (double)((Ktot + 32LL * sp - 1) / (32LL * sp));
      const double slot = slices * TWO[wide] + 10, tail = slices * LONE[wide] + 10;
      const double us = (double)(n / 512) * slot + (rest == 0 ? 0.0 : rest <= 256 ? tail : slot) +
                        (double)sp * M * N * 8 / 6e6;
      if (best.cols == 0 || us < least) {
        least = us;
        best = {gn, sp};
      }
    }
  }
  return best;
}

size_t grad_partial_floats(int T, int B, int D, int H, int bf16) {
  const long long Ktot = (long long)T * B;
  const size_t zu = (size_t)grad_splits(Ktot, 3 * H, H, bf16);
  const size_t zw = (size_t)grad_splits(Ktot, 3 * H, D, bf16);
  const size_t su = zu * 3 * H * H, sw = zw * 3 * H * D;
  return (su > sw ? su : sw) + (zu + zw) * 3 * H;
}

hipError_t launch_param_grads(const float* kap0, const float* w, const float* h, const void* x,
                              float* dW, float* dU, float* db_i, float* db_h, float* part,
                              size_t part_floats, int T, int B, int D, int H, int bf16,
                              int one_term, hipStream_t s) {
  const long long Ktot = (long long)T * B;
  const int M = 3 * H;
  prof_begin(3, s);
  auto done = [&] {
    prof_end(3, 2.0 * (double)Ktot * M * (H + D), 4.0 * (double)Ktot * (5.0 * H + H + H + D), s);
    return hipGetLastError();
  };
  auto problem = [&](int which, int tile_cols, int splits, int slice) {
    GradArgs a;
    a.kap0 = kap0;
    a.w = w;
    a.Bm = which == 0 ? (const void*)h : x;
    a.N = which == 0 ? H : D;
    a.third_off = which == 0 ? 2 * H : 4 * H;
    a.part = part;
    a.bpart = nullptr;
    a.Ktot = Ktot;
    a.B = B;
    a.H = H;
    a.mtiles = (M + GT - 1) / GT;
    a.ntiles = (a.N + tile_cols - 1) / tile_cols;
    const long long per = (Ktot + splits - 1) / splits;
    a.Kper = (per + slice - 1) / slice * slice;
    a.splits = splits;
    return a;
  };
  if (bf16 == 0) {
    // Small problems: both GEMMs in one launch and all sums in a second one, or, with one split, none.
    // At most one round over the slots of the kernel (larger ones gain nothing); the partials of both
    // have to fit, with no more rows per split than by itself (longer sums: 300 x 100 twice, 288 rows
    // instead of 160, 5 % further from 64 bits).  Gradients of 128 rows, 96 x 32 and 96 x 16 (five launches
    // before): 36 -> 17 us; 12800, 300 x 100 and 300 x 12 57 -> 41.
    const long long tiles = (long long)((M + GT - 1) / GT) * ((H + GT - 1) / GT + (D + GT - 1) / GT);
    long long z = (Ktot + 4 * GTK - 1) / (4 * GTK);
    if (z > 256) z = 256;
    const long long fit = (long long)part_floats / ((long long)M * (H + D + 2));
    if (z > 1 && z > fit) z = fit;
    if (z >= NXCD) z = z / NXCD * NXCD;
    auto slices = [&](long long splits) { return ((Ktot + splits - 1) / splits + GTK - 1) / GTK; };
    const int zu = grad_splits(Ktot, M, H, 0), zw = grad_splits(Ktot, M, D, 0);
    if (z >= 1 && tiles * z <= 768 && slices(z) <= slices(zu < zw ? zu : zw)) {
      const int splits = (int)z;
      GradPair pair = {{problem(0, GT, splits, GTK), problem(1, GT, splits, GTK)}, 0, nullptr, nullptr};
      GradArgs &u = pair.g[0], &v = pair.g[1];
      if (splits == 1) {
        u.part = dU;
        v.part = dW;
        pair.db_i = db_i;
        pair.db_h = db_h;
      } else {
        v.part = u.part + (size_t)splits * M * H;
        u.bpart = v.part + (size_t)splits * M * D;
        v.bpart = u.bpart + (size_t)splits * M;
      }
      pair.first = (unsigned)((u.mtiles * u.ntiles * splits + NXCD - 1) / NXCD * NXCD);
      hipLaunchKernelGGL((grad_gemm_kernel<float, true>), dim3(pair.first + v.mtiles * v.ntiles * splits),
                         dim3(256), 0, s, pair);
      if (splits > 1) {
        const unsigned per = splits >= 16 ? 32 : 256;   // (float4 of a workgroup)
        const unsigned bu = (unsigned)((3LL * H * H / 4 + per - 1) / per);
        const unsigned bw = (unsigned)((3LL * H * D / 4 + per - 1) / per);
        const dim3 grid(bu + bw + (3 * H + 31) / 32);
        if (per == 32)
          hipLaunchKernelGGL(reduce_pair_kernel<8>, grid, dim3(256), 0, s, pair, (floatx4*)dU,
                             (floatx4*)dW, db_i, db_h, bu, bw);
        else
          hipLaunchKernelGGL(reduce_pair_kernel<1>, grid, dim3(256), 0, s, pair, (floatx4*)dU,
                             (floatx4*)dW, db_i, db_h, bu, bw);
      }
      return done();
    }
  }
  // splits of the form that runs, if the caller's scratch has room for them, else of the fp32 form
  const int sform = grad_partial_floats(T, B, D, H, bf16) <= part_floats ? bf16 : 0;
  const size_t su = (size_t)grad_splits(Ktot, M, H, sform) * M * H;
  const size_t sw = (size_t)grad_splits(Ktot, M, D, sform) * M * D;
  float* bpart[2];
  int nbpart[2];
  bpart[0] = part + (su > sw ? su : sw);
  for (int which = 0; which < 2; ++which) {
    const int cols = which == 0 ? H : D;
    int splits = grad_splits(Ktot, M, cols, sform);
    int gn = grad_tile_n(cols, bf16);
    if (bf16 == 2) {
      const GradX3 shape = grad_x3_shape(Ktot, M, cols, splits);
      gn = shape.cols;
      splits = shape.splits;
    }
    GradArgs a = problem(which, gn, splits, bf16 == 1 ? HB_TK : GTK);   // (both multiples of 32)
    a.bpart = bpart[which];
    nbpart[which] = splits;
    if (which == 0) bpart[1] = bpart[0] + (size_t)nbpart[0] * M;
    dim3 grid((unsigned)((long long)a.mtiles * a.ntiles * splits));
    if (bf16 == 2) grid.x = (grid.x + NXCD - 1) / NXCD * NXCD;
    if (bf16 == 2 && gn == 2 * GT)
      hipLaunchKernelGGL(grad_gemm_x3_kernel<4>, grid, dim3(256), 0, s, a);
    else if (bf16 == 2)
      hipLaunchKernelGGL(grad_gemm_x3_kernel<2>, grid, dim3(256), 0, s, a);
    else if (bf16 && gn == TR_GN && which == 1 && one_term)
      hipLaunchKernelGGL((grad_gemm_tr_kernel<true, true>), grid, dim3(256), 0, s, a);
    else if (bf16 && gn == TR_GN && one_term)
      hipLaunchKernelGGL((grad_gemm_tr_kernel<false, true>), grid, dim3(256), 0, s, a);
    else if (bf16 && gn == TR_GN && which == 1)
      hipLaunchKernelGGL((grad_gemm_tr_kernel<true, false>), grid, dim3(256), 0, s, a);
    else if (bf16 && gn == TR_GN)
      hipLaunchKernelGGL((grad_gemm_tr_kernel<false, false>), grid, dim3(256), 0, s, a);
    else if (bf16 && which == 1)
      hipLaunchKernelGGL(grad_gemm_bf16_kernel<true>, grid, dim3(256), 0, s, a);
    else if (bf16)
      hipLaunchKernelGGL(grad_gemm_bf16_kernel<false>, grid, dim3(256), 0, s, a);
    else
      hipLaunchKernelGGL((grad_gemm_kernel<float, false>), grid, dim3(256), 0, s,
                         GradPair{{a, a}, grid.x, nullptr, nullptr});
    const long long n = (long long)M * a.N;
    // (3 H N is a multiple of four: so are H and N)
    const long long n4 = n / 4;
    floatx4* dst = (floatx4*)(which == 0 ? dU : dW);
    if (n4 < 65536 && splits >= 16)
      hipLaunchKernelGGL(reduce_partials_kernel<8>, dim3((unsigned)((n4 + 31) / 32)), dim3(256), 0,
                         s, (const floatx4*)part, dst, n4, splits);
    else
      hipLaunchKernelGGL(reduce_partials_kernel<1>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0,
                         s, (const floatx4*)part, dst, n4, splits);
  }
  hipLaunchKernelGGL(bias_reduce_kernel, dim3((3 * H + 31) / 32), dim3(256), 0, s, bpart[0],
                     nbpart[0], bpart[1], nbpart[1], db_i, db_h, H);
  return done();
}

}  // namespace mg

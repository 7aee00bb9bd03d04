// Forward kernels: input projection GEMM and the fused GRU level step
// Phi_gamma(x, h) (Eq. 1 gates + Eq. 16 / Eq. 3 update) with the MGRIT epilogues
// (relaxation update of Alg. 1, residual + restriction of Alg. 2 lines 2-3, the
// right-hand side of Eq. 11, and the adjoint coefficient vectors).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "gates.h"
#include "gemm_core.h"
#include "gemm_core_bf16.h"
#include "gemm_terms.h"
#include "phi_elem.h"
#include "skinny.h"

namespace mg {

// ---------------------------------------------------------------------------
// Projection: P[M,N] = X[M,K] W[N,K]^T + bias[N]       (input half of Eq. 1)
// ---------------------------------------------------------------------------
typedef TileCfg<2, 2, 2, 2, 1> ProjCfg;   // 128 x 128 tile, 256 threads

__global__ __launch_bounds__(ProjCfg::NT) void projection_kernel(
    const float* __restrict__ X, const float* __restrict__ W, const float* __restrict__ bias,
    float* __restrict__ P, long long M, int N, int K) {
  typedef ProjCfg C;
  __shared__ __attribute__((aligned(16))) float lds[C::LDS_FLOATS];
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const int tid = threadIdx.x;

  // rows beyond the matrix are clamped to its last row (their results are never
  // stored); k beyond K contributes zeros
  const float* arow[C::A_CHUNKS];
  const float* brow[C::B_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row<C>(s);
    arow[s] = X + (r < M ? r : M - 1) * K;
  }
#pragma unroll
  for (int s = 0; s < C::B_CHUNKS; ++s) {
    int r = n0 + chunk_row<C>(s);
    brow[s] = W + (long long)(r < N ? r : N - 1) * K;
  }
  Acc<C> acc;
  acc.zero();
  auto la = [&](int s, int k) { return ldg4(arow[s] + k); };
  auto lb = [&](int s, int k) { return ldg4(brow[s] + k); };
  if (K % C::TK == 0)
    gemm_nt_tile<C, false>(acc, K, la, lb, Identity4(), Identity4(), lds);
  else
    gemm_nt_tile<C, true>(acc, K, la, lb, Identity4(), Identity4(), lds);

#pragma unroll
  for (int a = 0; a < C::BM; ++a)
#pragma unroll
    for (int b = 0; b < C::BN; ++b) {
      int row, col;
      acc_coord<C>(a, b, 0, row, col);
      const int n = n0 + col;
      if (n >= N) continue;
      const float bv = bias[n];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc_coord<C>(a, b, e, row, col);
        const long long m = m0 + row;
        if (m < M) P[m * N + n] = acc.v[0][a][b][e] + bv;
      }
    }
}

// bf16 inputs and weights (ProjCfgB), or fp32 inputs with the weights given as their three
// bf16 terms W3[3][N,K] (ProjCfgS); fp32 accumulation and output
typedef TileCfgB<2, 2, 2, 2, 1, false> ProjCfgB;
typedef TileCfgB<2, 2, 2, 2, 1, true, 1, 1, 2, 3, 32, true, true> ProjCfgS;

template <class C>
__global__ __launch_bounds__(C::NT, C::NP == 3 ? 2 : 1) void projection_kernel_bf16(
    const void* __restrict__ Xv, const bf16_t* __restrict__ W, const float* __restrict__ Wf,
    const float* __restrict__ bias, float* __restrict__ P, long long M, int N, int K) {
  typedef typename std::conditional<C::SPLIT_A, float, bf16_t>::type AT;
  const AT* X = (const AT*)Xv;
  __shared__ __attribute__((aligned(16))) bf16_t lds[C::LDS_ELEMS];
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const AT* arow[C::A_CHUNKS];
  const bf16_t* brow[C::B_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row_b<C>(s);
    arow[s] = X + (r < M ? r : M - 1) * K;
  }
#pragma unroll
  for (int s = 0; s < C::B_CHUNKS; ++s) {
    int r = n0 + chunk_row_b<C>(s);
    brow[s] = W + (long long)(r < N ? r : N - 1) * K;
  }
  Acc<C> acc;
  acc.zero();
  if constexpr (C::NP == 3) {
    const long long term = (long long)N * K;
    auto la = [&](int s, int k) { return F32x8{ldg4(arow[s] + k), ldg4(arow[s] + k + 4)}; };
    auto lb = [&](int s, int k) {
      return Bf16x8x3{{ldg8h(brow[s] + k), ldg8h(brow[s] + term + k),
                       ldg8h(brow[s] + 2 * term + k)}};
    };
    auto fa = [](const F32x8& v) { return v; };
    if (K % C::TK == 0)
      gemm_nt_tile_bf16<C, false>(acc, K, la, lb, fa, lds);
    else
      gemm_nt_tile_bf16<C, true>(acc, K, la, lb, fa, lds);
    if (tile_not_finite<C>(acc))
      contract_f32<C>(acc, K,
                      [&](int r, int k) { return ldg4(X + (m0 + r < M ? m0 + r : M - 1) * K + k); },
                      [&](int r) { return Wf + (long long)(n0 + r < N ? n0 + r : N - 1) * K; });
  } else {
    auto la = [&](int s, int k) { return ldg8h(arow[s] + k); };
    auto lb = [&](int s, int k) { return ldg8h(brow[s] + k); };
    auto fa = [](const bf16x8& v) { return v; };
    if (K % C::TK == 0)
      gemm_nt_tile_bf16<C, false>(acc, K, la, lb, fa, lds);
    else
      gemm_nt_tile_bf16<C, true>(acc, K, la, lb, fa, lds);
  }
#pragma unroll
  for (int a = 0; a < C::BM; ++a)
#pragma unroll
    for (int b = 0; b < C::BN; ++b) {
      int row, col;
      acc_coord<C>(a, b, 0, row, col);
      const int n = n0 + col;
      if (n >= N) continue;
      const float bv = bias[n];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc_coord<C>(a, b, e, row, col);
        const long long m = m0 + row;
        if (m < M) P[m * N + n] = acc.v[0][a][b][e] + bv;
      }
    }
}

// The same by the data path of gemm_terms.h, W as packed terms: tiles of 128 x 256, 8 waves.  The split of X
// and the loads of W are paid per column tile, twice as wide here: 65536 rows, 1024 -> 1536 columns 1.12 ->
// 0.93 ms (222 TFLOP/s), 12800 rows, 1000 -> 3000 0.52 -> 0.38.  Same products, same errors.  Launches that leave CUs empty, and widths of one and a half such
// tiles or less, keep the 128 x 128 tiles.
typedef TileCfgB<2, 4, 2, 2, 1, true, 1, 1, 1, 3, 32, true, true> ProjCfgW;

__global__ __launch_bounds__(ProjCfgW::NT, 2) void projection_kernel_wide(
    const float* __restrict__ X, const void* __restrict__ Wt, const float* __restrict__ W,
    const float* __restrict__ bias, float* __restrict__ P, long long M, int N, int K) {
  typedef ProjCfgW C;
  __shared__ f16x8 lds[3 * TermGeom<C>::BUF];
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const float* arow[C::A_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    const long long r = m0 + chunk_row_b<C>(s);
    arow[s] = X + (r < M ? r : M - 1) * K;
  }
  TermAcc<C> acc;
  auto wrow = [&](int, int c) { return (long long)min(n0 + c, N - 1); };
  contract_terms_x3<C>(
      acc, K, [&](int s, int k) { return F32x8{ldg4(arow[s] + k), ldg4(arow[s] + k + 4)}; },
      [](const F32x8& v) { return v; }, Wt, wrow, lds,
      [&](int r, int k) { return ldg4(X + (m0 + r < M ? m0 + r : M - 1) * K + k); },
      [&](int g, int c) { return W + wrow(g, c) * K; });
  store_tile_terms<C>(acc, P, bias, m0, n0, M, N);
}

bool projection_is_wide(long long M, int N, int K) {
  typedef ProjCfgW C;
  return N >= 384 && ((M + C::TM - 1) / C::TM) * ((N + C::TN - 1) / C::TN) >= 192 &&
         6LL * N * K < (1LL << 32);
}

hipError_t launch_projection(const void* X, const void* W, const void* W3, const float* bias,
                             float* P, long long M, int N, int K, int bf16, hipStream_t s) {
  prof_begin(2, s);
  if (bf16 == 3) {
    typedef ProjCfgW C;
    dim3 grid((unsigned)xcd_grid((M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(projection_kernel_wide, grid, dim3(C::NT), 0, s, (const float*)X, W3,
                       (const float*)W, bias, P, M, N, K);
  } else if (bf16 == 2) {
    typedef ProjCfgS C;
    dim3 grid((unsigned)xcd_grid((M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(projection_kernel_bf16<C>, grid, dim3(C::NT), 0, s, X, (const bf16_t*)W3,
                       (const float*)W, bias, P, M, N, K);
  } else if (bf16) {
    typedef ProjCfgB C;
    dim3 grid((unsigned)xcd_grid((M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(projection_kernel_bf16<C>, grid, dim3(C::NT), 0, s, X, (const bf16_t*)W,
                       (const float*)nullptr, bias, P, M, N, K);
  } else {
    typedef ProjCfg C;
    dim3 grid((unsigned)xcd_grid((M + C::TM - 1) / C::TM, (N + C::TN - 1) / C::TN));
    hipLaunchKernelGGL(projection_kernel, grid, dim3(C::NT), 0, s, (const float*)X,
                       (const float*)W, bias, P, M, N, K);
  }
  const double esz = bf16 == 1 ? 2.0 : 4.0;
  prof_end(2, 2.0 * (double)M * N * K, esz * ((double)M * K + (double)N * K) + 4.0 * (double)M * N,
           s);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Fused level step
// ---------------------------------------------------------------------------
// Scalar form used by the few-row kernel: computes and stores one element of row ro.
template <int MODE>
__device__ inline void phi_epi_finish(const PhiArgs& a, const PhiRow& ro, int j, float sr,
                                      float sz, float sn, const PhiEpiIn& e, const PhiBias& bh,
                                      double& nrm, long long coarse_kappa_row = 0) {
  const int H = a.H;
  const PhiOut o =
      phi_elem<MODE>(a.gamma, a.propagator == MGRIT_PROP_IMPLICIT, sr, sz, sn, e, bh, a.gamma2);
  const long long oi = ro.o + j;
  if (MODE == STEP_RELAX) {
    a.u[oi] = o.v0;
  } else if (MODE == STEP_RELAX_RHS) {
    a.u[oi] = o.v0;
    a.gc[ro.a + j] = o.v1;
  } else if (MODE == STEP_RELAX_CK) {
    a.u[oi] = o.v0;
    float* kc = a.gc + coarse_kappa_row;
    kc[j] = o.c0;
    kc[H + j] = o.c1;
    kc[2 * H + j] = o.c2;
    kc[3 * H + j] = o.c3;
  } else if (MODE == STEP_RESID) {
    const long long ai = (ro.a & ~1LL) + j;
    a.gc[ai] = a.resid_adds ? e.prep + o.v0 : o.v0;
    a.uc[ai] = (ro.a & 1) ? o.v1 + o.v0 : o.v1;        // cur - r at the marked points
    nrm += (double)o.v0 * (double)o.v0;
  } else if (MODE == STEP_RHS) {
    a.g[oi] = o.v0;
  } else {
    if (MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2) a.u[oi] = o.v5;
    float* kp = a.uc + ro.a;
    kp[j] = o.v0;
    kp[H + j] = o.v1;
    kp[2 * H + j] = o.v2;
    kp[3 * H + j] = o.v3;
    if (a.kappa_width >= 5 * H) kp[4 * H + j] = o.v4;
    if (MODE == STEP_RELAX_KAPPA2) {
      float* kc = a.gc + coarse_kappa_row;
      kc[j] = o.c0;
      kc[H + j] = o.c1;
      kc[2 * H + j] = o.c2;
      kc[3 * H + j] = o.c3;
    }
  }
}

// Epilogue of one MFMA tile over the staged sums (see EpiStage): per pass a thread
// requests the operands of its items, the sums go through LDS, and each item is
// finished and stored as float4.
struct PhiEpiIn4 {
  floatx4 pr, pz, pn, h, gval, cur;
};
struct PhiEpiExtra4 {     // STEP_RELAX_RHS (pr2..cur2) and STEP_RESID with resid_adds (prep)
  floatx4 pr2, pz2, pn2, cur2, prep;
};

template <class C, int MODE>
__device__ inline void phi_tile_epilogue(const PhiArgs& a, const typename TileSums<C>::type& acc, const PhiRow* rowtab,
                                         float* stage, long long m0, int n0, long long R,
                                         double& nrm, const long long* rowtab2 = nullptr) {
  typedef EpiStage<C> E;
  const int H = a.H;
  const int c4 = E::col4();
  const int j = n0 + c4 * 4;
  const bool colok = E::active() && j < H;
  const int jc = colok ? j : H - 4;                     // clamped columns are never stored
  PhiBias bh[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bh[i] = phi_bias_load(a, jc + i);
  const float gamma = a.gamma;
  const bool implicit = a.propagator == MGRIT_PROP_IMPLICIT;

#pragma unroll
  for (int ba = 0; ba < C::BM; ++ba) {
    __syncthreads();                                    // staging area no longer read
    stage_write<C>(acc, ba, stage);
    // operands that do not depend on the sums: requested before the barrier
    PhiEpiIn4 in[E::ITEMS];
    constexpr bool CK = MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK;
    constexpr bool EXTRA = MODE == STEP_RELAX_RHS || MODE == STEP_RESID || CK;
    PhiEpiExtra4 ex[EXTRA ? E::ITEMS : 1];
    long long oo[E::ITEMS], oa[E::ITEMS];
    long long oa2[CK ? E::ITEMS : 1];
    int trow[E::ITEMS];
#pragma unroll
    for (int it = 0; it < E::ITEMS; ++it) {
      trow[it] = E::tile_row(E::staged_row(it), ba);
      const PhiRow ro = rowtab[trow[it]];               // rows beyond the launch hold its last row
      oo[it] = ro.o;
      oa[it] = ro.a;
      const float* pp = a.P + ro.p + jc;
      in[it].pr = ldg4_stream(pp);
      in[it].pz = ldg4_stream(pp + H);
      in[it].pn = ldg4_stream(pp + 2 * H);
      in[it].h = ldg4(a.u_in + ro.in + jc);
      if (MODE != STEP_KAPPA && a.g) in[it].gval = ldg4(a.g + ro.o + jc);
      else in[it].gval = zero4();
      if (MODE == STEP_RESID || MODE == STEP_RHS) in[it].cur = ldg4(a.u + ro.o + jc);
      else in[it].cur = zero4();
      if (MODE == STEP_RELAX_RHS || CK) {
        ex[it].pr2 = ldg4_stream(pp + a.dp2);
        ex[it].pz2 = ldg4_stream(pp + a.dp2 + H);
        ex[it].pn2 = ldg4_stream(pp + a.dp2 + 2 * H);
        if (MODE == STEP_RELAX_RHS) ex[it].cur2 = ldg4(a.u + ro.o + a.do2 + jc);
        if (CK) oa2[it] = rowtab2[trow[it]];
      }
      if (MODE == STEP_RESID)
        ex[it].prep = a.resid_adds ? ldg4(a.gc + (ro.a & ~1LL) + jc) : zero4();
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < E::ITEMS; ++it) {
      const int rp = E::staged_row(it);
      const floatx4 sr = E::read(stage, 0, rp, c4);
      const floatx4 sz = E::read(stage, 1, rp, c4);
      const floatx4 sn = E::read(stage, 2, rp, c4);
      floatx4 o0, o1, o2, o3, o4, o5;
      floatx4 q0, q1, q2, q3;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        PhiEpiIn e1{in[it].pr[i], in[it].pz[i], in[it].pn[i], in[it].h[i], in[it].gval[i],
                    in[it].cur[i], 0.f, 0.f, 0.f, 0.f, 0.f};
        if (MODE == STEP_RELAX_RHS || CK) {
          e1.pr2 = ex[it].pr2[i];
          e1.pz2 = ex[it].pz2[i];
          e1.pn2 = ex[it].pn2[i];
          if (MODE == STEP_RELAX_RHS) e1.cur2 = ex[it].cur2[i];
        }
        const PhiOut o = phi_elem<MODE>(gamma, implicit, sr[i], sz[i], sn[i], e1, bh[i], a.gamma2);
        o0[i] = o.v0; o1[i] = o.v1; o2[i] = o.v2; o3[i] = o.v3; o4[i] = o.v4; o5[i] = o.v5;
        q0[i] = o.c0; q1[i] = o.c1; q2[i] = o.c2; q3[i] = o.c3;
      }
      if (!colok || m0 + trow[it] >= R) continue;
      const long long oi = oo[it] + j;
      if (MODE == STEP_RELAX) {
        *reinterpret_cast<floatx4*>(a.u + oi) = o0;
      } else if (MODE == STEP_RELAX_RHS) {
        *reinterpret_cast<floatx4*>(a.u + oi) = o0;
        *reinterpret_cast<floatx4*>(a.gc + oa[it] + j) = o1;
      } else if (MODE == STEP_RELAX_CK) {
        *reinterpret_cast<floatx4*>(a.u + oi) = o0;
        float* kc = a.gc + oa2[it] + j;
        *reinterpret_cast<floatx4*>(kc) = q0;
        *reinterpret_cast<floatx4*>(kc + H) = q1;
        *reinterpret_cast<floatx4*>(kc + 2 * H) = q2;
        *reinterpret_cast<floatx4*>(kc + 3 * H) = q3;
      } else if (MODE == STEP_RESID) {
        const long long ai = (oa[it] & ~1LL) + j;
        // (adding the zero of a launch without a prepared half changes no value)
        *reinterpret_cast<floatx4*>(a.gc + ai) = ex[it].prep + o0;
        *reinterpret_cast<floatx4*>(a.uc + ai) = (oa[it] & 1) ? o1 + o0 : o1;   // cur - r if marked
#pragma unroll
        for (int i = 0; i < 4; ++i) nrm += (double)o0[i] * (double)o0[i];
      } else if (MODE == STEP_RHS) {
        *reinterpret_cast<floatx4*>(a.g + oi) = o0;
      } else {
        if (MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2)
          *reinterpret_cast<floatx4*>(a.u + oi) = o5;
        float* kp = a.uc + oa[it] + j;
        *reinterpret_cast<floatx4*>(kp) = o0;
        *reinterpret_cast<floatx4*>(kp + H) = o1;
        *reinterpret_cast<floatx4*>(kp + 2 * H) = o2;
        *reinterpret_cast<floatx4*>(kp + 3 * H) = o3;
        if (a.kappa_width >= 5 * H) *reinterpret_cast<floatx4*>(kp + 4 * H) = o4;
        if (MODE == STEP_RELAX_KAPPA2) {
          float* kc = a.gc + oa2[it] + j;
          *reinterpret_cast<floatx4*>(kc) = q0;
          *reinterpret_cast<floatx4*>(kc + H) = q1;
          *reinterpret_cast<floatx4*>(kc + 2 * H) = q2;
          *reinterpret_cast<floatx4*>(kc + 3 * H) = q3;
        }
      }
    }
  }
}

// ZS: the launch knows that the input states of the rows from a.zero_from on are zero (its
// own instantiation, so that kernel traces list these launches apart).
template <class C, int MODE, bool ZS = false>
__global__ __launch_bounds__(C::NT, C::MINWG) void phi_step_kernel(PhiArgs a) {
  constexpr int LDSF = C::LDS_FLOATS > EpiStage<C>::FLOATS ? C::LDS_FLOATS : EpiStage<C>::FLOATS;
  __shared__ __attribute__((aligned(16))) float lds[LDSF];
  const int H = a.H, B = a.B;
  const long long R = (long long)a.nk * B;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (H + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const int tid = threadIdx.x;
  __shared__ PhiRow rowtab[C::TM];
  __shared__ long long rowtab2[(MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK) ? C::TM : 1];
  if (tid < C::TM) {
    long long r = m0 + tid;
    if (r >= R) r = R - 1;
    rowtab[tid] = phi_row(a, r,
                          (MODE == STEP_KAPPA || MODE == STEP_RELAX_KAPPA ||
                           MODE == STEP_RELAX_KAPPA2) ? a.kappa_width : H);
    if (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
      rowtab2[tid] = phi_row_coarse_kappa(a, r);
  }
  // (visible to all waves after the barriers inside the contraction)

  // A rows: states of the points this tile covers (row = point*B + b); rows beyond
  // the launch are clamped to its last row and never stored.
  const float* arow[C::A_CHUNKS];
  const float* brow[C::B_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row<C>(s);
    if (r >= R) r = R - 1;
    const long long pt = (unsigned)r / (unsigned)B;   // rows < 2^31: 32-bit division
    const int b = (int)(r - pt * B);
    arow[s] = a.u_in + (a.in.at(pt) * B + b) * H;
  }
  // B rows: for gate g the rows n0.. of U_g.
#pragma unroll
  for (int s = 0; s < C::B_CHUNKS; ++s) {
    const int tr = chunk_row<C>(s);
    const int g = tr / C::TN;
    int j = n0 + tr % C::TN;
    if (j >= H) j = H - 1;
    brow[s] = (const float*)a.U + ((long long)g * H + j) * H;
  }
  Acc<C> acc;
  acc.zero();
  auto la = [&](int s, int k) { return ldg4(arow[s] + k); };
  auto lb = [&](int s, int k) { return ldg4(brow[s] + k); };
  // a tile whose input states are known to be zero keeps its zero sums (uniform per workgroup)
  const bool zero_in = ZS && m0 >= a.zero_from;
  if (zero_in) {
  } else if (H % C::TK == 0)
    gemm_nt_tile<C, false>(acc, H, la, lb, Identity4(), Identity4(), lds);
  else
    gemm_nt_tile<C, true>(acc, H, la, lb, Identity4(), Identity4(), lds);

  double nrm = 0.0;
  phi_tile_epilogue<C, MODE>(a, acc, rowtab, lds, m0, n0, R, nrm, rowtab2);
  if (MODE == STEP_RESID && a.norm) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if ((tid & 63) == 0) atomicAdd(a.norm, nrm);
  }
}

// bf16 weights: the fp32 state rows go to LDS as one bf16 tile or as hi + lo tiles (the
// configuration's A2, see gemm_core_bf16.h); gates, update and outputs stay fp32.  With NP = 3 the
// weights are fp32 values, contracted in fp16 terms (gemm_terms.h).
template <class C, int MODE, bool ZS = false>
__global__ __launch_bounds__(C::NT, C::MINWAVES) void phi_step_kernel_bf16(PhiArgs a) {
  constexpr int LDSF =
      C::LDS_ELEMS / 2 + 1 > EpiStage<C>::FLOATS ? C::LDS_ELEMS / 2 + 1 : EpiStage<C>::FLOATS;
  __shared__ __attribute__((aligned(16))) float ldsf[LDSF];
  bf16_t* lds = reinterpret_cast<bf16_t*>(ldsf);
  const int H = a.H, B = a.B;
  const long long R = (long long)a.nk * B;
  long long rt;
  int ct;
  if (!xcd_tile(blockIdx.x, (R + C::TM - 1) / C::TM, (H + C::TN - 1) / C::TN, rt, ct)) return;
  const long long m0 = rt * C::TM;
  const int n0 = ct * C::TN;
  const int tid = threadIdx.x;
  __shared__ PhiRow rowtab[C::TM];
  __shared__ long long rowtab2[(MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK) ? C::TM : 1];
  if (tid < C::TM) {
    long long r = m0 + tid;
    if (r >= R) r = R - 1;
    rowtab[tid] = phi_row(a, r,
                          (MODE == STEP_KAPPA || MODE == STEP_RELAX_KAPPA ||
                           MODE == STEP_RELAX_KAPPA2) ? a.kappa_width : H);
    if (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
      rowtab2[tid] = phi_row_coarse_kappa(a, r);
  }
  // (visible to all waves after the barriers inside the contraction)

  const float* arow[C::A_CHUNKS];
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) {
    long long r = m0 + chunk_row_b<C>(s);
    if (r >= R) r = R - 1;
    const long long pt = (unsigned)r / (unsigned)B;   // rows < 2^31: 32-bit division
    const int b = (int)(r - pt * B);
    arow[s] = a.u_in + (a.in.at(pt) * B + b) * H;
  }
  typename TileSums<C>::type acc;
  auto la = [&](int s, int k) { return F32x8{ldg4(arow[s] + k), ldg4(arow[s] + k + 4)}; };
  auto fa = [](const F32x8& v) { return v; };
  const bool zero_in = ZS && m0 >= a.zero_from;                // see phi_step_kernel
  if (zero_in) {
    acc.zero();
  } else if constexpr (C::NP == 3) {
    auto urow = [&](int g, int c) { return (long long)g * H + min(n0 + c, H - 1); };
    contract_terms<C>(
        acc, H, la, [&](int s) { return row_top<C>(s, H, [&](int k) { return la(s, k); }); }, fa,
        a.U3, 3LL * H, urow, lds,
        [&](int tr, int k) { return ldg4(a.u_in + rowtab[tr].in + k); },
        [&](int g, int c) { return (const float*)a.U + urow(g, c) * H; });
  } else {
    acc.zero();
    const bf16_t* brow[C::B_CHUNKS];
#pragma unroll
    for (int s = 0; s < C::B_CHUNKS; ++s) {
      const int tr = chunk_row_b<C>(s);
      const int g = tr / C::TN;
      int j = n0 + tr % C::TN;
      if (j >= H) j = H - 1;
      brow[s] = (const bf16_t*)a.U + ((long long)g * H + j) * H;
    }
    auto lb = [&](int s, int k) { return ldg8h(brow[s] + k); };
    if (H % C::TK == 0)
      gemm_nt_tile_bf16<C, false>(acc, H, la, lb, fa, lds);
    else
      gemm_nt_tile_bf16<C, true>(acc, H, la, lb, fa, lds);
  }

  double nrm = 0.0;
  phi_tile_epilogue<C, MODE>(a, acc, rowtab, ldsf, m0, n0, R, nrm, rowtab2);
  if (MODE == STEP_RESID && a.norm) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if ((tid & 63) == 0) atomicAdd(a.norm, nrm);
  }
}

// ---------------------------------------------------------------------------
// Few-row variant (coarsest-level propagation, serial scan): see skinny.h
// ---------------------------------------------------------------------------
// Workgroups with many columns keep RR x 3 CT sums plus their operands in registers:
// those instantiations are limited to 512 threads.
template <int CT>
struct PhiSkMaxNT {
  static constexpr int value = CT >= 4 ? 512 : SK_MAXNT;
};

template <int CT, int MODE, class WT>
__global__ __launch_bounds__(PhiSkMaxNT<CT>::value) void phi_skinny_kernel(PhiArgs a,
                                                                           int rows_block) {
  constexpr int NU = 3 * CT;
  constexpr int VP = sk_pow2_ceil(SK_RR * NU);
  __shared__ float red[(SK_MAXNT / 64) * VP];
  const int H = a.H;
  const int R = a.nk * a.B;
  const int r0 = blockIdx.y * rows_block;
  const int rows_here = min(rows_block, R - r0);
  const SkGeom geo = sk_geom(rows_block, H);
  const int ksl = geo.ksl;
  const int tid = threadIdx.x;
  const int ks = tid & (ksl - 1), rg = tid / ksl;
  const int j0 = blockIdx.x * CT;
  const int aux_w =
      (MODE == STEP_KAPPA || MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2) ? a.kappa_width
                                                                                    : H;

  // this thread's output element (if any): its operands are requested first so
  // that their latency overlaps the dot products
  const int n_out = rows_here * CT;
  const bool epi = tid < n_out && j0 + tid % CT < H;
  int e_j = 0;
  PhiRow ero = {};
  PhiEpiIn ein = {};
  PhiBias ebh = {};
  if (epi) {
    ero = phi_row(a, r0 + tid / CT, aux_w);
    e_j = j0 + tid % CT;
    ein = phi_epi_load<MODE>(a, ero, e_j);
    ebh = phi_bias_load(a, e_j);
  }

  // rows beyond the block are clamped to its last row (their sums are never used)
  const float* hrow[SK_RR];
#pragma unroll
  for (int i = 0; i < SK_RR; ++i) {
    const int r = r0 + min(rg * SK_RR + i, rows_here - 1);
    const long long pt = (unsigned)r / (unsigned)a.B;   // rows < 2^31: 32-bit division
    const int b = r - (int)pt * a.B;
    hrow[i] = a.u_in + (a.in.at(pt) * a.B + b) * H;
  }
  const WT* urow[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int g = u / CT, j = min(j0 + u % CT, H - 1);
    urow[u] = (const WT*)a.U + ((long long)g * H + j) * H;
  }
  float acc[SK_RR][NU];
  skinny_dot<NU, WT>(acc, H, ks, ksl, urow, [&](int i, int k) { return ldg4(hrow[i] + k); });
  float v[VP];
#pragma unroll
  for (int q = 0; q < VP; ++q) v[q] = q < SK_RR * NU ? acc[q / NU][q % NU] : 0.f;
  skinny_reduce<VP>(v, red, rg, ks, ksl);
  __syncthreads();

  double nrm = 0.0;
  for (int e = tid; e < n_out; e += geo.nt) {
    const int row = e / CT, c = e % CT;
    const int j = j0 + c;
    if (j >= H) continue;
    const int grp = row / SK_RR, base = (row % SK_RR) * NU;
    const float sr = skinny_sum<VP>(red, grp, base + c, ksl);
    const float sz = skinny_sum<VP>(red, grp, base + CT + c, ksl);
    const float sn = skinny_sum<VP>(red, grp, base + 2 * CT + c, ksl);
    if (e == tid && epi) {
      phi_epi_finish<MODE>(a, ero, e_j, sr, sz, sn, ein, ebh, nrm,
                           (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
                               ? phi_row_coarse_kappa(a, r0 + row) : 0);
    } else {   // more outputs than threads (tiny K only)
      const PhiRow ro = phi_row(a, r0 + row, aux_w);
      phi_epi_finish<MODE>(a, ro, j, sr, sz, sn, phi_epi_load<MODE>(a, ro, j), phi_bias_load(a, j),
                           nrm,
                           (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
                               ? phi_row_coarse_kappa(a, r0 + row) : 0);
    }
  }
  if (MODE == STEP_RESID && a.norm && nrm != 0.0) atomicAdd(a.norm, nrm);
}

// ---------------------------------------------------------------------------
// Few-row step on the matrix pipe
// ---------------------------------------------------------------------------
// The same step for up to 64 rows with the contraction on v_mfma_f32_16x16x4_f32, which sums
// over k inside the instruction: no partial sums travel between lanes, and a step needs a
// quarter of the waves of the vector form above (a dependent step waits for its slowest wave).
// A workgroup owns one block of 16 rows and FR_NC hidden columns; the three gates of those
// columns are the 16 columns of the MFMA block (3 x 5, one idle).  Its waves split K: wave w
// contracts k in [w kslice, (w + 1) kslice), every load of its slice issued before the first
// MFMA, and the 16 x 16 partial blocks meet in LDS.  Operand layout of the instruction: lane l
// supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16]; a lane loads four
// consecutive k of its row (k = 16 s + 4 (l / 16) + e, e = 0..3) and feeds four MFMAs, so A and
// B agree on the k each of them contracts; result register v of lane l is D[4 (l / 16) + v][l % 16].
constexpr int FR_NC = 5;       // hidden columns per workgroup
constexpr int FR_KB = 8;       // blocks of sixteen k whose loads a wave keeps in flight
constexpr int FR_MAXW = 8;     // waves per workgroup at most

template <int MODE, class WT>
__global__ __launch_bounds__(64 * FR_MAXW) void phi_fewrow_kernel(PhiArgs a, int kslice) {
  __shared__ float part[FR_MAXW][16][17];
  const int H = a.H;
  const int R = a.nk * a.B;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nt = blockDim.x, nw = nt >> 6;
  const int li = lane & 15, kq = lane >> 4;
  const int j0 = blockIdx.x * FR_NC;
  const int r0 = blockIdx.y * 16;
  const int rows_here = min(16, R - r0);
  const int aux_w =
      (MODE == STEP_KAPPA || MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2) ? a.kappa_width
                                                                                    : H;
  // this thread's output element (if any): its operands are requested first so that their
  // latency overlaps the contraction
  const int n_out = rows_here * FR_NC;
  const bool epi = tid < n_out && j0 + tid % FR_NC < H;
  int e_j = 0;
  PhiRow ero = {};
  PhiEpiIn ein = {};
  PhiBias ebh = {};
  if (epi) {
    ero = phi_row(a, r0 + tid / FR_NC, aux_w);
    e_j = j0 + tid % FR_NC;
    ein = phi_epi_load<MODE>(a, ero, e_j);
    ebh = phi_bias_load(a, e_j);
  }

  // A: state row of this lane (rows beyond the block are clamped; their sums are never used)
  const int r = r0 + min(li, rows_here - 1);
  const long long pt = (unsigned)r / (unsigned)a.B;   // rows < 2^31: 32-bit division
  const int b = r - (int)pt * a.B;
  const float* hrow = a.u_in + (a.in.at(pt) * a.B + b) * H;
  // B: weight row of this lane's MFMA column: gate li / FR_NC, hidden column j0 + li % FR_NC
  // (column 15 idles on a copy of column 14)
  const int lc = min(li, 3 * FR_NC - 1);
  const WT* urow = (const WT*)a.U +
                   ((long long)(lc / FR_NC) * H + min(j0 + lc % FR_NC, H - 1)) * H;

  // two accumulators: consecutive MFMAs do not wait for each other's result
  floatx4 acc = zero4(), acc1 = zero4();
  const int k_end = min(H, (wv + 1) * kslice);
  for (int kb = wv * kslice; kb < k_end; kb += 16 * FR_KB) {
    floatx4 av[FR_KB], bv[FR_KB];
#pragma unroll
    for (int s = 0; s < FR_KB; ++s) {
      const int k = kb + 16 * s + 4 * kq;
      const int kc = min(k, H - 4);                  // H is a multiple of 4
      av[s] = ldg4(hrow + kc);
      bv[s] = ldg4w(urow + kc);
    }
    // all loads of the slice are in flight before anything waits for one of them
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < FR_KB; ++s) {
      if (kb + 16 * s + 4 * kq >= k_end) av[s] = zero4();
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s][e], bv[s][e], acc, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s][e + 1], bv[s][e + 1], acc1, 0, 0, 0);
      }
    }
  }
  acc += acc1;
#pragma unroll
  for (int v = 0; v < 4; ++v) part[wv][4 * kq + v][li] = acc[v];
  __syncthreads();

  double nrm = 0.0;
  for (int e = tid; e < n_out; e += nt) {
    const int row = e / FR_NC, c = e % FR_NC;
    const int j = j0 + c;
    if (j >= H) continue;
    float sr = 0.f, sz = 0.f, sn = 0.f;
    for (int w = 0; w < nw; ++w) {
      sr += part[w][row][c];
      sz += part[w][row][FR_NC + c];
      sn += part[w][row][2 * FR_NC + c];
    }
    if (e == tid && epi) {
      phi_epi_finish<MODE>(a, ero, e_j, sr, sz, sn, ein, ebh, nrm,
                           (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
                               ? phi_row_coarse_kappa(a, r0 + row) : 0);
    } else {   // more outputs than threads (one-wave workgroups only)
      const PhiRow ro = phi_row(a, r0 + row, aux_w);
      phi_epi_finish<MODE>(a, ro, j, sr, sz, sn, phi_epi_load<MODE>(a, ro, j), phi_bias_load(a, j),
                           nrm,
                           (MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK)
                               ? phi_row_coarse_kappa(a, r0 + row) : 0);
    }
  }
  if (MODE == STEP_RESID && a.norm && nrm != 0.0) atomicAdd(a.norm, nrm);
}

typedef TileCfg<2, 2, 2, 1, 3> PhiBig;    // 128 rows x 64 hidden columns (x3 gates), 256 threads
typedef TileCfg<2, 2, 1, 1, 3> PhiMid;    //  64 rows x 64 hidden columns, 256 threads
// few rows:  32 rows x 32 hidden columns, 4 waves splitting K (slices of 128)
typedef TileCfg<1, 1, 1, 1, 3, 128, 1, 4> PhiSmall;
typedef TileCfgB<2, 2, 2, 1, 3, true> PhiBigB;
typedef TileCfgB<2, 2, 1, 1, 3, true> PhiMidB;
typedef TileCfgB<1, 1, 1, 1, 3, true, 4> PhiSmallB;
// the same tiles with the state as one bf16 term
typedef TileCfgB<2, 2, 2, 1, 3, true, 1, 1, 2, 1, 64, false> PhiBigF;
typedef TileCfgB<2, 2, 1, 1, 3, true, 1, 1, 2, 1, 64, false> PhiMidF;
typedef TileCfgB<1, 1, 1, 1, 3, true, 4, 1, 2, 1, 64, false> PhiSmallF;
// 64 x 64 with two groups of four waves splitting K (slices of 128): half the dependent slices
// per workgroup, for launches whose tiles do not fill the CUs twice anyway (one workgroup per
// CU: 110 KB of LDS with both groups' sums staged); 22.5 -> 20.3 us at 512 rows x 1024
typedef TileCfgB<2, 2, 1, 1, 3, true, 2, 1, 1, 1, 64, false> PhiMidFK;
// fp32 operands in terms: K-slices of 32 keep two workgroups' tiles in a CU's LDS
typedef TileCfgB<2, 2, 2, 1, 3, true, 1, 1, 2, 3, 32> PhiBigS;
typedef TileCfgB<2, 2, 1, 1, 3, true, 1, 1, 2, 3, 32> PhiMidS;
// 64 x 32 with two groups of two waves splitting K, for few tiles of 64 x 64 (us, 64 x 64 : this): 1024 rows
// x 264 (80 tiles) 10.8 : 9.0, 2048 x 264 (160) 11.6 : 12.7, 1024 x 520 (144) 16.3 : 16.4, 2048 x 512 (256) 17.8 :
// 17.6, 1600 x 776 (325) 31 : 40, 4096 x 512 (512) 26 : 32.  (Up to 511 tiles by a line drawn on three bf16
// terms: 64 : 50 at 1024 x 1024.)
typedef TileCfgB<2, 1, 1, 1, 3, true, 2, 1, 2, 3, 32> PhiNarrowS;
// 64 x 64 as eight waves, two groups splitting K, one workgroup per CU, for one round of them: 1024 rows x
// 1024 (256 tiles) 25 us, 28 without the split and 29 with 64 x 32; 2048 x 512 (256) 16, 18 and 18.  From 384
// columns on, where there are slices to split
typedef TileCfgB<2, 2, 1, 1, 3, true, 2, 1, 1, 3, 32> PhiMidKS;

#define MG_LAUNCH_BY_MODE(KERNEL, ...)                                                   \
  switch (a.mode) {                                                                      \
    case STEP_RELAX:                                                                     \
      if (a.zero_from > 0)                                                               \
        hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX, true>), grid, block, 0, s, a); \
      else                                                                               \
        hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX>), grid, block, 0, s, a);     \
      break;                                                                             \
    case STEP_RESID:                                                                     \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RESID>), grid, block, 0, s, a);       \
      break;                                                                             \
    case STEP_RHS:                                                                       \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RHS>), grid, block, 0, s, a);         \
      break;                                                                             \
    case STEP_RELAX_KAPPA:                                                               \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX_KAPPA>), grid, block, 0, s, a); \
      break;                                                                             \
    case STEP_RELAX_CK:                                                                  \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX_CK>), grid, block, 0, s, a);    \
      break;                                                                             \
    case STEP_RELAX_KAPPA2:                                                              \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX_KAPPA2>), grid, block, 0, s, a); \
      break;                                                                             \
    case STEP_RELAX_RHS:                                                                 \
      if (a.zero_from > 0)                                                               \
        hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX_RHS, true>), grid, block, 0, s, a); \
      else                                                                               \
        hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_RELAX_RHS>), grid, block, 0, s, a); \
      break;                                                                             \
    default:                                                                             \
      hipLaunchKernelGGL((KERNEL<__VA_ARGS__, STEP_KAPPA>), grid, block, 0, s, a);       \
  }

template <class CS>
static void launch_phi_x3(const PhiArgs& a, hipStream_t s) {
  const long long R = (long long)a.nk * a.B;
  dim3 grid((unsigned)xcd_grid((R + CS::TM - 1) / CS::TM, (a.H + CS::TN - 1) / CS::TN));
  dim3 block(CS::NT);
  MG_LAUNCH_BY_MODE(phi_step_kernel_bf16, CS)
}

// CS: tile of the form in terms; void: such a launch runs on the fp32 tile (the 32 x 32 tiles of
// the smallest launches: a training step of 128 x 100 x 1000, whose serial steps are such launches,
// takes 7.27 ms with them in fp32 and 7.51 with terms, 256 x 65 x 184 2.45 and 2.67)
template <class C, class CB, class CS, class CF>
static void launch_phi_cfg(const PhiArgs& a, hipStream_t s) {
  const long long R = (long long)a.nk * a.B;
  static_assert(CF::TM == CB::TM && CF::TN == CB::TN, "tile shapes must agree");
  if constexpr (!std::is_void<CS>::value) {
    if (a.bf16 == 2) return launch_phi_x3<CS>(a, s);
  }
  if (a.bf16 == 1 && a.one_term) {
    dim3 grid((unsigned)xcd_grid((R + CF::TM - 1) / CF::TM, (a.H + CF::TN - 1) / CF::TN));
    dim3 block(CF::NT);
    MG_LAUNCH_BY_MODE(phi_step_kernel_bf16, CF)
  } else if (a.bf16 == 1) {
    dim3 grid((unsigned)xcd_grid((R + CB::TM - 1) / CB::TM, (a.H + CB::TN - 1) / CB::TN));
    dim3 block(CB::NT);
    MG_LAUNCH_BY_MODE(phi_step_kernel_bf16, CB)
  } else {
    dim3 grid((unsigned)xcd_grid((R + C::TM - 1) / C::TM, (a.H + C::TN - 1) / C::TN));
    dim3 block(C::NT);
    MG_LAUNCH_BY_MODE(phi_step_kernel, C)
  }
}

constexpr int PHI_SK_ROWS = 32;   // rows per workgroup of the few-row forward step

static int phi_sk_rows(long long R) { return R < PHI_SK_ROWS ? (int)R : PHI_SK_ROWS; }

template <int CT, int MODE>
static void launch_phi_skinny_mode(const PhiArgs& a, dim3 grid, hipStream_t s) {
  const int rb = phi_sk_rows((long long)a.nk * a.B);
  const dim3 block(sk_geom(rb, a.H).nt);
  if (a.bf16 == 1)
    hipLaunchKernelGGL((phi_skinny_kernel<CT, MODE, bf16_t>), grid, block, 0, s, a, rb);
  else
    hipLaunchKernelGGL((phi_skinny_kernel<CT, MODE, float>), grid, block, 0, s, a, rb);
}

template <int MODE>
static void launch_phi_fewrow_mode(const PhiArgs& a, hipStream_t s) {
  const int R = a.nk * a.B;
  // waves per workgroup: K slices of 128 (two blocks of loads in flight at most beyond that)
  int nw = (a.H + 127) / 128;
  nw = nw < 1 ? 1 : (nw > FR_MAXW ? FR_MAXW : nw);
  const int kslice = ((a.H + nw - 1) / nw + 15) / 16 * 16;
  const dim3 grid((unsigned)((a.H + FR_NC - 1) / FR_NC), (unsigned)((R + 15) / 16));
  const dim3 block(64 * nw);
  if (a.bf16 == 1)
    hipLaunchKernelGGL((phi_fewrow_kernel<MODE, bf16_t>), grid, block, 0, s, a, kslice);
  else
    hipLaunchKernelGGL((phi_fewrow_kernel<MODE, float>), grid, block, 0, s, a, kslice);
}

static void launch_phi_fewrow(const PhiArgs& a, hipStream_t s) {
  switch (a.mode) {
    case STEP_RELAX: launch_phi_fewrow_mode<STEP_RELAX>(a, s); break;
    case STEP_RESID: launch_phi_fewrow_mode<STEP_RESID>(a, s); break;
    case STEP_RHS: launch_phi_fewrow_mode<STEP_RHS>(a, s); break;
    case STEP_RELAX_KAPPA: launch_phi_fewrow_mode<STEP_RELAX_KAPPA>(a, s); break;
    case STEP_RELAX_RHS: launch_phi_fewrow_mode<STEP_RELAX_RHS>(a, s); break;
    case STEP_RELAX_KAPPA2: launch_phi_fewrow_mode<STEP_RELAX_KAPPA2>(a, s); break;
    case STEP_RELAX_CK: launch_phi_fewrow_mode<STEP_RELAX_CK>(a, s); break;
    default: launch_phi_fewrow_mode<STEP_KAPPA>(a, s);
  }
}

template <int CT>
static void launch_phi_skinny(const PhiArgs& a, dim3 grid, hipStream_t s) {
  switch (a.mode) {
    case STEP_RELAX: launch_phi_skinny_mode<CT, STEP_RELAX>(a, grid, s); break;
    case STEP_RESID: launch_phi_skinny_mode<CT, STEP_RESID>(a, grid, s); break;
    case STEP_RHS: launch_phi_skinny_mode<CT, STEP_RHS>(a, grid, s); break;
    case STEP_RELAX_KAPPA: launch_phi_skinny_mode<CT, STEP_RELAX_KAPPA>(a, grid, s); break;
    case STEP_RELAX_RHS: launch_phi_skinny_mode<CT, STEP_RELAX_RHS>(a, grid, s); break;
    case STEP_RELAX_KAPPA2: launch_phi_skinny_mode<CT, STEP_RELAX_KAPPA2>(a, grid, s); break;
    case STEP_RELAX_CK: launch_phi_skinny_mode<CT, STEP_RELAX_CK>(a, grid, s); break;
    default: launch_phi_skinny_mode<CT, STEP_KAPPA>(a, grid, s);
  }
}

// MGRIT_FEWROW_VECTOR=1 in the environment selects the vector-FMA form of the few-row step
// (kept for widths below 16 and for comparison)
static bool getenv_vector_fewrow() {
  static const bool v = [] {
    const char* e = std::getenv("MGRIT_FEWROW_VECTOR");
    return e && e[0] == '1';
  }();
  return v;
}

hipError_t launch_phi_step(const PhiArgs& a, hipStream_t s) {
  if (a.nk <= 0) return hipSuccess;
  if (a.propagator == PROP_ODE_DEMO) return launch_ode_step(a, s);
  if (prop_is_lstm(a.propagator)) return launch_lstm_step(a, s);
  const long long R = (long long)a.nk * a.B;
  auto tiles = [&](int tm, int tn) { return ((R + tm - 1) / tm) * ((a.H + tn - 1) / tn); };
  const int kind = R <= 2 * SK_MAXROWS ? 4 : 0;
  // a launch that skips the contraction of its zero-input tiles is its own shape class for
  // the event timings (mode + 16), and only the rows it contracts count as work
  prof_begin(kind, s, R, kind == 0 && a.zero_from > 0 ? a.mode + 16 : a.mode);
  long long rows_done = R;
  auto contracted = [&](int tm) {
    if (a.zero_from > 0) rows_done = std::min<long long>(R, (a.zero_from + tm - 1) / tm * tm);
  };
  if (R <= 2 * SK_MAXROWS && a.H >= 16 && !getenv_vector_fewrow()) {
    launch_phi_fewrow(a, s);
  } else if (R <= 2 * SK_MAXROWS) {
    // two hidden columns (six weight rows) per workgroup measured best from H = 512 up
    // (6.2 us per step at 32 rows x 512, 5.5 at 4 rows x 1024; four columns: +0.5 us)
    const int rb = phi_sk_rows(R);
    const int nrb = (int)((R + rb - 1) / rb);
    const int ct = a.H * nrb >= 512 ? 2 : 1;
    dim3 grid((unsigned)((a.H + ct - 1) / ct), (unsigned)nrb);
    if (ct == 2)
      launch_phi_skinny<2>(a, grid, s);
    else
      launch_phi_skinny<1>(a, grid, s);
  } else if (tiles(PhiBig::TM, PhiBig::TN) >= 384) {
    contracted(PhiBig::TM);
    launch_phi_cfg<PhiBig, PhiBigB, PhiBigS, PhiBigF>(a, s);
  } else if (R > 32 && tiles(PhiMid::TM, PhiMid::TN) >= 128) {
    contracted(PhiMid::TM);
    const long long mid = tiles(PhiMid::TM, PhiMid::TN);
    if (a.bf16 == 2 && a.H >= 384 && mid >= 192 && mid <= 256)
      launch_phi_x3<PhiMidKS>(a, s);
    else if (a.bf16 == 2 && mid < 512)
      launch_phi_x3<PhiNarrowS>(a, s);
    else if (a.bf16 == 1 && a.one_term && tiles(PhiMid::TM, PhiMid::TN) <= 256)
      launch_phi_cfg<PhiMid, PhiMidB, PhiMidS, PhiMidFK>(a, s);
    else
      launch_phi_cfg<PhiMid, PhiMidB, PhiMidS, PhiMidF>(a, s);
  } else {
    contracted(PhiSmall::TM);
    launch_phi_cfg<PhiSmall, PhiSmallB, void, PhiSmallF>(a, s);
  }
  prof_end(kind, 6.0 * (double)rows_done * a.H * a.H, 20.0 * (double)R * a.H, s);
  return hipGetLastError();
}

}  // namespace mg

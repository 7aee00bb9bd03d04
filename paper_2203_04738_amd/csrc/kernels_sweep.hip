// Sweeps of narrow layers: all sub-steps of a relaxation sweep in one launch.
//
// Up to 128 hidden columns the recurrent weights of a layer (196 KB in fp32) fit the registers of
// one workgroup, so a workgroup can take four rows through every sub-step of their interval without
// leaving the CU: wave w holds the weights of hidden columns 16 w .. 16 w + 15 (all gates, all K: 96
// registers) and contracts in quads of rows (quad.h), a lane ends up with the sums of one row and
// column, applies the epilogue of the sub-step's mode, and the new state goes to the other waves
// through LDS (two buffers, one barrier per sub-step).  A chain of step launches costs 6.6 to 10 us
// per sub-step at 100 columns whatever the number of rows, nearly all of it launch, index arithmetic
// and the latency of a tile's only K slice; here a further sub-step costs about 1.4 us (half of it
// MFMAs of the CU's fp32 pipe, the rest LDS, gates and the barrier).  Forward + backward of two layers
// of 128 steps x 100 x 100: 1.76 -> 1.19 ms, training step 64 x 2 x 32: 0.45 -> 0.27 ms, 16384 x 4 x
// 64: 11.2 -> 3.4 ms (its levels of up to 8192 rows; the finest is on tiles, see sweeps_fused in
// api.hip).  Two quads per workgroup at a time spill and gain nothing (800 quads: 30 against 25 us per
// launch).  The same kernel takes the serial solves of these layers (one interval, N sub-steps), whose
// state then travels through LDS instead of memory.  Workgroups loop over quads of rows, so that the
// weights are loaded once per workgroup.
#include <algorithm>

#include "phi_elem.h"
#include "quad.h"

namespace mg {

constexpr int SWP_LD = SWEEP_MAX_H + 16;     // row stride of the state in LDS: 16 (mod 64 banks), so
                                             // that the four rows of a read fall on different banks
constexpr int SWP_MAXWG = 256;               // one workgroup per CU (registers)

struct SweepSteps {
  int n, mid, last, quads;
  long long pstep;
};

// Weights of this lane: column min(16 wave + lane % 16, H - 1), k = 64 c + 16 (lane / 16) + 0..15
// (zero beyond H); at(g, j, k) points at four of them.
template <int NCH, class At>
__device__ inline void sweep_weights(float (&w)[3][NCH][16], int H, At at) {
  const int lane = threadIdx.x & 63;
  const int j = min((int)(threadIdx.x >> 6) * 16 + (lane & 15), H - 1);
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 64 * c + 16 * (lane >> 4) + 4 * q;
        const floatx4 v = k < H ? ldg4(at(g, j, k)) : zero4();
#pragma unroll
        for (int e = 0; e < 4; ++e) w[g][c][4 * q + e] = v[e];
      }
}

template <int NCH>
__global__ __launch_bounds__(256 * NCH, 2) void phi_sweep_kernel(PhiArgs a, SweepSteps sw) {
  __shared__ __attribute__((aligned(16))) float hs[2][4][SWP_LD];
  const int H = a.H, B = a.B, R = a.nk * B;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row = quad_row(lane), col = wv * 16 + (lane & 15), cc = min(col, H - 1);
  float w[3][NCH][16];
  sweep_weights<NCH>(w, H, [&](int g, int j, int k) {
    return (const float*)a.U + ((long long)g * H + j) * H + k;
  });
  const PhiBias bh = phi_bias_load(a, cc);
  const bool implicit = a.propagator == MGRIT_PROP_IMPLICIT;
  for (int e = tid; e < 2 * 4 * SWP_LD; e += blockDim.x) (&hs[0][0][0])[e] = 0.f;
  const long long dP = sw.pstep * B * 3LL * H, dO = (long long)B * H;
  double nrm = 0.0;

  for (int q = blockIdx.x; q < sw.quads; q += gridDim.x) {
    __syncthreads();                          // the last block's reads of the state are done
    const int h4 = H / 4;
    for (int e = tid; e < 4 * h4; e += blockDim.x) {
      const int r = min(4 * q + e / h4, R - 1), pt = r / B;
      *reinterpret_cast<floatx4*>(&hs[0][e / h4][e % h4 * 4]) =
          ldg4(a.u_in + (a.in.at(pt) * B + (r - pt * B)) * H + e % h4 * 4);
    }
    // output elements of this lane (rows beyond the launch repeat its last row and store nothing)
    const int rr = 4 * q + row, r = min(rr, R - 1);
    const long long pt = r / B;
    const int b = r - (int)pt * B;
    const bool ok = rr < R && col < H;
    const float* pp = a.P + (a.p.at(pt) * B + b) * (3LL * H) + cc;
    const long long oi = (a.o.at(pt) * B + b) * H + cc;
    const long long ca = (a.a.at(pt) * B + b) * H + cc;
    const long long ki = (a.o.at(pt) * B + b) * a.kappa_width + cc;
    const bool mark = a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem;
    // operands of a sub-step that no sub-step produces: requested two sub-steps ahead (a sub-step
    // is shorter than a trip to memory)
    struct Ops {
      float pr, pz, pn, g;
    };
    auto request = [&](int j) {
      j = min(j, sw.n - 1);
      const float* p = pp + j * dP;
      return Ops{p[0], p[H], p[2 * H], a.g ? a.g[oi + j * dO] : 0.f};
    };
    Ops n0 = request(0), n1 = request(1);
    __syncthreads();
    float state = hs[0][row][cc], half = 0.f;

    for (int j = 0; j < sw.n; ++j) {
      const int mode = j == 0 ? a.mode : j == sw.n - 1 ? sw.last : sw.mid, buf = j & 1;
      floatx4 op[NCH];
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        op[c] = *reinterpret_cast<const floatx4*>(
            &hs[buf][(lane & 3)][64 * c + 4 * (lane >> 2)]);
      PhiEpiIn e{n0.pr, n0.pz, n0.pn, state, n0.g, 0.f, 0.f, 0.f, 0.f, 0.f, half};
      n0 = n1;
      n1 = request(j + 2);
      // what only the first or last sub-step needs: behind the contraction
      if (mode == STEP_RESID) {
        e.cur = a.u[oi + j * dO];
        if (a.resid_adds && j == 0) e.prep = a.gc[ca];
      }
      if (mode == STEP_RELAX_RHS || mode == STEP_RELAX_KAPPA2 || mode == STEP_RELAX_CK) {
        const float* p2 = pp + j * dP + a.dp2;
        e.pr2 = p2[0];
        e.pz2 = p2[H];
        e.pn2 = p2[2 * H];
        if (mode == STEP_RELAX_RHS) e.cur2 = a.u[oi + j * dO + a.do2];
      }
      floatx4 acc[1][3][1];
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[0][g][0] = zero4();
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        quad_mma<1, 3, 1>(acc, [&](int, int) { return op[c]; },
                           [&](int g) -> const float (&)[16] { return w[g][c]; });
      const float sr = quad_fold(acc[0][0][0]), sz = quad_fold(acc[0][1][0]),
                  sn = quad_fold(acc[0][2][0]);
      const long long o = oi + j * dO;
      if (mode == STEP_RELAX) {
        state = phi_elem<STEP_RELAX>(a.gamma, implicit, sr, sz, sn, e, bh).v0;
        if (ok) a.u[o] = state;
      } else if (mode == STEP_RELAX_RHS) {
        const PhiOut x =
            phi_elem<STEP_RELAX_RHS>(a.gamma, implicit, sr, sz, sn, e, bh, a.gamma2);
        state = x.v0;
        half = x.v1;                     // completed by the residual, in this sweep or later
        if (ok) {
          a.u[o] = x.v0;
          a.gc[ca] = x.v1;
        }
      } else if (mode == STEP_RESID) {
        const PhiOut x = phi_elem<STEP_RESID>(a.gamma, implicit, sr, sz, sn, e, bh);
        if (ok) {
          a.gc[ca] = a.resid_adds ? e.prep + x.v0 : x.v0;
          a.uc[ca] = mark ? x.v1 + x.v0 : x.v1;       // cur - r at the marked points
          nrm += (double)x.v0 * (double)x.v0;
        }
      } else if (mode == STEP_RELAX_CK) {
        const PhiOut x =
            phi_elem<STEP_RELAX_CK>(a.gamma, implicit, sr, sz, sn, e, bh, a.gamma2);
        state = x.v0;
        if (ok) {
          a.u[o] = x.v0;
          float* kc = a.gc + (ca - cc) * 4 + cc;
          kc[0] = x.c0;
          kc[H] = x.c1;
          kc[2 * H] = x.c2;
          kc[3 * H] = x.c3;
        }
      } else {  // STEP_RELAX_KAPPA, STEP_RELAX_KAPPA2
        const bool two = mode == STEP_RELAX_KAPPA2;
        const PhiOut x =
            two ? phi_elem<STEP_RELAX_KAPPA2>(a.gamma, implicit, sr, sz, sn, e, bh, a.gamma2)
                : phi_elem<STEP_RELAX_KAPPA>(a.gamma, implicit, sr, sz, sn, e, bh);
        state = x.v5;
        if (ok) {
          a.u[o] = x.v5;
          float* kp = a.uc + ki + j * (long long)B * a.kappa_width;
          kp[0] = x.v0;
          kp[H] = x.v1;
          kp[2 * H] = x.v2;
          kp[3 * H] = x.v3;
          if (a.kappa_width >= 5 * H) kp[4 * H] = x.v4;
          if (two) {
            float* kc = a.gc + (ca - cc) * 4 + cc;
            kc[0] = x.c0;
            kc[H] = x.c1;
            kc[2 * H] = x.c2;
            kc[3 * H] = x.c3;
          }
        }
      }
      if (j + 1 < sw.n && col < H) hs[buf ^ 1][row][col] = state;
      if (j + 1 < sw.n) __syncthreads();
    }
  }
  if (a.norm && (a.mode == STEP_RESID || sw.last == STEP_RESID)) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if (lane == 0) atomicAdd(a.norm, nrm);
  }
}

template <int NCH>
__global__ __launch_bounds__(256 * NCH, 2) void adj_sweep_kernel(AdjArgs a, SweepSteps sw) {
  __shared__ __attribute__((aligned(16))) float ws[2][4][SWP_LD];
  const int H = a.H, B = a.B, R = a.nk * B;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row = quad_row(lane), col = wv * 16 + (lane & 15), cc = min(col, H - 1);
  float w[3][NCH][16];
  sweep_weights<NCH>(w, H, [&](int g, int j, int k) {
    return (const float*)a.UT + (long long)j * 3 * H + g * H + k;
  });
  for (int e = tid; e < 2 * 4 * SWP_LD; e += blockDim.x) (&ws[0][0][0])[e] = 0.f;
  const long long dK = (long long)B * a.kw, dO = (long long)B * H;
  double nrm = 0.0;

  for (int q = blockIdx.x; q < sw.quads; q += gridDim.x) {
    __syncthreads();                          // the last block's reads of the state are done
    const int h4 = H / 4;
    for (int e = tid; e < 4 * h4; e += blockDim.x) {
      const int r = min(4 * q + e / h4, R - 1), pt = r / B;
      *reinterpret_cast<floatx4*>(&ws[0][e / h4][e % h4 * 4]) =
          ldg4(a.w_in + (a.in.at(pt) * B + (r - pt * B)) * H + e % h4 * 4);
    }
    const int rr = 4 * q + row, r = min(rr, R - 1);
    const long long pt = r / B;
    const int b = r - (int)pt * B;
    const bool ok = rr < R && col < H;
    const float* kd = a.kap + (a.k.at(pt) * B + b) * (long long)a.kw + 3 * H + cc;
    const long long oi = (a.o.at(pt) * B + b) * H + cc;
    const long long ca = (a.a.at(pt) * B + b) * H + cc;
    const bool mark = a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem;
    // coefficient row of the contraction operand of this lane
    const int rk = min(4 * q + (lane & 3), R - 1), ptk = rk / B;
    const float* kr = a.kap + (a.k.at(ptk) * B + (rk - ptk * B)) * (long long)a.kw;
    struct Ops {                              // requested one sub-step ahead (two gain nothing)
      floatx4 k[3][NCH];
      float kd, g;
    };
    auto request = [&](int j) {
      j = min(j, sw.n - 1);
      Ops o;
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
          const int k = 64 * c + 4 * (lane >> 2);
          o.k[g][c] = k < H ? ldg4(kr - j * dK + g * H + k) : zero4();
        }
      o.kd = kd[-j * dK];
      o.g = a.g ? a.g[oi - j * dO] : 0.f;
      return o;
    };
    Ops next = request(0);
    __syncthreads();
    float state = ws[0][row][cc];

    for (int j = 0; j < sw.n; ++j) {
      const int mode = j == 0 ? a.mode : j == sw.n - 1 ? sw.last : sw.mid, buf = j & 1;
      floatx4 op[3][NCH];
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(
            &ws[buf][(lane & 3)][64 * c + 4 * (lane >> 2)]);
#pragma unroll
        for (int g = 0; g < 3; ++g) op[g][c] = next.k[g][c] * v;
      }
      const float kdv = next.kd, gv = next.g;
      const float cur = mode == STEP_RESID ? a.w[oi - j * dO] : 0.f;
      next = request(j + 1);
      floatx4 acc[1][3][1];
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[0][g][0] = zero4();
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        quad_mma<1, 3, 1>(acc, [&](int, int g) { return op[g][c]; },
                           [&](int g) -> const float (&)[16] { return w[g][c]; });
      const float dot = quad_fold(acc[0][0][0] + acc[0][1][0] + acc[0][2][0]);
      const float wn = kdv * state + dot;
      if (mode == STEP_RELAX) {
        state = wn + gv;
        if (ok) a.w[oi - j * dO] = state;
      } else {  // STEP_RESID
        const float res = cur - wn - gv;
        if (ok) {
          a.gc[ca] = -res;
          a.wc[ca] = mark ? -res : 0.f;     // zero guess; -r at the marked points
          nrm += (double)res * (double)res;
        }
      }
      if (j + 1 < sw.n && col < H) ws[buf ^ 1][row][col] = state;
      if (j + 1 < sw.n) __syncthreads();
    }
  }
  if (a.norm && (a.mode == STEP_RESID || sw.last == STEP_RESID)) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nrm += __shfl_down(nrm, off, 64);
    if (lane == 0) atomicAdd(a.norm, nrm);
  }
}

// One timing record per epilogue mode of the sweep, each standing for the sub-steps of that mode.
template <class Launch>
static hipError_t record_sweep(int kind, long long R, int H, double bytes, int n, int first, int mid,
                               int last, hipStream_t s, Launch launch) {
  int modes[3], counts[3], nm = 0;
  auto add = [&](int mode, int count) {
    if (count <= 0) return;
    for (int i = 0; i < nm; ++i)
      if (modes[i] == mode) {
        counts[i] += count;
        return;
      }
    modes[nm] = mode;
    counts[nm++] = count;
  };
  add(first, 1);
  add(mid, n - 2);
  if (n > 1) add(last, 1);
  for (int i = 0; i < nm; ++i) prof_begin(kind, s, R, modes[i]);
  launch();
  const hipError_t err = hipGetLastError();
  for (int i = nm - 1; i >= 0; --i)
    prof_end(kind, 6.0 * (double)R * H * H * counts[i], bytes * (double)R * H * counts[i], s,
             counts[i], (double)counts[i] / n);
  return err;
}

#define MG_SWEEP_LAUNCH(KERNEL)                                                              \
  const int R = a.nk * a.B, quads = (R + 3) / 4;                                             \
  const dim3 grid((unsigned)std::min(quads, SWP_MAXWG)), block(64 * ((a.H + 15) / 16));      \
  auto launch = [&] {                                                                        \
    if (a.H <= 64)                                                                           \
      hipLaunchKernelGGL(KERNEL<1>, grid, block, 0, s, a, SweepSteps{n, mid, last, quads, pstep}); \
    else                                                                                     \
      hipLaunchKernelGGL(KERNEL<2>, grid, block, 0, s, a, SweepSteps{n, mid, last, quads, pstep}); \
  };

hipError_t launch_phi_sweep(const PhiArgs& a, int n, int mid, int last, long long pstep,
                            hipStream_t s) {
  if (a.nk <= 0 || n <= 0) return hipSuccess;
  if (a.H > SWEEP_MAX_H || a.bf16 == 1) return hipErrorInvalidValue;
  MG_SWEEP_LAUNCH(phi_sweep_kernel)
  return record_sweep(R <= 64 ? 4 : 0, R, a.H, 20.0, n, a.mode, mid, last, s, launch);
}

hipError_t launch_adj_sweep(const AdjArgs& a, int n, int mid, int last, hipStream_t s) {
  if (a.nk <= 0 || n <= 0) return hipSuccess;
  if (a.H > SWEEP_MAX_H || a.bf16 == 1) return hipErrorInvalidValue;
  const long long pstep = 0;
  MG_SWEEP_LAUNCH(adj_sweep_kernel)
  return record_sweep(R <= 64 ? 5 : 1, R, a.H, 28.0, n, a.mode, mid, last, s, launch);
}
#undef MG_SWEEP_LAUNCH

}  // namespace mg

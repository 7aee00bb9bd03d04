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
// api.hip).  Where the workgroups would have three quads or more one after the other, they take sixteen
// rows at a time through v_mfma_f32_16x16x4_f32 instead (phi_sweep_kernel16, adj_sweep_kernel16): the
// weights are held the same way, the sums need no adding up over lanes, and the latency of a sub-step is
// paid for sixteen rows.  The serial solves of these layers (one interval, N sub-steps) are such sweeps too, on
// the quad kernels up to 2048 rows; their state then travels through LDS instead of memory.  Workgroups loop
// over quads of rows, so that the weights are loaded once per workgroup.
#include <algorithm>
#include <type_traits>

#include "phi_elem.h"
#include "quad.h"

namespace mg {

constexpr int SWP_LD = SWEEP_MAX_H + 16;     // row stride of the state in LDS: 16 (mod 64 banks), so
                                             // that the four rows of a read fall on different banks
constexpr int SWP_LD16 = SWEEP_MAX_H + 4;    // sixteen rows: 4 (mod 64 banks)
constexpr int SWP_MAXWG = 256;               // one workgroup per CU (registers)

struct SweepSteps {
  int n, mid, last, blocks;                  // blocks of rows
  long long pstep;
  const float* coarse;                       // not null: points of the coarse level to take over first
};

// The correction at the coarse points rides on the sweep that starts from them: interval i starts from
// point i of the coarse level and leaves it at its point of this level (the last interval the last point
// too, from which no interval starts).  Adjoint: w + e, interval i starts from point i + 1, and the first one
// corrects point 0.  Training call without the six launches: 64 x 2 x 32 columns, two levels, three cycles 257 ->
// 254 us; two layers of 128 x 100 x 100, twelve launches, 1050 -> 1041.
__device__ inline floatx4 take_over(const PhiArgs& a, const SweepSteps& sw, long long r, bool ok, int c) {
  const int B = a.B;
  const long long pt = r / B, b = r - pt * B;
  auto level = [&](long long q) { return a.u + (a.in.at(q) * B + b) * a.H + c; };
  if (pt == a.nk - 1 && ok)
    *reinterpret_cast<floatx4*>(level(pt + 1)) = ldg4(sw.coarse + (r + B) * a.H + c);
  if (pt == 0) return ldg4(level(0));
  const floatx4 v = ldg4(sw.coarse + r * a.H + c);
  if (ok) *reinterpret_cast<floatx4*>(level(pt)) = v;
  return v;
}
__device__ inline float corrected(const AdjArgs& a, const SweepSteps& sw, long long r, bool ok, int c) {
  const int B = a.B;
  const long long pt = r / B, b = r - pt * B;
  const long long step = a.in.at(1) - a.in.at(0);
  auto level = [&](long long q) { return a.w + ((a.in.at(0) + (q - 1) * step) * B + b) * a.H + c; };
  if (pt == 0 && ok) *level(0) += sw.coarse[r * a.H + c];
  float v = *level(pt + 1);
  if (pt < a.nk - 1) {
    v += sw.coarse[(r + B) * a.H + c];
    if (ok) *level(pt + 1) = v;
  }
  return v;
}

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

// The same for v_mfma_f32_16x16x4_f32: column as above, k = 16 s + 4 (lane / 16) + 0..3.
template <int NKB, class At>
__device__ inline void sweep_weights16(floatx4 (&w)[3][NKB], int H, At at) {
  const int lane = threadIdx.x & 63;
  const int j = min((int)(threadIdx.x >> 6) * 16 + (lane & 15), H - 1);
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int s = 0; s < NKB; ++s) {
      const int k = 16 * s + 4 * (lane >> 4);
      w[g][s] = k < H ? ldg4(at(g, j, k)) : zero4();
    }
}
// Three sums of a wave's 16 x 16 block over K, one gate after the other, every fourth k apart (the chains
// of additions are as long as those of a quad: with two sums per gate the states were 1 %, the adjoint 4 %
// further from 64 bits): lane l holds rows 4 (l / 16) + 0..3 of column l % 16.  a(g, s): operand of gate
// g, k = 16 s + 4 (l / 16) + 0..3 of row l % 16.
template <int NKB, class GetA>
__device__ inline void sweep_mma16(floatx4 (&sum)[3], const floatx4 (&w)[3][NKB], int H, GetA a) {
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    floatx4 acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = zero4();
#pragma unroll
    for (int s = 0; s < NKB; ++s) {
      if (16 * s >= H) break;
      const floatx4 v = a(g, s);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], w[g][s][e], acc[e], 0, 0, 0);
    }
    sum[g] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
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

  for (int q = blockIdx.x; q < sw.blocks; q += gridDim.x) {
    __syncthreads();                          // the last block's reads of the state are done
    const int h4 = H / 4;
    for (int e = tid; e < 4 * h4; e += blockDim.x) {
      const int r = min(4 * q + e / h4, R - 1), pt = r / B;
      *reinterpret_cast<floatx4*>(&hs[0][e / h4][e % h4 * 4]) =
          sw.coarse ? take_over(a, sw, r, 4 * q + e / h4 < R, e % h4 * 4)
                    : ldg4(a.u_in + (a.in.at(pt) * B + (r - pt * B)) * H + e % h4 * 4);
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

// Sixteen rows of a workgroup at a time.
template <int NCH>
__global__ __launch_bounds__(256 * NCH, 2) void phi_sweep_kernel16(PhiArgs a, SweepSteps sw) {
  __shared__ __attribute__((aligned(16))) float hs[2][16][SWP_LD16];
  const int H = a.H, B = a.B, R = a.nk * B;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row0 = 4 * (lane >> 4), col = wv * 16 + (lane & 15), cc = min(col, H - 1);
  floatx4 w[3][4 * NCH];
  sweep_weights16<4 * NCH>(w, H, [&](int g, int j, int k) {
    return (const float*)a.U + ((long long)g * H + j) * H + k;
  });
  const PhiBias bh = phi_bias_load(a, cc);
  const bool implicit = a.propagator == MGRIT_PROP_IMPLICIT;
  for (int e = tid; e < 2 * 16 * SWP_LD16; e += blockDim.x) (&hs[0][0][0])[e] = 0.f;
  double nrm = 0.0;

  for (int q = blockIdx.x; q < sw.blocks; q += gridDim.x) {
    __syncthreads();                          // the last block's reads of the state are done
    const int h4 = H / 4;
    for (int e = tid; e < 16 * h4; e += blockDim.x) {
      const int r = min(16 * q + e / h4, R - 1), pt = r / B;
      *reinterpret_cast<floatx4*>(&hs[0][e / h4][e % h4 * 4]) =
          sw.coarse ? take_over(a, sw, r, 16 * q + e / h4 < R, e % h4 * 4)
                    : ldg4(a.u_in + (a.in.at(pt) * B + (r - pt * B)) * H + e % h4 * 4);
    }
    // output elements of this lane (rows beyond the launch repeat its last row and store nothing):
    // rows of the arrays
    int ro[4], rp[4], ra[4];
    bool ok[4], mark[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int rr = 16 * q + row0 + v, r = min(rr, R - 1);
      const int pt = r / B, b = r - pt * B;
      ok[v] = rr < R && col < H;
      rp[v] = (int)(a.p.at(pt) * B) + b;
      ro[v] = (int)(a.o.at(pt) * B) + b;
      ra[v] = (int)(a.a.at(pt) * B) + b;
      mark[v] = a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem;
    }
    // operands of a sub-step that no sub-step produces, requested one ahead
    struct Ops {
      float pr[4], pz[4], pn[4], g[4];
    };
    auto p_at = [&](int v, int j) {
      return a.P + ((long long)rp[v] + j * sw.pstep * B) * (3LL * H) + cc;
    };
    auto o_at = [&](int v, int j) { return ((long long)ro[v] + (long long)j * B) * H + cc; };
    auto request = [&](int j) {
      j = min(j, sw.n - 1);
      Ops o;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float* p = p_at(v, j);
        o.pr[v] = p[0];
        o.pz[v] = p[H];
        o.pn[v] = p[2 * H];
        o.g[v] = a.g ? a.g[o_at(v, j)] : 0.f;
      }
      return o;
    };
    Ops next = request(0);
    __syncthreads();
    float state[4], half[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      state[v] = hs[0][row0 + v][cc];
      half[v] = 0.f;
    }

    // one sub-step; the code of each mode by itself, so that only its operands are in registers
    auto sub_step = [&](auto m, int j) {
      constexpr int MODE = decltype(m)::value;
      const int buf = j & 1;
      // (addresses are formed again in every sub-step rather than kept)
#pragma unroll
      for (int v = 0; v < 4; ++v) asm volatile("" : "+v"(rp[v]), "+v"(ro[v]), "+v"(ra[v]));
      PhiEpiIn e[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        e[v] = PhiEpiIn{next.pr[v], next.pz[v], next.pn[v], state[v], next.g[v], 0.f, 0.f, 0.f, 0.f, 0.f, half[v]};
      next = request(j + 1);
      // what only the first or last sub-step needs: behind the contraction
      if (MODE == STEP_RESID) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          e[v].cur = a.u[o_at(v, j)];
          if (a.resid_adds && j == 0) e[v].prep = a.gc[(long long)ra[v] * H + cc];
        }
      }
      if (MODE == STEP_RELAX_RHS || MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float* p2 = p_at(v, j) + a.dp2;
          e[v].pr2 = p2[0];
          e[v].pz2 = p2[H];
          e[v].pn2 = p2[2 * H];
          if (MODE == STEP_RELAX_RHS) e[v].cur2 = a.u[o_at(v, j) + a.do2];
        }
      }
      floatx4 sum[3];
      sweep_mma16<4 * NCH>(sum, w, H, [&](int, int s) {
        return *reinterpret_cast<const floatx4*>(&hs[buf][lane & 15][16 * s + 4 * (lane >> 4)]);
      });
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const long long o = o_at(v, j), ca = (long long)ra[v] * H + cc;
        const PhiOut x =
            phi_elem<MODE>(a.gamma, implicit, sum[0][v], sum[1][v], sum[2][v], e[v], bh, a.gamma2);
        if (MODE == STEP_RELAX || MODE == STEP_RELAX_RHS || MODE == STEP_RELAX_CK) {
          state[v] = x.v0;
          if (ok[v]) a.u[o] = x.v0;
        }
        if (MODE == STEP_RELAX_RHS) {
          half[v] = x.v1;                     // completed by the residual, in this sweep or later
          if (ok[v]) a.gc[ca] = x.v1;
        }
        if (MODE == STEP_RESID && ok[v]) {
          a.gc[ca] = a.resid_adds ? e[v].prep + x.v0 : x.v0;
          a.uc[ca] = mark[v] ? x.v1 + x.v0 : x.v1;       // cur - r at the marked points
          nrm += (double)x.v0 * (double)x.v0;
        }
        if (MODE == STEP_RELAX_KAPPA || MODE == STEP_RELAX_KAPPA2) {
          state[v] = x.v5;
          if (ok[v]) {
            a.u[o] = x.v5;
            float* kp = a.uc + ((long long)ro[v] + (long long)j * B) * a.kappa_width + cc;
            kp[0] = x.v0;
            kp[H] = x.v1;
            kp[2 * H] = x.v2;
            kp[3 * H] = x.v3;
            if (a.kappa_width >= 5 * H) kp[4 * H] = x.v4;
          }
        }
        if ((MODE == STEP_RELAX_KAPPA2 || MODE == STEP_RELAX_CK) && ok[v]) {
          float* kc = a.gc + (ca - cc) * 4 + cc;
          kc[0] = x.c0;
          kc[H] = x.c1;
          kc[2 * H] = x.c2;
          kc[3 * H] = x.c3;
        }
        if (j + 1 < sw.n && col < H) hs[buf ^ 1][row0 + v][col] = state[v];
      }
    };
    for (int j = 0; j < sw.n; ++j) {
      const int mode = j == 0 ? a.mode : j == sw.n - 1 ? sw.last : sw.mid;
      if (mode == STEP_RELAX) sub_step(std::integral_constant<int, STEP_RELAX>(), j);
      else if (mode == STEP_RELAX_RHS) sub_step(std::integral_constant<int, STEP_RELAX_RHS>(), j);
      else if (mode == STEP_RESID) sub_step(std::integral_constant<int, STEP_RESID>(), j);
      else if (mode == STEP_RELAX_CK) sub_step(std::integral_constant<int, STEP_RELAX_CK>(), j);
      else if (mode == STEP_RELAX_KAPPA2) sub_step(std::integral_constant<int, STEP_RELAX_KAPPA2>(), j);
      else sub_step(std::integral_constant<int, STEP_RELAX_KAPPA>(), j);
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

  for (int q = blockIdx.x; q < sw.blocks; q += gridDim.x) {
    __syncthreads();                          // the last block's reads of the state are done
    const int h4 = H / 4;
    for (int e = tid; e < 4 * h4; e += blockDim.x) {
      const int r = min(4 * q + e / h4, R - 1), pt = r / B;
      floatx4 v;
      if (sw.coarse) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          v[c] = corrected(a, sw, r, 4 * q + e / h4 < R, e % h4 * 4 + c);
      } else {
        v = ldg4(a.w_in + (a.in.at(pt) * B + (r - pt * B)) * H + e % h4 * 4);
      }
      *reinterpret_cast<floatx4*>(&ws[0][e / h4][e % h4 * 4]) = v;
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

// Sixteen rows of a workgroup at a time.  The products of the state with the coefficients of the next
// sub-step are made by the lane that makes an element and go to the waves through LDS, three vectors
// instead of one; in adj_sweep_kernel every wave loads the coefficients of all K.
template <int NCH>
__global__ __launch_bounds__(256 * NCH, 2) void adj_sweep_kernel16(AdjArgs a, SweepSteps sw) {
  __shared__ __attribute__((aligned(16))) float ps[2][3][16][SWP_LD16];
  const int H = a.H, B = a.B, R = a.nk * B;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int row0 = 4 * (lane >> 4), col = wv * 16 + (lane & 15), cc = min(col, H - 1);
  floatx4 w[3][4 * NCH];
  sweep_weights16<4 * NCH>(w, H, [&](int g, int j, int k) {
    return (const float*)a.UT + (long long)j * 3 * H + g * H + k;
  });
  for (int e = tid; e < 2 * 3 * 16 * SWP_LD16; e += blockDim.x) (&ps[0][0][0][0])[e] = 0.f;
  double nrm = 0.0;

  for (int q = blockIdx.x; q < sw.blocks; q += gridDim.x) {
    int ri[4], rk[4], ro[4], ra[4];
    bool ok[4], mark[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int rr = 16 * q + row0 + v, r = min(rr, R - 1);
      const int pt = r / B, b = r - pt * B;
      ok[v] = rr < R && col < H;
      ri[v] = (int)(a.in.at(pt) * B) + b;
      rk[v] = (int)(a.k.at(pt) * B) + b;
      ro[v] = (int)(a.o.at(pt) * B) + b;
      ra[v] = (int)(a.a.at(pt) * B) + b;
      mark[v] = a.ff_cf > 0 && a.a.at(pt) % a.ff_cf == a.ff_rem;
    }
    auto o_at = [&](int v, int j) { return ((long long)ro[v] - (long long)j * B) * H + cc; };
    struct Ops {                              // of sub-step j: three coefficients, k_d, right-hand side
      float k[3][4], kd[4], g[4];
    };
    auto request = [&](int j) {
      j = min(j, sw.n - 1);
      Ops o;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float* kr = a.kap + ((long long)rk[v] - (long long)j * B) * a.kw + cc;
#pragma unroll
        for (int g = 0; g < 3; ++g) o.k[g][v] = kr[g * H];
        o.kd[v] = kr[3 * H];
        o.g[v] = a.g ? a.g[o_at(v, j)] : 0.f;
      }
      return o;
    };
    Ops ops = request(0);
    float state[4];
#pragma unroll
    for (int v = 0; v < 4; ++v)
      state[v] = sw.coarse ? corrected(a, sw, min(16 * q + row0 + v, R - 1), ok[v], cc)
                           : a.w_in[(long long)ri[v] * H + cc];
    __syncthreads();                          // the last block's reads of the products are done
    for (int j = 0; j < sw.n; ++j) {
      const int mode = j == 0 ? a.mode : j == sw.n - 1 ? sw.last : sw.mid, buf = j & 1;
      if (col < H) {
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
          for (int v = 0; v < 4; ++v) ps[buf][g][row0 + v][col] = ops.k[g][v] * state[v];
      }
      float kd[4], gv[4], cur[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        kd[v] = ops.kd[v];
        gv[v] = ops.g[v];
        if (mode == STEP_RESID) cur[v] = a.w[o_at(v, j)];
      }
      __syncthreads();
      ops = request(j + 1);
      floatx4 sum[3];
      sweep_mma16<4 * NCH>(sum, w, H, [&](int g, int s) {
        return *reinterpret_cast<const floatx4*>(&ps[buf][g][lane & 15][16 * s + 4 * (lane >> 4)]);
      });
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float wn = kd[v] * state[v] + (sum[0][v] + sum[1][v] + sum[2][v]);
        if (mode == STEP_RELAX) {
          state[v] = wn + gv[v];
          if (ok[v]) a.w[o_at(v, j)] = state[v];
        } else {  // STEP_RESID
          const float res = cur[v] - wn - gv[v];
          if (ok[v]) {
            const long long ca = (long long)ra[v] * H + cc;
            a.gc[ca] = -res;
            a.wc[ca] = mark[v] ? -res : 0.f;     // zero guess; -r at the marked points
            nrm += (double)res * (double)res;
          }
        }
      }
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

// Sixteen rows of a workgroup at a time from the third round of quads on.  Forward / adjoint launches of a
// level, cf 4, us, quads : sixteen rows: 1024 rows x 100 columns 96 / 13 : 104 / 18, 2048 115 / 18 : 114 / 20,
// 2560 128 / 24 : 122 / 20, 3200 148 / 28 : 127 / 20, 4096 162 / 29 : 140 / 22, 8192 232 / 49 : 193 / 33; 3200 x 32
// 92 / 16 : 78 / 13, 8192 x 128 236 / 62 : 211 / 38; cf 8: 2560 x 100 179 / 41 : 169 / 34, 3200 218 / 52 : 174 /
// 35, 8192 382 / 100 : 293 / 62.
static bool sweep_wide(int R) { return R > 2 * 4 * SWP_MAXWG; }
#define MG_SWEEP_LAUNCH(QUADS1, QUADS2, ROWS1, ROWS2)                                         \
  const int R = a.nk * a.B;                                                                   \
  const bool wide = sweep_wide(R);                                                            \
  const int blocks = wide ? (R + 15) / 16 : (R + 3) / 4;                                      \
  const dim3 grid((unsigned)std::min(blocks, SWP_MAXWG)), block(64 * ((a.H + 15) / 16));      \
  const SweepSteps sw{n, mid, last, blocks, pstep, coarse};                                   \
  auto launch = [&] {                                                                         \
    if (a.H <= 64 && wide) hipLaunchKernelGGL((ROWS1), grid, block, 0, s, a, sw);             \
    else if (a.H <= 64) hipLaunchKernelGGL((QUADS1), grid, block, 0, s, a, sw);               \
    else if (wide) hipLaunchKernelGGL((ROWS2), grid, block, 0, s, a, sw);                     \
    else hipLaunchKernelGGL((QUADS2), grid, block, 0, s, a, sw);                              \
  };

hipError_t launch_phi_sweep(const PhiArgs& a, int n, int mid, int last, long long pstep,
                            hipStream_t s, const float* coarse) {
  if (a.nk <= 0 || n <= 0) return hipSuccess;
  if (a.H > SWEEP_MAX_H || a.bf16 == 1) return hipErrorInvalidValue;
  MG_SWEEP_LAUNCH(phi_sweep_kernel<1>, phi_sweep_kernel<2>, phi_sweep_kernel16<1>, phi_sweep_kernel16<2>)
  return record_sweep(R <= 64 ? 4 : 0, R, a.H, 20.0, n, a.mode, mid, last, s, launch);
}

hipError_t launch_adj_sweep(const AdjArgs& a, int n, int mid, int last, hipStream_t s,
                            const float* coarse) {
  if (a.nk <= 0 || n <= 0) return hipSuccess;
  if (a.H > SWEEP_MAX_H || a.bf16 == 1) return hipErrorInvalidValue;
  const long long pstep = 0;
  MG_SWEEP_LAUNCH(adj_sweep_kernel<1>, adj_sweep_kernel<2>, adj_sweep_kernel16<1>, adj_sweep_kernel16<2>)
  return record_sweep(R <= 64 ? 5 : 1, R, a.H, 28.0, n, a.mode, mid, last, s, launch);
}
#undef MG_SWEEP_LAUNCH

}  // namespace mg

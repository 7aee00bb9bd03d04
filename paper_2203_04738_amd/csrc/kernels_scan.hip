// Serial propagation of a few rows as ONE launch.
//
// A chain of dependent launches costs 4.7 us (forward) to 7.3 us (adjoint) per step at 32 rows x
// 512, of which the arithmetic is a tenth: the rest is the launch, reading the weights again, and
// round trips to L2.  Here the workgroups stay resident for all N steps.  Workgroup (cg, rb) owns
// 16 hidden columns (cg) of RB x 4 rows (rb) and keeps its share of the recurrent weights in
// registers for the whole solve; what travels between workgroups is the state alone.
//
// Exchange.  Every element of the state array is written exactly once, so the data is its own
// flag: the rows a solve will write are first filled with a NaN bit pattern that no step stores
// (SENTINEL), and a workgroup that needs a row reads it until no element of it shows the pattern.
// One trip to the memory side and back per step, no barrier between workgroups, no ordering
// between different words (each word carries its own validity).  Stores and polls use agent scope
// (sc1): visible across the XCDs whichever XCD a workgroup runs on.  Measured for the exchange
// alone: 1.1-1.6 us per step among 16-32 workgroups of 512 columns, 1.7-1.9 us among 32-64 of
// 1024, 3-4 us among 256 (many small column groups): hence 16 columns per workgroup and as many
// row blocks as the rows give.
//
// Contraction in quads of rows (see quad.h): each workgroup needs few rows, where a 16-row MFMA would
// idle on three quarters of its rows.
// Waves split K as well; the groups are added by lane swaps, the waves through LDS (one barrier
// per step, two buffers).
//
// Shapes whose row blocks each fit one XCD run there and exchange through its L2 (kernels_scan_xcd.hip;
// the rule and what both measure are at scan_shape_xcd); this file has the form for the others, what both
// share on the host, and the launch that takes over what neither could start.
//
// Of a step of 3 x 500, 2.0 us, about 1.3 us are the exchange, 0.3 us MFMAs, the rest LDS sums and gates.
// us per step of the shapes that are left to this form: 8 x 1024 3.1 (adjoint, gradients included, 4.3; on
// bf16 weights 3.9), 3 x 1000 2.7, LSTM 8 x 1000 3.4.
//
// Residency.  Each workgroup keeps its columns for the whole solve, which needs all of them resident
// at once: each announces itself and waits, with a time limit, until all have arrived before it takes
// the first step (the grid is limited to one workgroup per CU).  If the limit passes (other work holds
// CUs: two more solves on other streams, say), every workgroup leaves, and the launch behind takes the
// solve over, which returns at once otherwise.  There a workgroup takes one (step, columns, rows) item
// after the other from a counter.  An item waits only for items with smaller numbers, and those are
// held by workgroups that run, so any number of resident workgroups gets through.  The weights are
// loaded again for every item.  The arithmetic of an element is the same code on the same operands, so
// the results do not depend on which launch computes them, bit for bit; an element both have computed
// is written twice with one value.  Measured with the takeover forced (chain of step launches : this :
// all resident in this form, us per step): 8 x 1024 on bf16 weights, contracted in fp32, 5.9 : 8.5 : 3.1, 64 x
// 1024 17.6 : 12.4 : 10.0, 3 x 500 4.1 : 3.6 : 2.1, 16 x 256 4.0 : 3.8 : 1.6, LSTM 32 x 512 5.2 : 6.7 : 3.0;
// three streams at once, ms: bptt of 256 x 32 x 1024 24.0 : 23.4, scans of 256 x 64 x 1024 9.8 : 11.5, LSTM 512
// x 32 x 512 6.3 : 9.2.  Behind the form inside the XCDs, one XCD allowed and no wait (chain : this : inside the
// XCDs): 100 x 512 13.3 : 12.4 : 3.5, 100 x 1000 26.0 : 24.3 : 9.9, LSTM 100 x 200 10.7 : 5.4 : 1.8, ODE 100 x
// 512 7.3 : 6.9 : 1.8, back-propagation 100 x 512 20.3 : 13.6 : 5.3 and 100 x 1000 41.9 : 50.2 : 22.5; on terms
// (this : inside) 100 x 512 10.6 : 2.5, 100 x 1000 16.7 : 4.5, 1 x 1024 2.4 : 1.4.
#include <atomic>
#include <cstdlib>

#include "scan_exchange.h"

namespace mg {

// next item of a solve whose workgroups are not all resident
__device__ inline long long ctl_take(int* ctl) {
  return (long long)__hip_atomic_fetch_add((unsigned long long*)(ctl + 2), 1ULL, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
}
// One element of a state row that another workgroup may still be writing.
__device__ inline float scan_own(const float* p) {
  unsigned b = SENTINEL;
  for (int polls = 0; b == SENTINEL && polls < SCAN_MAX_POLLS; ++polls)
    b = __hip_atomic_load((const unsigned*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __uint_as_float(b);
}
// Weights of gate g, chunk c: column j, k = k0 + 64 c + 0..15 (zero beyond H, a multiple of 4).
template <int KIND, int NG, int NCH, class WT>
__device__ inline void scan_weights(float (&w)[NG][NCH][16], const WT* Wt, int H, int j, int k0) {
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + 64 * c + 4 * q;
        const int kc = min(k, H - 4);
        const WT* p = Wt + (KIND == SCAN_ADJOINT ? (long long)j * 3 * H + g * H + kc
                                                 : ((long long)g * H + j) * H + kc);
        const floatx4 v = k < H ? ldg4w(p) : zero4();
#pragma unroll
        for (int e = 0; e < 4; ++e) w[g][c][4 * q + e] = v[e];
      }
}
// NCH: chunks of 64 k per wave; RB: groups of four rows per workgroup.  Registers: NG 16 NCH
// weights; one workgroup per CU is planned for (two waves per SIMD at eight waves).
// ITEMS: the workgroup takes (step, unit) items from the counter until none are left; otherwise it
// takes every step of the unit it was launched as, once all workgroups of the solve are resident, and
// leaves what remains to the launch with ITEMS behind it if they are not (see the top of the file).
// TERMS (items behind an xcd_scan_kernel on terms): its contraction, for the same bits.
template <int KIND, int NCH, int RB, class WT, bool ITEMS, bool TERMS>
__global__ __launch_bounds__(64 * SCAN_MAXW, 2) void scan_kernel(ScanArgs a, int nrb, int xcd_quads) {
  constexpr int NG = ScanGates<KIND>::value;
  constexpr bool ADJ = KIND == SCAN_ADJOINT;
  constexpr int NS = ADJ ? 1 : NG;                    // sums an output needs
  constexpr int NL = RB * NCH;
  constexpr int NP = NG == 1 ? 2 : 1;                 // sums per gate and row group
  __shared__ float part[2][SCAN_MAXW][RB][NS][64];
  __shared__ int stop[2];
  __shared__ long long item;
  __shared__ uintx4 frag[TERMS ? SCAN_MAXW : 1][TERMS ? 128 : 1];   // 64 k of a quad in terms, per wave
  const int H = a.H, B = a.B, N = a.N;
  const int W = KIND == SCAN_LSTM ? 2 * H : H;        // state row
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
  const int nwg = gridDim.x;
  const int kw0 = wv * 64 * NCH;                      // K slice of this wave
  const bool epi = wv < RB;                           // wave r finishes row group r
  // points: forward step i = 0..N-1 goes from point i to i + 1, adjoint from N - i to N - i - 1
  const long long BW = (long long)B * W;
  auto in_pt = [&](int i) { return (long long)(ADJ ? N - i : i); };
  auto out_pt = [&](int i) { return (long long)(ADJ ? N - i - 1 : i + 1); };

  long long mine = 0;                                 // thread 0: the item after the current one
  int unit = blockIdx.x, first = 0, last = N;
  int done = 0;                                       // row quads before this one are solved
  if (ITEMS) {
    // (the workspace is left as if the rows had gone through the output array alone: its bytes do not
    // tell who has solved)
    for (long long q = (long long)blockIdx.x * blockDim.x + tid; q < a.ring4;
         q += (long long)gridDim.x * blockDim.x)
      ((uintx4*)a.ring)[q] = uintx4{0, 0, 0, 0};
    // done: all were resident, or the XCDs have taken every row block
    if (a.ring) {
      if (ctl_load(a.ctl + CTL_ABORT) == 0)
        done = xcd_groups((unsigned)ctl_load(a.ctl + CTL_WORD)) * xcd_quads;
      if (done * 4 >= B) return;
    } else if (ctl_load(a.ctl + 1) == 0) {
      return;
    }
    if (tid == 0) mine = ctl_take(a.ctl);
  }
  if (tid < 2) stop[tid] = 0;

  do {
    if (ITEMS) {
      // one barrier between the items, which also keeps part apart: its readers are through
      if (tid == 0) item = mine;
      __syncthreads();
      const long long t = item;
      if (t >= (long long)N * nwg) return;
      if (tid == 0) mine = ctl_take(a.ctl);           // (arrives behind this item's work)
      first = (int)(t / nwg);
      unit = (int)(t % nwg);
      last = first + 1;
    }
    const int rb = unit % nrb, cg = unit / nrb;
    if (ITEMS && (rb + 1) * RB <= done) {
      __syncthreads();                                 // (every thread has read item)
      continue;
    }
    const int r0 = rb * RB * 4, j0 = cg * SCAN_CP;
    // weights: column j0 + lane % 16, k = kw0 + 64 c + 16 (lane / 16) + 0..15 (zero beyond H; columns
    // beyond H repeat the last one and are never stored)
    float w[NG][NCH][16];
    bf16x8 wt[NG][NCH * 2];
    bool plain = false;                               // TERMS: contract in fp32 all the same (per wave)
    if constexpr (TERMS) {
      const int j = min(j0 + (lane & 15), H - 1);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            wt[g][2 * c + b] = term_weights((const bf16_t*)a.Wt + ((long long)g * H + j) * H,
                                            kw0 + 64 * c + 32 * b + 8 * (lane >> 4), H);
      frag[wv][(lane >> 5) * 64 + (lane >> 3 & 3) * 16 + 12 + (lane & 3)] = uintx4{0, 0, 0, 0};
      plain = term_weights_infinite(wt);
    } else {
      scan_weights<KIND>(w, (const WT*)a.Wt, H, min(j0 + (lane & 15), H - 1), kw0 + 16 * (lane >> 4));
    }
    // polled operand: rows r0 + 4 r + lane % 4, k = kw0 + 64 c + 4 (lane / 4) + 0..3; lanes beyond
    // the rows or columns read a valid place and contribute nothing
    unsigned off[NL];
    bool live[NCH];
    unsigned koff[ADJ ? RB : 1];
    int kk[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int k = kw0 + 64 * c + 4 * (lane >> 2);
      live[c] = k < H;
      kk[c] = min(k, H - 4);
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int row = min(r0 + 4 * r + (lane & 3), B - 1);
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        off[r * NCH + c] = ((unsigned)row * W + kk[c]) * 4u;
      if (ADJ) koff[r] = (unsigned)row * a.kw;
    }
    // output element of this lane
    const int orow = r0 + 4 * wv + quad_row(lane), oj = j0 + (lane & 15);
    const bool ok = epi && orow < B && oj < H;
    const int er = min(orow, B - 1), ej = min(oj, H - 1);
    const long long eo = (long long)er * W + ej;
    float bias[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g)
      bias[g] = (KIND == SCAN_GRU || KIND == SCAN_LSTM) ? a.b_h[g * H + ej] : 0.f;

    if (!ITEMS) {   // all workgroups of the solve are resident before the first step
      __syncthreads();
      if (tid == 0) {
        __hip_atomic_fetch_add(a.ctl, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const long long t0 = ticks();
        while (true) {
          bool leave = ctl_load(a.ctl + 1) != 0;
          if (!leave && ticks() - t0 >= a.wait_ticks) {
            __hip_atomic_store(a.ctl + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            leave = true;
          }
          if (leave) {
            stop[0] = 1;
            break;
          }
          if (ctl_load(a.ctl) >= nwg) break;
          __builtin_amdgcn_s_sleep(2);
        }
      }
      __syncthreads();
      if (stop[0]) return;
      __syncthreads();
    }

    // operands that do not depend on the state, requested one step ahead
    float ep[NG], eg = 0.f, egc = 0.f, ekd = 0.f;
    floatx4 kv[ADJ ? RB : 1][ADJ ? NG : 1][NCH];
    auto request = [&](int i) {
      if (ADJ) {
        const float* kr = a.kap + in_pt(i) * B * a.kw;
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int c = 0; c < NCH; ++c)
              kv[ADJ ? r : 0][ADJ ? g : 0][c] = ldg4(kr + koff[ADJ ? r : 0] + g * H + kk[c]);
        if (epi) ekd = kr[(long long)er * a.kw + 3 * H + ej];
      } else if (epi) {
        const float* pr =
            a.P + (((long long)(i + 1) * a.pstep - 1) * B + er) * ((long long)NG * H) + ej;
#pragma unroll
        for (int g = 0; g < NG; ++g) ep[g] = pr[g * H];
      }
      if (epi && a.g) {
        eg = a.g[out_pt(i) * BW + eo];
        if (KIND == SCAN_LSTM) egc = a.g[out_pt(i) * BW + eo + H];
      }
    };
    request(first);
    float prev = 0.f, prevc = 0.f;                     // own state element of the input point
    if (epi) {
      const float* p = a.u + in_pt(first) * BW + eo;
      prev = first > 0 ? scan_own(p) : *p;
      if (KIND == SCAN_LSTM) prevc = first > 0 ? scan_own(p + H) : p[H];
    }

    for (int i = first; i < last; ++i) {
      const int buf = i & 1;
      uintx4 v[NL];
      const float* src = scan_uniform(a.u + in_pt(i) * BW);
      scan_load(v, src, off);
      if (i > 0) {
        int polls = 0;
        long long t0 = 0;
        while (true) {
          bool wait = false;
#pragma unroll
          for (int q = 0; q < NL; ++q)
            wait |= v[q][0] == SENTINEL || v[q][1] == SENTINEL || v[q][2] == SENTINEL ||
                    v[q][3] == SENTINEL;
          if (!__any(wait)) break;
          if ((++polls & 127) == 0) {
            bool leave;
            if (ITEMS) {
              leave = polls >= SCAN_MAX_POLLS;
            } else {
              if (t0 == 0) t0 = ticks();
              leave = ticks() - t0 > SCAN_STEP_TICKS;
              if (leave)
                __hip_atomic_store(a.ctl + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              leave |= ctl_load(a.ctl + 1) != 0;
            }
            if (leave) {
              stop[buf] = 1;
              break;
            }
          }
          scan_load(v, src, off);
        }
      }
      // operands of the contraction; those of the next step are requested as soon as these are
      // formed, so that they arrive behind the contraction and the exchange
      floatx4 op[NCH][RB][ADJ ? NG : 1];
#pragma unroll
      for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          const floatx4 h = __builtin_bit_cast(floatx4, v[r * NCH + c]);
#pragma unroll
          for (int g = 0; g < (ADJ ? NG : 1); ++g)
            op[c][r][g] = live[c] ? (ADJ ? kv[ADJ ? r : 0][g][c] * h : h) : zero4();
        }
      float cp[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) cp[g] = ep[g];
      const float cgv = eg, cgc = egc, ckd = ekd;
      if (i + 1 < last) request(i + 1);
      floatx4 acc[RB][NG][NP];
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
          for (int q = 0; q < NP; ++q) acc[r][g][q] = zero4();
      if constexpr (TERMS) {
        if (!plain) {
          // each wave sorts its rows into fragments through LDS of its own
          typedef unsigned u2 __attribute__((ext_vector_type(2)));
          u2* const put = (u2*)frag[wv] + ((lane >> 5) * 64 + (lane >> 3 & 3) * 16 + (lane & 3)) * 2 +
                           (lane >> 2 & 1);
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            floatx4 sum[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) sum[g] = zero4();
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
              StateTerms t[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) t[e] = state_terms(op[c][r][0][e]);
              auto lo = [](unsigned a0, unsigned a1) { return (a0 & 0xffffu) | (a1 << 16); };
              auto hi = [](unsigned a0, unsigned a1) { return (a0 >> 16) | (a1 & 0xffff0000u); };
              put[0] = u2{lo(t[0].t01, t[1].t01), lo(t[2].t01, t[3].t01)};
              put[8] = u2{hi(t[0].t01, t[1].t01), hi(t[2].t01, t[3].t01)};
              put[16] = u2{lo(t[0].t2, t[1].t2), lo(t[2].t2, t[3].t2)};
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
              const uintx4 f[2] = {frag[wv][lane], frag[wv][64 + lane]};
              __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
#pragma unroll
              for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int g = 0; g < NG; ++g) sum[g] = term_mma(f[b], wt[g][2 * c + b], sum[g]);
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) part[buf][wv][r][g][lane] = term_fold(sum[g]);
          }
        } else {                                       // (registers: a gate and a chunk at a time)
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            floatx4 sum[RB][1][1];
#pragma unroll
            for (int r = 0; r < RB; ++r) sum[r][0][0] = zero4();
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
              asm volatile("" ::: "memory");
              float w1[1][1][16];
              scan_weights<KIND>(w1, (const WT*)a.Wt + (long long)g * H * H, H, min(j0 + (lane & 15), H - 1),
                                 kw0 + 64 * c + 16 * (lane >> 4));
              quad_mma<RB, 1, 1>(sum, [&](int r, int) { return op[c][r][0]; },
                                 [&](int) -> const float (&)[16] { return w1[0][0]; });
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) part[buf][wv][r][g][lane] = quad_fold(sum[r][0][0]);
          }
        }
      } else {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
          quad_mma<RB, NG, NP>(acc, [&](int r, int g) { return op[c][r][ADJ ? g : 0]; },
                               [&](int g) -> const float (&)[16] { return w[g][c]; });
#pragma unroll
        for (int r = 0; r < RB; ++r) {
          floatx4 sum[NG];
#pragma unroll
          for (int g = 0; g < NG; ++g)
            sum[g] = NP > 1 ? acc[r][g][0] + acc[r][g][NP - 1] : acc[r][g][0];
          if (ADJ) {
            part[buf][wv][r][0][lane] = quad_fold(sum[0] + sum[NG > 1 ? 1 : 0] + sum[NG - 1]);
          } else {
#pragma unroll
            for (int g = 0; g < NG; ++g) part[buf][wv][r][ADJ ? 0 : g][lane] = quad_fold(sum[g]);
          }
        }
      }
      __syncthreads();
      const int stopped = stop[buf];
      if (epi) {
        // partial sums of all waves (every read in flight before the first addition)
        float s[NS], ps[NS][SCAN_MAXW];
#pragma unroll
        for (int g = 0; g < NS; ++g)
#pragma unroll
          for (int q = 0; q < SCAN_MAXW; ++q) ps[g][q] = part[buf][q < nw ? q : 0][wv][g][lane];
        if (stopped) return;
#pragma unroll
        for (int g = 0; g < NS; ++g) {
#pragma unroll
          for (int q = 0; q < SCAN_MAXW; ++q) ps[g][q] = q < nw ? ps[g][q] : 0.f;
          s[g] = ((ps[g][0] + ps[g][1]) + (ps[g][2] + ps[g][3])) +
                 ((ps[g][4] + ps[g][5]) + (ps[g][6] + ps[g][7]));
        }
        float out, outc = 0.f;
        scan_element<KIND>(a, s, cp, bias, ckd, prev, prevc, cgv, cgc, out, outc);
        float* dst = a.u + out_pt(i) * BW + eo;
        const uintx4 quad = scan_quad(out);
        if (ok && (tid & 3) == 0) scan_store_agent(dst, quad);
        if (KIND == SCAN_LSTM && ok) {
          if (ITEMS)                                   // (read by the workgroup of the next step)
            __hip_atomic_store((unsigned*)dst + H, scan_bits(outc), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
          else
            dst[H] = outc;
        }
        prev = out;
        prevc = outc;
      } else if (stopped) {
        return;
      }
    }
  } while (ITEMS);
}

// Marks the points the solve will write (behind a solve inside the XCDs only the takeover reads these marks,
// 21 us for 2048 x 32 x 512), clears its control words and fills the rings (ring4 units of
// four floats; see kernels_scan_xcd.hip): slot 0 is the state u0 the solve starts from (adjoint: its
// products with the coefficients k0 of the first step), the others are marked.  closed: XCDs that take no
// part, as in CTL_WORD.
__global__ __launch_bounds__(256) void scan_mark_kernel(uintx4* p, long long n4, ScanArgs a,
                                                        const float* u0, const float* k0, int W, int rows,
                                                        int hp, int terms, unsigned closed) {
  if (blockIdx.x == 0 && threadIdx.x < CTL_WORDS)
    a.ctl[threadIdx.x] = threadIdx.x == CTL_WORD ? (int)closed : 0;
  const uintx4 s = {SENTINEL, SENTINEL, SENTINEL, SENTINEL};
  const long long t0 = (long long)blockIdx.x * 256 + threadIdx.x, dt = 256LL * gridDim.x;
  for (long long i = t0; i < n4; i += dt) p[i] = s;
  if (terms) {     // [row block][slot][row quad][k / 32][k / 8 % 4][term][row] of eight bf16
    for (long long i = t0; i < a.ring4; i += dt) {
      const int row4 = (int)(i & 3), t = (int)(i >> 2 & 3), k = (int)(i / 16 % (hp / 8)) * 8;
      const long long q = i / 16 / (hp / 8);
      const int quads = rows / 4, row = ((int)(q / quads / 4) * quads + (int)(q % quads)) * 4 + row4;
      uintx4 v = s;
      if (t == 3 || k >= a.H) {
        v = uintx4{0, 0, 0, 0};
      } else if ((q / quads & 3) == 0) {
        unsigned h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const StateTerms x = state_terms(row < a.B ? u0[(long long)row * W + k + e] : 0.f);
          h[e] = t == 0 ? x.t01 & 0xffffu : t == 1 ? x.t01 >> 16 : x.t2;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = h[2 * e] | (h[2 * e + 1] << 16);
      }
      ((uintx4*)a.ring)[i] = v;
    }
    return;
  }
  const int vec4 = rows / 4 * hp, nvec = k0 ? 3 : 1;   // units of a vector: [row quad][k / 4][row]
  for (long long i = t0; i < a.ring4; i += dt) {
    const int q = (int)(i % vec4), vec = (int)(i / vec4 % nvec);
    const long long slot = i / vec4 / nvec;
    const int k = q % hp / 4 * 4;
    uintx4 v = s;
    if (k >= a.H) {
      v = uintx4{0, 0, 0, 0};
    } else if ((slot & 3) == 0) {
      const int row = (int)(slot >> 2) * rows + q / hp * 4 + (q & 3);
      floatx4 f = zero4();
      if (row < a.B) {
        f = ldg4(u0 + (long long)row * W + k);
        if (k0) f *= ldg4(k0 + (long long)row * a.kw + vec * a.H + k);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = scan_bits(f[e]);
    }
    ((uintx4*)a.ring)[i] = v;
  }
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
// Workgroups that can be resident whatever the kernel's registers: one per CU of the current device
// (a partition of the GPU has fewer than the whole).
static int scan_max_wg() {
  constexpr int MAX_DEV = 64;
  static std::atomic<int> cus[MAX_DEV];                // 0: not asked yet
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEV) return 0;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n < SCAN_MAXWG ? n : SCAN_MAXWG;
}
// MGRIT_SCAN_XCDS in the environment: a mask of the XCDs that may take row blocks, none of them: exchange
// through memory (tests: both forms and every way of sharing a solve between them and the takeover).
static unsigned scan_xcds() {
  const char* e = std::getenv("MGRIT_SCAN_XCDS");
  return e ? (unsigned)std::strtoul(e, nullptr, 0) & 0xffu : 0xffu;
}
static ScanShape scan_shape(int B, int H) {
  const int max_wg = scan_max_wg(), quads = (B + 3) / 4;
  ScanShape s;
  s.nch = H > 64 * SCAN_MAXW ? 2 : 1;
  s.nw = (H + 64 * s.nch - 1) / (64 * s.nch);
  s.ncg = (H + SCAN_CP - 1) / SCAN_CP;
  s.rb = 1;
  while (s.rb < 8 && (quads + s.rb - 1) / s.rb * s.ncg > max_wg) s.rb *= 2;
  s.nrb = (quads + s.rb - 1) / s.rb;
  if (s.nw < s.rb) s.nw = s.rb;                       // wave r finishes row group r
  return s;
}

// A row block per XCD (kernels_scan_xcd.hip): false if the shape does not fit or gains nothing.
// Up to 512 columns, 16 per workgroup, us per step here : all CUs through memory, forward / adjoint:
// 32 x 512 1.27 / 1.27 : 1.81 / 2.54, 64 x 512 1.9 / 1.9 : 3.7 / 4.0, 16 x 256 0.97 / 0.91 : 1.50 / 1.59,
// 3 x 500 1.22 / 1.23 : 2.00 / 2.23, LSTM 32 x 512 1.54 : 2.87.  Beyond, 32 per workgroup fill the
// registers of a CU and the fp32 matrix pipe takes half of the step: 32 x 1024 2.6 / 2.9 : 5.8 / 6.0, 16 x
// 768 2.6 / 2.9 : 2.9 / 3.4, but 8 x 1024 2.7 / 3.0 : 3.0 / 3.6, and a second solve on another stream,
// for which the other form leaves half of the CUs, would wait: only where that form takes more.  Beside other
// work (4096^3 bf16 products on another stream, this : the other form, us per step) it stays the faster one:
// 32 x 512 2.7 : 3.2, 3 x 500 2.0 : 2.5, 32 x 1000 3.8 : 6.4, 64 x 512 4.0 : 5.6, 8 x 1024 on bf16 weights 2.4 : 3.8.
// More rows than one quad for each XCD follow each other within the step, up to four quads; the step launches
// (a launch per step above 64 rows) : this, us per step of the whole call: scan 100 x 512 13.3 : 4.4, 100 x
// 1000 26.0 : 10.8, 64 x 1000 10.2 : 6.1, 256 x 256 9.0 : 3.3, LSTM 100 x 200 10.7 : 2.5, ODE 100 x 512 7.3 :
// 2.5, scan + back-propagation 100 x 512 33.6 : 10.8, 100 x 1000 67.9 : 33.5.
// On terms of the state (ScanArgs): 8 x 512 1.01 : 2.00, 1 x 1024 1.42 : 2.25, 8 x
// 1024 1.53 : 3.02, 64 x 1024 2.3 : 9.4, at any number of rows (two solves of 8 x 1024 at once 0.89 : 1.82 ms).
constexpr int SCAN_XCD_MAX_QUADS = 4;                  // per row block
static bool scan_shape_xcd(int kind, int B, int H, bool terms, ScanShape& s) {
  if (scan_max_wg() != SCAN_XCDS * SCAN_XCD_CUS || scan_xcds() == 0) return false;
  const int quads = (B + 3) / 4;
  s.terms = terms;
  s.ct = H > 512 ? 2 : 1;
  s.hp = H > 512 ? 1024 : H > 256 ? 512 : 256;
  s.ncg = (H + s.ct * SCAN_CP - 1) / (s.ct * SCAN_CP);
  const int fit = SCAN_XCD_CUS / s.ncg * SCAN_XCDS;    // row blocks, each with all its columns in one XCD
  if (fit == 0) return false;
  s.rb = (quads + fit - 1) / fit;
  if (s.ct == 2) {
    const int ncg16 = (H + SCAN_CP - 1) / SCAN_CP;
    if (kind == SCAN_LSTM || (!s.terms && quads * ncg16 <= SCAN_MAXWG / 2)) return false;   // (LSTM: registers)
  }
  if (s.rb > SCAN_XCD_MAX_QUADS) return false;
  s.nrb = (quads + s.rb - 1) / s.rb;
  s.gpx = (s.nrb + SCAN_XCDS - 1) / SCAN_XCDS;
  s.nx = (s.nrb + s.gpx - 1) / s.gpx;
  return true;
}
size_t scan_ring_floats(int kind, int B, int H, bool terms) {
  ScanShape s;
  if (!scan_shape_xcd(kind, B, H, terms, s)) return 0;
  return (size_t)16 * s.rb * s.nrb * s.hp * (kind == SCAN_ADJOINT ? 3 : s.terms ? 2 : 1);
}

// Registers of scan_kernel: the adjoint holds three coefficient rows per state row, the LSTM four gates.
static int scan_max_quads(int kind, int nch) { return kind == SCAN_ADJOINT && nch == 2 ? 2 : 4; }

// 16 to 1024 columns, up to 64 rows (the few-row range of the step kernels), with a row block per XCD up
// to 16 rows for each.  A solve costs three launches (mark, scan, items) whatever its length: below eight
// steps the chain of step launches is as fast.
bool scan_covers(int kind, long long N, int B, int H, bool terms, bool ring) {
  if (N < 8 || N > (1LL << 30) || H < 16 || H > 128 * SCAN_MAXW) return false;
  ScanShape s;
  if (ring && scan_shape_xcd(kind, B, H, terms, s)) return true;
  if (B > 64) return false;
  s = scan_shape(B, H);
  return s.rb <= scan_max_quads(kind, s.nch) && s.nrb * s.ncg <= scan_max_wg();
}

// xs: the shape of the form with a row block per XCD, null: this form.  Each launch's error is looked at
// by itself: the items take a solve that never started for one that is done.
template <int KIND, int NCH, int RB, class WT>
static hipError_t launch_scan_shape(const ScanArgs& a, const ScanShape& s, const ScanShape* xs,
                                    hipStream_t st) {
  const dim3 grid((unsigned)(s.nrb * s.ncg)), block(64 * s.nw);
  hipError_t err;
  if (xs) {
    err = launch_scan_xcd(KIND, a, *xs, st);
  } else {
    hipLaunchKernelGGL((scan_kernel<KIND, NCH, RB, WT, false, false>), grid, block, 0, st, a, s.nrb, 0);
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  if constexpr (KIND == SCAN_GRU && sizeof(WT) == 2) {
    if (xs && xs->terms) {
      hipLaunchKernelGGL((scan_kernel<KIND, NCH, RB, WT, true, true>), grid, block, 0, st, a, s.nrb,
                         xs->gpx * xs->rb);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((scan_kernel<KIND, NCH, RB, WT, true, false>), grid, block, 0, st, a, s.nrb,
                     xs ? xs->gpx * xs->rb : 0);
  return hipGetLastError();
}
template <int KIND, class WT>
static hipError_t launch_scan_kind(const ScanArgs& a, const ScanShape* xs, hipStream_t st) {
  ScanShape s = scan_shape(a.B, a.H);
  const int max_rb = scan_max_quads(KIND, s.nch);
  if (s.rb > max_rb) {                                // (behind xs: any number of workgroups will do)
    s.rb = max_rb;
    s.nrb = ((a.B + 3) / 4 + s.rb - 1) / s.rb;
  }
#define MG_SCAN_CASE(NCH, RB) \
  if (s.nch == NCH && s.rb == RB) return launch_scan_shape<KIND, NCH, RB, WT>(a, s, xs, st);
  MG_SCAN_CASE(1, 1)
  MG_SCAN_CASE(1, 2)
  MG_SCAN_CASE(1, 4)
  MG_SCAN_CASE(2, 1)
  MG_SCAN_CASE(2, 2)
  if constexpr (KIND != SCAN_ADJOINT) {
    MG_SCAN_CASE(2, 4)
  }
#undef MG_SCAN_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_scan(int kind, const ScanArgs& a0, hipStream_t st) {
  ScanArgs a = a0;
  a.wait_ticks = a.N * SCAN_ARRIVE_PER_STEP;
  if (a.wait_ticks < SCAN_ARRIVE_MIN) a.wait_ticks = SCAN_ARRIVE_MIN;
  if (a.wait_ticks > SCAN_ARRIVE_MAX) a.wait_ticks = SCAN_ARRIVE_MAX;
  // MGRIT_SCAN_WAIT_TICKS in the environment: another limit for the wait (tests use 0: no wait)
  if (const char* e = std::getenv("MGRIT_SCAN_WAIT_TICKS")) a.wait_ticks = std::atoll(e);
  const int W = kind == SCAN_LSTM ? 2 * a.H : a.H;
  const int prof = kind == SCAN_GRU ? 4 : kind == SCAN_ADJOINT ? 5 : kind == SCAN_LSTM ? 9 : 8;
  prof_begin(prof, st, a.B, STEP_RELAX);
  ScanShape xshape{};
  const bool xcd = a.ring && scan_shape_xcd(kind, a.B, a.H, a.terms, xshape);
  const ScanShape* xs = xcd ? &xshape : nullptr;
  if (!xcd) a.ring = nullptr;
  a.ring4 = xcd ? (long long)scan_ring_floats(kind, a.B, a.H, a.terms) / 4 : 0;
  const long long n4 = (long long)a.N * a.B * W / 4, BW = (long long)a.B * W;
  const long long nb = (n4 + 255) / 256;
  unsigned closed = 0;
  for (int x = 0; x < SCAN_XCDS; ++x)
    if (xcd && !(scan_xcds() >> x & 1)) closed |= XCD_CLOSED << 4 * x;
  hipLaunchKernelGGL(scan_mark_kernel, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256), 0, st,
                     (uintx4*)(a.u + (kind == SCAN_ADJOINT ? 0 : BW)), n4, a,
                     a.u + (kind == SCAN_ADJOINT ? a.N * BW : 0),
                     kind == SCAN_ADJOINT ? a.kap + (long long)a.N * a.B * a.kw : nullptr, W,
                     4 * xshape.rb, xshape.hp, xshape.terms, closed);
  hipError_t err = hipGetLastError();
  const bool h16 = a.bf16 == 1;
  if (err != hipSuccess) {
    // (nothing is marked)
  } else if (kind == SCAN_GRU) {
    err = h16 ? launch_scan_kind<SCAN_GRU, bf16_t>(a, xs, st) : launch_scan_kind<SCAN_GRU, float>(a, xs, st);
  } else if (kind == SCAN_ADJOINT) {
    err = h16 ? launch_scan_kind<SCAN_ADJOINT, bf16_t>(a, xs, st)
              : launch_scan_kind<SCAN_ADJOINT, float>(a, xs, st);
  } else if (kind == SCAN_LSTM) {
    err = launch_scan_kind<SCAN_LSTM, float>(a, xs, st);
  } else {
    err = launch_scan_kind<SCAN_ODE, float>(a, xs, st);
  }
  const double rows = (double)a.N * a.B;
  const int ng = kind == SCAN_LSTM ? 4 : kind == SCAN_ODE ? 1 : 3;
  const double bytes = kind == SCAN_ADJOINT ? 28.0 : kind == SCAN_GRU ? 20.0 : kind == SCAN_LSTM ? 32.0 : 16.0;
  prof_end(prof, 2.0 * ng * rows * a.H * a.H, bytes * rows * a.H, st);
  return err;
}

}  // namespace mg

// Serial propagation of a few rows as one launch, each block of rows inside one XCD.
//
// The rows of a batch do not meet in a serial solve, so a block of rows needs no other XCD than the one
// that computes it, if that XCD holds all recurrent weights (its 32 CUs have 16 MB of registers).  The
// state then travels through the L2 of the XCD instead of the memory side (see kernels_scan.hip for the
// rest of the scheme, which is the same: weights in registers, row quads, waves split K).
//
// Exchange.  A row block has a ring of four state rows, [slot][row quad][k / 4][row][4]: a workgroup's
// columns of a quad are contiguous, and so are 64 k of a quad for the wave that loads them.  (The adjoint
// has three vectors per slot, the products of the state with the coefficients of the step: who makes
// an element multiplies it, and nobody else loads the coefficients.)  Slot i % 4
// receives state i; every word is marked (SENTINEL) before it is written and polled until it has changed.
// With state i + 1 a workgroup marks its part of slot i - 1 again: it has seen all of state i, so every
// workgroup has read all of state i - 1.  The mark is in the L2 before the workgroup's part of state i + 2
// is sent (its epilogue waves wait for their stores when they poll for state i + 1), and nobody looks at
// that slot for the mark's successor, state i + 3, before it has seen all of state i + 2.  Stores go to
// the L2 (vector stores pass through the L1), polls at agent scope pass by the L1.  The ring stays in L2:
// rows of the output array polled there instead cost 0.83 us per exchange (each line is fetched from
// memory first), the ring 0.53 us, the exchange through memory 1.37 us (32 workgroups of 16 columns, four
// rows; the exchange alone).
//
// TERMS: a serial scan of the GRU on bf16 weights contracts on the bf16 matrix pipe, which is 16 times as
// fast: the state travels as three bf16 terms (exact: state_terms), which fill 12 of the 16 rows of
// v_mfma_f32_16x16x32_bf16 for four state rows, [slot][row quad][k / 32][k / 8 % 4][term][row][8]; products
// of terms and weights are exact, the sums fp32.  8 x 1024: 0.3 instead of 1.3 us of MFMAs per step, half
// the registers.  The instruction rounds its sums down where the fp32 one rounds to nearest; it makes fewer
// of them, and the states are no further from 64 bits (five inputs each: 1024 steps of 8 x 1024 1.07e-7
// against 1.09e-7 with fp32 MFMAs, 2048 of 1 x 512 1.04 : 1.05, 1024 of 3 x 264 1.03 : 1.04), nor to one
// side of it (sum of the errors over sum of their sizes, mean of the five -0.3 % : -0.2 % at 8 x 1024).
//
// An infinite weight cannot be contracted so (term_weights_infinite): the workgroup that holds one gives up
// the solve, and the takeover launch contracts those weights in fp32.
//
// Which XCD a workgroup runs on it reads from the hardware (XCC_ID).  The launch has enough workgroups
// to fill what it needs on every XCD; the XCD whose workgroups have all arrived takes the next group of
// row blocks (xcd_role), the others leave when all are taken.  A group that is taken has all its
// workgroups resident and needs nothing else.  If an XCD does not fill up in time, its workgroups leave.
// The takeover launch solves the row blocks that no XCD has taken, for whatever reason
// (scan_kernel<.., true>), with the same bits.
#include "scan_exchange.h"

namespace mg {

// Stores to the L2 of this XCD.
__device__ inline void ring_store(float* p, uintx4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// XCD this wave runs on (hardware register XCC_ID, bits 2:0).
__device__ inline int scan_xcd() { return __builtin_amdgcn_s_getreg((2 << 11) | (0 << 6) | 20); }
// One thread per workgroup.  The group of row blocks the XCD of this workgroup takes, -1: none.  The
// workgroup that completes the `per` workgroups of an XCD claims the next of the `need` groups for it;
// the others wait for that, until all groups are given away, or until the time limit, when they close
// their XCD (nobody may start there any more) and leave the rest to the launch behind.
__device__ inline int xcd_role(int* ctl, int xcd, int ticket, int per, int need, long long wait_ticks) {
  if (ticket >= per) return -1;
  unsigned* word = (unsigned*)ctl + CTL_WORD;
  const int sh = 4 * xcd;
  const long long t0 = ticks();
  while (true) {
    unsigned w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned v = (w >> sh) & 15;
    if (v) return v == XCD_CLOSED ? -1 : (int)v - 1;
    const int n = xcd_groups(w);
    if (n >= need) return -1;
    const bool closes = ticket < per - 1 && ticks() - t0 >= wait_ticks;
    if (closes || ticket == per - 1) {
      const unsigned mine = closes ? XCD_CLOSED : (unsigned)n + 1;
      if (__hip_atomic_compare_exchange_strong(word, &w, w | (mine << sh), __ATOMIC_RELAXED,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        return closes ? -1 : n;
      }
      continue;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
__device__ inline void ring_store(float* p, uintx2 v) {
  asm volatile("global_store_dwordx2 %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// A 16-byte load at agent scope (passes by the L1), never merged with another one.
__device__ inline uintx4 ring_load(__amdgpu_buffer_rsrc_t ring, unsigned off, unsigned slot) {
  constexpr int SC1_VOLATILE = (1 << 4) | (1 << 31);
  return __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(ring, (int)off, (int)slot,
                                                                          SC1_VOLATILE));
}
constexpr int WAIT_VMCNT_0 = 0x0f70;                   // (no other counter)
template <int NL>
__device__ inline bool ring_waits(const uintx4 (&v)[NL]) {
  unsigned top = 0;                                    // SENTINEL is the largest word
#pragma unroll
  for (int q = 0; q < NL; ++q)
    top = max(max(max(top, v[q][0]), max(v[q][1], v[q][2])), v[q][3]);
  return top == SENTINEL;
}
// Units of 64 clocks between the barrier of a step and the first look for the next state of a wave that
// does not finish elements: about what the sums, the gates, the stores and their way to the L2 take.
// Looks before that fail, hold up the stores in the L2, and the one that would succeed waits for the last
// of them.  us per step without : with (every value from 1 to 14 was tried): adjoint 32 x 512 1.29 : 1.15,
// 16 x 256 0.91 : 0.87, GRU 32 x 512 1.30 : 1.19, 3 x 500 1.24 : 1.14, 16 x 256 0.98 : 0.97, 8 x 512 on bf16
// weights 1.01 : 0.95, LSTM 32 x 512 1.56 : 1.50; two to four quads a step hide it.
__device__ constexpr int first_look(int kind, int ct) {
  return kind == SCAN_GRU ? (ct == 2 ? 13 : 10) : kind == SCAN_LSTM ? 12 : 6;
}
// x in another register, now: left to the compiler, the copy comes behind the load that overwrites x, and
// waits for it.
__device__ inline float moved(float x) {
  float y;
  asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
  return y;
}
// NW waves of NV x NCH chunks of 64 k (NV sums over NCH chunks each: what a wave of scan_kernel sums, so
// the bits are the same); RB row quads one after the other, CT tiles of 16 columns per workgroup.  The
// waves also finish the elements (waves of their own for that are no faster: 1.38 against 1.35 us per
// step at 32 x 512, where they make nine of eight).  With two column tiles the weights leave few registers:
// the adjoint spills 50 to 59 of 512 with three or four quads and 14 with two on bf16 weights, the fp32
// contraction of the GRU 4 to 7 of 256 with two or more; the times at scan_shape_xcd are with that.
template <int KIND, int CT, int NV, int NCH, int NW, int RB, class WT, bool TERMS>
__device__ __forceinline__ void xcd_solve(const ScanArgs& a, const ScanShape& sh) {
  constexpr int NG = ScanGates<KIND>::value;
  constexpr bool ADJ = KIND == SCAN_ADJOINT;
  constexpr int NS = ADJ ? 1 : NG;
  constexpr int AG = ScanVectors<KIND>::value;
  constexpr int NC = NV * NCH;
  constexpr int NL = (TERMS ? 2 : AG) * NC;     // loads per row quad
  constexpr bool AHEAD = RB > 1 && NL <= 8;            // (registers)
  constexpr int NE = (RB * CT + NW - 1) / NW;          // elements a lane finishes
  constexpr int NP = NG == 1 ? 2 : 1;
  constexpr int HP = 64 * NC * NW;                     // columns of a ring row, zero from H on
  constexpr int KB = 2 * NC;                           // TERMS: blocks of 32 k per wave
  constexpr unsigned VEC = RB * HP * 4, SLOT = TERMS ? 2 * VEC : AG * VEC;    // floats
  __shared__ float part[2][NW * NV][RB * CT][NS][64];
  __shared__ int stop, role;
  const int H = a.H, B = a.B, N = a.N;
  const int W = KIND == SCAN_LSTM ? 2 * H : H;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  if (tid == 0) {
    const int x = scan_xcd();
    const int ticket = __hip_atomic_fetch_add(a.ctl + CTL_TICKETS + x, 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
    const int g = xcd_role(a.ctl, x, ticket, sh.gpx * sh.ncg, sh.nx, a.wait_ticks);
    const int r = g * sh.gpx + ticket / sh.ncg;
    role = g < 0 || r >= sh.nrb ? -1 : ticket % sh.ncg * sh.nrb + r;
    stop = 0;
  }
  __syncthreads();
  const int unit = __builtin_amdgcn_readfirstlane(role);
  if (unit < 0) return;
  const int rb = unit % sh.nrb, cg = unit / sh.nrb;
  const int r0 = rb * RB * 4, j0 = cg * CT * SCAN_CP;
  const long long BW = (long long)B * W;
  auto in_pt = [&](int i) { return (long long)(ADJ ? N - i : i); };
  auto out_pt = [&](int i) { return (long long)(ADJ ? N - i - 1 : i + 1); };
  float* const ring = a.ring + (long long)rb * 4 * SLOT;
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(ring, 0, 4 * SLOT * 4, 0x00027000);

  const int kw0 = wv * 64 * NC;
  // weights: column j0 + 16 t + lane % 16, k = kw0 + 64 c + 16 (lane / 16) + 0..15 (zero beyond H;
  // columns beyond H repeat the last one and are never stored)
  float w[NC][CT * NG][16];
  bf16x8 wt[KB][CT * NG];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int j = min(j0 + t * SCAN_CP + (lane & 15), H - 1);
    if constexpr (TERMS) {
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int b = 0; b < KB; ++b)
          wt[b][t * NG + g] = term_weights((const bf16_t*)a.Wt + ((long long)g * H + j) * H,
                                           kw0 + 32 * b + 8 * (lane >> 4), H);
      continue;
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int k = kw0 + 64 * c + 16 * (lane >> 4) + 4 * q;
          const int kc = min(k, H - 4);
          const WT* p = (const WT*)a.Wt +
                        (ADJ ? (long long)j * 3 * H + g * H + kc : ((long long)g * H + j) * H + kc);
          const floatx4 v = k < H ? ldg4w(p) : zero4();
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            w[c][t * NG + g][4 * q + e] = v[e];
            if (sizeof(WT) == 2) asm volatile("" : "+v"(w[c][t * NG + g][4 * q + e]));   // (as floats)
          }
        }
  }
  if constexpr (TERMS) {
    if (term_weights_infinite(wt)) {      // (out like a wave that has waited too long, below)
      if (lane == 0) __hip_atomic_store(a.ctl + CTL_ABORT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      stop = 1;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_endpgm();
    }
  }
  // polled operand: row quad r, row lane % 4, k = kw0 + 64 c + 4 (lane / 4) + 0..3; lanes beyond the
  // rows read a row that is there (their sums are not stored)
  unsigned off[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const int row = min(r0 + 4 * r + (lane & 3), B - 1) - r0;
    if (TERMS)
      off[r] = (unsigned)(((row >> 2) * (HP >> 5) + (kw0 >> 5)) * 64 + (lane & ~3) + (row & 3)) * 16u;
    else
      off[r] = (unsigned)(((row >> 2) * (HP >> 2) + (kw0 >> 2) + (lane >> 2)) * 16 + (row & 3) * 4) * 4u;
  }
  // (terms: lane l reads term l / 4 % 4 of row l % 4, k = kw0 + 32 b + 8 (l / 16) + 0..7)
  // elements of this lane: wave e (and e + NW) finishes quad e % RB, tile e / RB.  Lane q of four stores 16
  // bytes: 0 the new state (adjoint: 0..2 its products with the three coefficients of the next step; terms:
  // 0..2 eight bytes each) to the ring, 1 (0..2) the mark, 2 (3) the output
  constexpr int OUT_LANE = ADJ || TERMS ? 3 : 2;
  constexpr uintx4 MARK = {SENTINEL, SENTINEL, SENTINEL, SENTINEL};
  const int q4 = lane & 3;
  auto mine = [&](int n) { return wv + n * NW < RB * CT; };
  bool ok[NE];
  unsigned eo[NE], po[NE], kqo[NE];
  float* base[NE];
  float bias[NE][NG], prev[NE], prevc[NE];             // prev: element of the row the step starts from
  float p[NE][NG], kd[NE], g[NE], gc[NE];
  floatx4 kq[NE];
  // what step i needs beside the state (kq: of the step behind it)
  auto request = [&](int n, int i) {
    if (ADJ) {
      kd[n] = (a.kap + in_pt(i) * B * a.kw + 3 * H)[po[n]];
      kq[n] = ldg4(a.kap + in_pt(min(i + 1, N - 1)) * B * a.kw + kqo[n]);
    } else {
      const float* pr = a.P + ((long long)(i + 1) * a.pstep - 1) * B * ((long long)NG * H);
#pragma unroll
      for (int q = 0; q < NG; ++q) p[n][q] = (pr + q * H)[po[n]];
    }
    if (a.g) {
      const float* gr = a.g + out_pt(i) * BW;
      g[n] = gr[eo[n]];
      if (KIND == SCAN_LSTM) gc[n] = (gr + H)[eo[n]];
    }
  };
#pragma unroll
  for (int n = 0; n < NE; ++n) {
    const int e = wv + n * NW, er = e % RB, et = e / RB;
    const int orow = r0 + 4 * er + quad_row(lane), oj = j0 + et * SCAN_CP + (lane & 15);
    const int erow = min(orow, B - 1), ej = min(oj, H - 1);
    ok[n] = mine(n) && orow < B && oj < H;
    eo[n] = (unsigned)erow * W + ej;
    po[n] = (unsigned)erow * (ADJ ? a.kw : NG * H) + ej;
    kqo[n] = (unsigned)erow * (ADJ ? a.kw : 0) + min(q4, 2) * H + (ej & ~3);
    const unsigned quado =
        TERMS ? (unsigned)((((er * (HP >> 5) + (ej >> 5)) * 4 + (ej >> 3 & 3)) * 16 + min(q4, 2) * 4 +
                            quad_row(lane)) * 4 + (ej >> 2 & 1) * 2)
              : (unsigned)((er * (HP >> 2) + (ej >> 2)) * 16 + quad_row(lane) * 4);
    base[n] = q4 == OUT_LANE ? a.u + (eo[n] & ~3u) : ring + quado + (ADJ ? q4 * VEC : 0);
    kd[n] = g[n] = gc[n] = prev[n] = prevc[n] = 0.f;
    kq[n] = zero4();
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      bias[n][q] = (KIND == SCAN_GRU || KIND == SCAN_LSTM) && mine(n) ? a.b_h[q * H + ej] : 0.f;
      p[n][q] = 0.f;
    }
    if (mine(n)) {
      request(n, 0);
      const float* u0 = a.u + in_pt(0) * BW;           // element of the row the step starts from
      prev[n] = u0[eo[n]];
      if (KIND == SCAN_LSTM) prevc[n] = (u0 + H)[eo[n]];
    }
  }

  for (int i = 0; i < N; ++i) {
    const unsigned slot = (unsigned)(i & 3) * (SLOT * 4);
    uintx4 v[AHEAD ? 2 : 1][NL];                       // a quad (and the one behind it on its way)
    auto load = [&](uintx4 (&d)[NL], int r) {
#pragma unroll
      for (int c = 0; c < NL / (TERMS ? 1 : AG); ++c)
#pragma unroll
        for (int g2 = 0; g2 < (TERMS ? 1 : AG); ++g2)
          d[c * (TERMS ? 1 : AG) + g2] = ring_load(rsrc, off[r] + c * 1024 + g2 * VEC * 4, slot);
    };
    float (*pt)[RB * CT][NS][64] = part[i & 1];
    float cp[NE][NG] = {}, cgv[NE], cgc[NE] = {}, ckd[NE] = {};
    floatx4 ckq[NE];
    float* sp[NE];
    if (i > 0 && !mine(0)) __builtin_amdgcn_s_sleep(first_look(KIND, CT));
    load(v[0], 0);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      uintx4 (&vr)[NL] = v[AHEAD ? r & 1 : 0];
      bool leave = false;
      for (int polls = 1; __any(ring_waits(vr)); ++polls) {
        if ((polls & 127) == 0) {
          if (polls >= SCAN_MAX_POLLS)
            __hip_atomic_store(a.ctl + CTL_ABORT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          leave = ctl_load(a.ctl + CTL_ABORT) != 0;
          if (leave) break;
        }
        load(vr, r);
      }
      if (leave) {      // the other waves see it behind the barrier, which does not wait for waves that ended
        stop = 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_endpgm();
      }
      if (r == 0) {
        // the marks this wave made in the step before are in the L2 (the loads above are younger: no wait)
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT_0);
      }
      if (AHEAD && r + 1 < RB) load(v[AHEAD ? (r + 1) & 1 : 0], r + 1);
      if (r == 0) {
#pragma unroll
        for (int n = 0; n < NE; ++n) {
          cgv[n] = moved(g[n]);
          if constexpr (ADJ) {
            ckd[n] = moved(kd[n]);
#pragma unroll
            for (int q = 0; q < 4; ++q) ckq[n][q] = moved(kq[n][q]);
          } else {
#pragma unroll
            for (int q = 0; q < NG; ++q) cp[n][q] = moved(p[n][q]);
          }
          if constexpr (KIND == SCAN_LSTM) cgc[n] = moved(gc[n]);
          if (mine(n)) request(n, min(i + 1, N - 1));
          // where this lane stores 16 bytes
          const int sl = ADJ || TERMS ? (i + 1) & 3 : (i + 1 + 2 * (q4 & 1)) & 3;
          sp[n] = base[n] + (q4 == OUT_LANE ? out_pt(i) * BW : (long long)(sl * (int)SLOT));
          asm volatile("" : "+v"(sp[n]));              // (computed before the barrier)
        }
      }
      if constexpr (TERMS) {
        floatx4 acc[CT * NG];
#pragma unroll
        for (int q = 0; q < CT * NG; ++q) acc[q] = zero4();
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int q = 0; q < CT * NG; ++q) acc[q] = term_mma(vr[b], wt[b][q], acc[q]);
#pragma unroll
        for (int q = 0; q < CT * NG; ++q) pt[wv][q / NG * RB + r][q % NG][lane] = term_fold(acc[q]);
      }
#pragma unroll
      for (int h = 0; h < (TERMS ? 0 : NV); ++h) {
        floatx4 acc[1][CT * NG][NP];
#pragma unroll
        for (int q = 0; q < CT * NG; ++q)
#pragma unroll
          for (int n = 0; n < NP; ++n) acc[0][q][n] = zero4();
#pragma unroll
        for (int c = h * NCH; c < (h + 1) * NCH; ++c)
          quad_mma<1, CT * NG, NP>(
              acc, [&](int, int q) { return __builtin_bit_cast(floatx4, vr[c * AG + (ADJ ? q % NG : 0)]); },
              [&](int q) -> const float (&)[16] { return w[c][q]; });
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          floatx4 sum[NG];
#pragma unroll
          for (int q = 0; q < NG; ++q)
            sum[q] = NP > 1 ? acc[0][t * NG + q][0] + acc[0][t * NG + q][NP - 1] : acc[0][t * NG + q][0];
          if (ADJ) {
            pt[wv * NV + h][t * RB + r][0][lane] = quad_fold(sum[0] + sum[NG > 1 ? 1 : 0] + sum[NG - 1]);
          } else {
#pragma unroll
            for (int q = 0; q < NG; ++q)
              pt[wv * NV + h][t * RB + r][ADJ ? 0 : q][lane] = quad_fold(sum[q]);
          }
        }
      }
      if (!AHEAD && r + 1 < RB) load(v[0], r + 1);
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NE; ++n) {
      if (!mine(n)) continue;
      // partial sums (every read in flight before the first addition)
      float s[NS], ps[NS][SCAN_MAXW];
#pragma unroll
      for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int m = 0; m < SCAN_MAXW; ++m)
          ps[q][m] = m < NW * NV ? pt[m < NW * NV ? m : 0][wv + n * NW][q][lane] : 0.f;
      const int stopped = stop;
#pragma unroll
      for (int q = 0; q < NS; ++q)
        s[q] = ((ps[q][0] + ps[q][1]) + (ps[q][2] + ps[q][3])) +
               ((ps[q][4] + ps[q][5]) + (ps[q][6] + ps[q][7]));
      float out, outc = 0.f;
      scan_element<KIND>(a, s, cp[n], bias[n], ckd[n], prev[n], prevc[n], cgv[n], cgc[n], out, outc);
      const uintx4 quad = scan_quad(out);
      if (stopped) return;
      if constexpr (ADJ) {
        uintx4 pr;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned b = scan_bits(ckq[n][e] * __uint_as_float(quad[e]));
          pr[e] = q4 == OUT_LANE ? quad[e] : b;
        }
        if (ok[n]) {
          ring_store(sp[n], pr);
          if (q4 != OUT_LANE) ring_store(base[n] + ((i + 3) & 3) * (int)SLOT, MARK);
        }
      } else if constexpr (TERMS) {
        // lane q < 3 of four stores term q of the four columns
        const StateTerms st = state_terms(out);
        unsigned y[4];
#define MG_GATHER(e, ctrl)                                                        \
  {                                                                               \
    const unsigned y01 = __builtin_amdgcn_mov_dpp(st.t01, ctrl, 0xf, 0xf, true);  \
    const unsigned y2 = __builtin_amdgcn_mov_dpp(st.t2, ctrl, 0xf, 0xf, true);    \
    y[e] = q4 == 2 ? y2 : y01;                                                    \
  }
        MG_GATHER(0, 0x00) MG_GATHER(1, 0x55) MG_GATHER(2, 0xaa) MG_GATHER(3, 0xff)
#undef MG_GATHER
        const unsigned half = q4 == 1 ? 0x07060302u : 0x05040100u;
        const uintx2 d = {__builtin_amdgcn_perm(y[1], y[0], half), __builtin_amdgcn_perm(y[3], y[2], half)};
        if (ok[n]) {
          if (q4 != OUT_LANE) {
            ring_store(sp[n], d);
            ring_store(base[n] + ((i + 3) & 3) * (int)SLOT, uintx2{SENTINEL, SENTINEL});
          } else {
            ring_store(sp[n], quad);
          }
        }
      } else {
        uintx4 d;
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = q4 == 1 ? SENTINEL : quad[e];
        if (ok[n] && q4 <= OUT_LANE) ring_store(sp[n], d);
        if (KIND == SCAN_LSTM && ok[n]) (a.u + out_pt(i) * BW + H)[eo[n]] = outc;
      }
      prev[n] = out;
      prevc[n] = outc;
    }
  }
}

template <int KIND, int CT, int NV, int NCH, int NW, int RB, class WT, bool TERMS>
__global__ __launch_bounds__(64 * NW) void xcd_scan_kernel(ScanArgs a, ScanShape sh) {
  xcd_solve<KIND, CT, NV, NCH, NW, RB, WT, TERMS>(a, sh);
}
template <int KIND, int CT, int NV, int NCH, int NW, int RB, class WT, bool TERMS>
__global__ __launch_bounds__(64 * NW) void adj_xcd_scan_kernel(ScanArgs a, ScanShape sh) {
  xcd_solve<KIND, CT, NV, NCH, NW, RB, WT, TERMS>(a, sh);
}

template <int KIND, int CT, int NV, int NCH, int NW, int RB, class WT, bool TERMS>
static void launch(const ScanArgs& a, const ScanShape& s, hipStream_t st) {
  // (workgroups go to the XCDs in turn)
  const dim3 grid((unsigned)(SCAN_XCDS * s.gpx * s.ncg)), block(64 * NW);
  if constexpr (KIND == SCAN_ADJOINT)
    hipLaunchKernelGGL((adj_xcd_scan_kernel<KIND, CT, NV, NCH, NW, RB, WT, TERMS>), grid, block, 0, st, a, s);
  else
    hipLaunchKernelGGL((xcd_scan_kernel<KIND, CT, NV, NCH, NW, RB, WT, TERMS>), grid, block, 0, st, a, s);
}
template <int KIND, int CT, int NV, int NCH, int NW, class WT, bool TERMS>
static void launch_rows(const ScanArgs& a, const ScanShape& s, hipStream_t st) {
  if (s.rb == 1) launch<KIND, CT, NV, NCH, NW, 1, WT, TERMS>(a, s, st);
  else if (s.rb == 2) launch<KIND, CT, NV, NCH, NW, 2, WT, TERMS>(a, s, st);
  if constexpr (KIND != SCAN_GRU || sizeof(WT) == 4 || TERMS) {     // (otherwise up to 64 rows: two quads)
    if (s.rb == 3) launch<KIND, CT, NV, NCH, NW, 3, WT, TERMS>(a, s, st);
    else if (s.rb == 4) launch<KIND, CT, NV, NCH, NW, 4, WT, TERMS>(a, s, st);
  }
}
template <int KIND, class WT, bool TERMS = false>
static void launch_kind(const ScanArgs& a, const ScanShape& s, hipStream_t st) {
  if (s.ct == 1 && s.hp == 256) return launch_rows<KIND, 1, 1, 1, 4, WT, TERMS>(a, s, st);
  if (s.ct == 1 && s.hp == 512) return launch_rows<KIND, 1, 1, 1, 8, WT, TERMS>(a, s, st);
  if constexpr (KIND == SCAN_ADJOINT) {
    if (s.ct == 2) launch_rows<KIND, 2, 2, 2, 4, WT, TERMS>(a, s, st);
  } else if constexpr (KIND != SCAN_LSTM) {
    if (s.ct == 2) launch_rows<KIND, 2, 1, 2, 8, WT, TERMS>(a, s, st);
  }
}

hipError_t launch_scan_xcd(int kind, const ScanArgs& a, const ScanShape& s, hipStream_t st) {
  const bool h16 = a.bf16 == 1;
  if (kind == SCAN_GRU) {
    if (s.terms) launch_kind<SCAN_GRU, bf16_t, true>(a, s, st);
    else if (h16) launch_kind<SCAN_GRU, bf16_t>(a, s, st);
    else launch_kind<SCAN_GRU, float>(a, s, st);
  } else if (kind == SCAN_ADJOINT) {
    if (h16) launch_kind<SCAN_ADJOINT, bf16_t>(a, s, st);
    else launch_kind<SCAN_ADJOINT, float>(a, s, st);
  } else if (kind == SCAN_LSTM) {
    launch_kind<SCAN_LSTM, float>(a, s, st);
  } else {
    launch_kind<SCAN_ODE, float>(a, s, st);
  }
  return hipGetLastError();
}

}  // namespace mg

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
// Measured against the chain of step launches: serial scan + back-propagation of 2048 steps x 32 x
// 512 fp32 31.4 -> 14.7 ms (of which 4.4 ms are the GEMMs both share), scan of 512 steps x 8 x 1024
// on bf16 weights 3.20 -> 1.61 ms, of 777 steps x 3 x 500 3.09 -> 1.61 ms (2.0 us per step: about
// 1.3 us of exchange, 0.3 us of MFMAs, the rest LDS sums and gates).  A ninth wave that takes the
// epilogue off the polling waves is slower (15.3 ms).
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
// all resident, us per step): 8 x 1024 bf16 5.9 : 8.5 : 3.1, 64 x 1024 17.6 : 12.4 : 10.0, 3 x 500 4.1 :
// 3.6 : 2.1, 16 x 256 4.0 : 3.8 : 1.6, LSTM 32 x 512 5.2 : 6.7 : 3.0; three streams at once, ms: bptt of
// 256 x 32 x 1024 24.0 : 23.4, scans of 256 x 64 x 1024 9.8 : 11.5, LSTM 512 x 32 x 512 6.3 : 9.2.
#include <atomic>
#include <cstdlib>

#include "gates.h"
#include "gemm_core_bf16.h"
#include "quad.h"
#include "scan.h"

namespace mg {

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
constexpr unsigned SENTINEL = 0xffffffffu;
constexpr int SCAN_MAXW = 8;                 // waves per workgroup
constexpr int SCAN_MAXWG = 256;              // workgroups of a solve at most (one per CU)
constexpr int SCAN_CP = 16;                  // hidden columns per workgroup
// Limit of the wait for all workgroups, in ticks of the 100 MHz clock: half a microsecond per step (a
// quarter of the solve), 50 us (several times what an arrival on a free GPU takes) to 5 ms.
constexpr long long SCAN_ARRIVE_PER_STEP = 50, SCAN_ARRIVE_MIN = 5000, SCAN_ARRIVE_MAX = 500000;
constexpr long long SCAN_STEP_TICKS = 200000000;     // 2 s: bound of a single wait, all resident
constexpr int SCAN_MAX_POLLS = 1 << 24;              // the same, items from the counter (counted in
                                                     // polls: a GPU that is taken away counts none)

template <int KIND>
struct ScanGates {
  static constexpr int value = KIND == SCAN_LSTM ? 4 : KIND == SCAN_ODE ? 1 : 3;
};

// N 16-byte loads at agent scope, all in flight together; base is uniform, off[] are byte offsets
// of the lane.  The wait is part of the block: the results are valid when it ends.  So are the five
// wait states between a vector instruction that writes the scalar base (v_readfirstlane) and the
// first load that reads it: the compiler keeps that distance for its own instructions only.
__device__ inline void scan_load(uintx4 (&v)[1], const float* base, const unsigned (&off)[1]) {
  asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(v[0]) : "v"(off[0]), "s"(base) : "memory");
}
__device__ inline void scan_load(uintx4 (&v)[2], const float* base, const unsigned (&off)[2]) {
  asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %2, %4 sc1\n\tglobal_load_dwordx4 %1, %3, %4 sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]) : "v"(off[0]), "v"(off[1]), "s"(base) : "memory");
}
__device__ inline void scan_load(uintx4 (&v)[4], const float* base, const unsigned (&off)[4]) {
  asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %4, %8 sc1\n\tglobal_load_dwordx4 %1, %5, %8 sc1\n\t"
               "global_load_dwordx4 %2, %6, %8 sc1\n\tglobal_load_dwordx4 %3, %7, %8 sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
               : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory");
}
__device__ inline void scan_load(uintx4 (&v)[8], const float* base, const unsigned (&off)[8]) {
  asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %8, %16 sc1\n\tglobal_load_dwordx4 %1, %9, %16 sc1\n\t"
               "global_load_dwordx4 %2, %10, %16 sc1\n\tglobal_load_dwordx4 %3, %11, %16 sc1\n\t"
               "global_load_dwordx4 %4, %12, %16 sc1\n\tglobal_load_dwordx4 %5, %13, %16 sc1\n\t"
               "global_load_dwordx4 %6, %14, %16 sc1\n\tglobal_load_dwordx4 %7, %15, %16 sc1\n\t"
               "s_waitcnt vmcnt(0)"
               : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]),
                 "=&v"(v[6]), "=&v"(v[7])
               : "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "v"(off[4]), "v"(off[5]),
                 "v"(off[6]), "v"(off[7]), "s"(base) : "memory");
}

// The address is the same in every lane of the wave; this puts it into scalar registers.
__device__ inline const float* scan_uniform(const float* p) {
  const unsigned long long b = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  return (const float*)(((unsigned long long)hi << 32) | lo);
}

__device__ inline int ctl_load(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
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
__device__ inline long long ticks() { return (long long)__builtin_amdgcn_s_memrealtime(); }

// A result that happens to be the sentinel (a NaN) is stored as another NaN.
__device__ inline unsigned scan_bits(float val) {
  const unsigned b = __float_as_uint(val);
  return b == SENTINEL ? 0x7fc00000u : b;
}
// Column l % 16 of quad column 0 gathers its quad: lanes with l % 4 == 0 hold four consecutive
// columns of a row and store them as one 16-byte access at agent scope.
__device__ inline void scan_store(float* p, float val, bool ok) {
  const unsigned b = scan_bits(val);
  uintx4 v;
  v[0] = b;
  v[1] = __builtin_amdgcn_mov_dpp(b, 0x55, 0xf, 0xf, true);   // quad_perm [1,1,1,1]
  v[2] = __builtin_amdgcn_mov_dpp(b, 0xaa, 0xf, 0xf, true);
  v[3] = __builtin_amdgcn_mov_dpp(b, 0xff, 0xf, 0xf, true);
  if (ok && (threadIdx.x & 3) == 0)
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// NCH: chunks of 64 k per wave; RB: groups of four rows per workgroup.  Registers: NG 16 NCH
// weights; one workgroup per CU is planned for (two waves per SIMD at eight waves).
// ITEMS: the workgroup takes (step, unit) items from the counter until none are left; otherwise it
// takes every step of the unit it was launched as, once all workgroups of the solve are resident, and
// leaves what remains to the launch with ITEMS behind it if they are not (see the top of the file).
template <int KIND, int NCH, int RB, class WT, bool ITEMS>
__global__ __launch_bounds__(64 * SCAN_MAXW, 2) void scan_kernel(ScanArgs a, int nrb) {
  constexpr int NG = ScanGates<KIND>::value;
  constexpr bool ADJ = KIND == SCAN_ADJOINT;
  constexpr int NS = ADJ ? 1 : NG;                    // sums an output needs
  constexpr int NL = RB * NCH;
  constexpr int NP = RB * NG == 1 ? 2 : 1;            // sums per gate and row group
  __shared__ float part[2][SCAN_MAXW][RB][NS][64];
  __shared__ int stop[2];
  __shared__ long long item;
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
  if (ITEMS) {
    if (ctl_load(a.ctl + 1) == 0) return;             // all were resident: the solve is done
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
    const int r0 = rb * RB * 4, j0 = cg * SCAN_CP;
    // weights: column j0 + lane % 16, k = kw0 + 64 c + 16 (lane / 16) + 0..15 (zero beyond H; columns
    // beyond H repeat the last one and are never stored)
    float w[NG][NCH][16];
    {
      const int j = min(j0 + (lane & 15), H - 1);
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int k = kw0 + 64 * c + 16 * (lane >> 4) + 4 * q;
            const int kc = min(k, H - 4);             // H is a multiple of 4
            const WT* p = (const WT*)a.Wt +
                          (ADJ ? (long long)j * 3 * H + g * H + kc : ((long long)g * H + j) * H + kc);
            const floatx4 v = k < H ? ldg4w(p) : zero4();
#pragma unroll
            for (int e = 0; e < 4; ++e) w[g][c][4 * q + e] = v[e];
          }
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
      for (int c = 0; c < NCH; ++c) off[r * NCH + c] = ((unsigned)row * W + kk[c]) * 4u;
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
        if constexpr (KIND == SCAN_GRU) {
          const float rg = sigmoidf_(cp[0] + s[0] + bias[0]);
          const float zg = sigmoidf_(cp[1] + s[1] + bias[1]);
          const float n = tanhf_(cp[2] + rg * (s[2] + bias[2]));
          const float c = a.gamma * (1.0f - zg);
          out = a.implicit_ ? (prev + c * n) * fast_rcp(1.0f + c) : prev + c * (n - prev);
        } else if constexpr (KIND == SCAN_LSTM) {
          const float ig = sigmoidf_(s[0] + cp[0] + bias[0]);
          const float fg = sigmoidf_(s[1] + cp[1] + bias[1]);
          const float gg = tanhf_(s[2] + cp[2] + bias[2]);
          const float og = sigmoidf_(s[3] + cp[3] + bias[3]);
          if (a.implicit_) {
            outc = (prevc + a.gamma * ig * gg) * fast_rcp(1.0f + a.gamma * (1.0f - fg));
            out = (prev + a.gamma * og * tanhf_(outc)) * fast_rcp(1.0f + a.gamma);
          } else {
            outc = prevc + a.gamma * (ig * gg - (1.0f - fg) * prevc);
            out = prev + a.gamma * (og * tanhf_(outc) - prev);
          }
          outc += cgc;
        } else if constexpr (KIND == SCAN_ODE) {
          out = prev + a.gamma * (sigmoidf_(s[0] + cp[0]) - 0.5f * prev);
        } else {
          out = ckd * prev + s[0];
        }
        out += cgv;
        float* dst = a.u + out_pt(i) * BW + eo;
        scan_store(dst, out, ok);
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

// Marks the points the solve will write and clears its control words.
__global__ __launch_bounds__(256) void scan_mark_kernel(uintx4* p, long long n4, int* ctl) {
  if (blockIdx.x == 0 && threadIdx.x < 4) ctl[threadIdx.x] = 0;
  const uintx4 s = {SENTINEL, SENTINEL, SENTINEL, SENTINEL};
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n4; i += 256LL * gridDim.x)
    p[i] = s;
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
struct ScanShape {
  int nch, nw, rb, nrb, ncg;
};
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
static ScanShape scan_shape(int B, int H) {
  const int max_wg = scan_max_wg();
  ScanShape s;
  s.nch = H > 64 * SCAN_MAXW ? 2 : 1;
  s.nw = (H + 64 * s.nch - 1) / (64 * s.nch);
  s.ncg = (H + SCAN_CP - 1) / SCAN_CP;
  const int quads = (B + 3) / 4;
  s.rb = 1;
  while (s.rb < 8 && (quads + s.rb - 1) / s.rb * s.ncg > max_wg) s.rb *= 2;
  s.nrb = (quads + s.rb - 1) / s.rb;
  if (s.nw < s.rb) s.nw = s.rb;                       // wave r finishes row group r
  return s;
}

// Up to 64 rows (the few-row range of the step kernels) of 16 to 1024 columns.  A solve costs
// three launches (mark, scan, items) whatever its length: below eight steps the chain of step launches
// is as fast.
bool scan_covers(int kind, long long N, int B, int H) {
  if (N < 8 || N > (1LL << 30) || B > 64 || H < 16 || H > 128 * SCAN_MAXW) return false;
  const ScanShape s = scan_shape(B, H);
  // registers: the adjoint holds three coefficient rows per state row, the LSTM four gates
  const int limit = kind == SCAN_ADJOINT && s.nch == 2 ? 2 : 4;
  return s.rb <= limit && s.nrb * s.ncg <= scan_max_wg();
}

template <int KIND, int NCH, int RB, class WT>
static void launch_scan_shape(const ScanArgs& a, dim3 grid, dim3 block, int nrb, hipStream_t st) {
  hipLaunchKernelGGL((scan_kernel<KIND, NCH, RB, WT, false>), grid, block, 0, st, a, nrb);
  hipLaunchKernelGGL((scan_kernel<KIND, NCH, RB, WT, true>), grid, block, 0, st, a, nrb);
}
template <int KIND, class WT>
static void launch_scan_kind(const ScanArgs& a, hipStream_t st) {
  const ScanShape s = scan_shape(a.B, a.H);
  const dim3 grid((unsigned)(s.nrb * s.ncg)), block(64 * s.nw);
#define MG_SCAN_CASE(NCH, RB)                                                                  \
  if (s.nch == NCH && s.rb == RB)                                                              \
    launch_scan_shape<KIND, NCH, RB, WT>(a, grid, block, s.nrb, st);
  MG_SCAN_CASE(1, 1)
  MG_SCAN_CASE(1, 2)
  MG_SCAN_CASE(1, 4)
  MG_SCAN_CASE(2, 1)
  MG_SCAN_CASE(2, 2)
  if constexpr (KIND != SCAN_ADJOINT) {
    MG_SCAN_CASE(2, 4)
  }
#undef MG_SCAN_CASE
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
  const long long n4 = (long long)a.N * a.B * W / 4;
  const long long nb = (n4 + 255) / 256;
  hipLaunchKernelGGL(scan_mark_kernel, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256), 0, st,
                     (uintx4*)(a.u + (kind == SCAN_ADJOINT ? 0 : (long long)a.B * W)), n4, a.ctl);
  const bool h16 = a.bf16 == 1;
  if (kind == SCAN_GRU) {
    if (h16) launch_scan_kind<SCAN_GRU, bf16_t>(a, st);
    else launch_scan_kind<SCAN_GRU, float>(a, st);
  } else if (kind == SCAN_ADJOINT) {
    if (h16) launch_scan_kind<SCAN_ADJOINT, bf16_t>(a, st);
    else launch_scan_kind<SCAN_ADJOINT, float>(a, st);
  } else if (kind == SCAN_LSTM) {
    launch_scan_kind<SCAN_LSTM, float>(a, st);
  } else {
    launch_scan_kind<SCAN_ODE, float>(a, st);
  }
  const double rows = (double)a.N * a.B;
  const int ng = kind == SCAN_LSTM ? 4 : kind == SCAN_ODE ? 1 : 3;
  const double bytes = kind == SCAN_ADJOINT ? 28.0 : kind == SCAN_GRU ? 20.0 : kind == SCAN_LSTM ? 32.0 : 16.0;
  prof_end(prof, 2.0 * ng * rows * a.H * a.H, bytes * rows * a.H, st);
  return hipGetLastError();
}

}  // namespace mg

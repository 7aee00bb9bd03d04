// What the two forms of the one-launch serial solves share (kernels_scan.hip, kernels_scan_xcd.hip):
// shapes, the words they exchange, polling loads and the elements they compute.
#pragma once
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
// quarter of a solve through memory, a fifth to a half of one inside the XCDs), 50 us (several times what an arrival on a free GPU takes) to 5 ms.
constexpr long long SCAN_ARRIVE_PER_STEP = 50, SCAN_ARRIVE_MIN = 5000, SCAN_ARRIVE_MAX = 500000;
constexpr long long SCAN_STEP_TICKS = 200000000;     // 2 s: bound of a single wait, all resident
constexpr int SCAN_MAX_POLLS = 1 << 24;              // the same, items from the counter (counted in
                                                     // polls: a GPU that is taken away counts none)

constexpr int SCAN_XCDS = 8, SCAN_XCD_CUS = 32;
// How a solve is cut into workgroups.
struct ScanShape {
  int rb, nrb;         // row quads per row block, row blocks
  int ncg;             // column groups
  int nch, nw;         // kernels_scan.hip: chunks of 64 k per wave, waves that split K
  int ct, hp;          // kernels_scan_xcd.hip: tiles of 16 columns per workgroup, columns of a ring row
                       // (256, 512 or 1024)
  int gpx, nx;         // row blocks per XCD, XCDs needed
  int terms;           // the contraction is on terms (ScanArgs)
};
// control words beyond the four of ScanArgs: XCDs given away (xcd_groups), a wait passed its bound,
// workgroups that have arrived per XCD
constexpr int CTL_WORD = 4, CTL_ABORT = 5, CTL_TICKETS = 8, CTL_WORDS = 16;

template <int KIND>
struct ScanGates {
  static constexpr int value = KIND == SCAN_LSTM ? 4 : KIND == SCAN_ODE ? 1 : 3;
};

// Vectors of a state row that the contraction reads (adjoint: products with the coefficients).
template <int KIND>
struct ScanVectors {
  static constexpr int value = KIND == SCAN_ADJOINT ? 3 : 1;
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

__device__ inline long long ticks() { return (long long)__builtin_amdgcn_s_memrealtime(); }

__device__ inline int ctl_load(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A result that happens to be the sentinel (a NaN) is stored as another NaN.
__device__ inline unsigned scan_bits(float val) {
  const unsigned b = __float_as_uint(val);
  return b == SENTINEL ? 0x7fc00000u : b;
}
// Column l % 16 of quad column 0 gathers its quad: lanes with l % 4 == 0 hold four consecutive
// columns of a row, for one 16-byte store.
__device__ inline uintx4 scan_quad(float val) {
  const unsigned b = scan_bits(val);
  uintx4 v;
  v[0] = __builtin_amdgcn_mov_dpp(b, 0x00, 0xf, 0xf, true);   // quad_perm [0,0,0,0]
  v[1] = __builtin_amdgcn_mov_dpp(b, 0x55, 0xf, 0xf, true);
  v[2] = __builtin_amdgcn_mov_dpp(b, 0xaa, 0xf, 0xf, true);
  v[3] = __builtin_amdgcn_mov_dpp(b, 0xff, 0xf, 0xf, true);
  return v;
}
// Exact terms of a state value on the bf16 matrix pipe, whose 16 rows hold four state rows three times:
// row 4 t + r is term t of row r, rows 12..15 are zero.  x = t0 + 2^-8 t1 + 2^-16 t2, each term eight bits
// of the value (cut, not rounded: nothing overflows, and the scaled lower terms have the exponent of the
// value, so that none of them is subnormal where the value is not).  Not finite: the first alone.
struct StateTerms {
  unsigned t01, t2;                                    // bf16 t0 (low half) and t1; t2
};
__device__ inline StateTerms state_terms(float x) {
  const unsigned b = x == x ? __float_as_uint(x) : 0x7fc00000u;    // (no bf16 pair is SENTINEL)
  const bool finite = (b & 0x7f800000u) != 0x7f800000u;
  const float r1 = (x - __uint_as_float(b & 0xffff0000u)) * 256.f;
  const unsigned b1 = finite ? __float_as_uint(r1) : 0u;
  const float r2 = (r1 - __uint_as_float(b1 & 0xffff0000u)) * 256.f;
  const unsigned b2 = finite ? __float_as_uint(r2) : 0u;
  return {(b >> 16) | (b1 & 0xffff0000u), b2 >> 16};
}
// Sum of the terms' rows of a 16 x 16 block: as quad_fold, with the weights of the terms.
__device__ inline float term_fold(const floatx4& a) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  auto u = [](float f) { return __float_as_uint(f); };
  auto fold = [](u2 s, float w) { return fmaf(__uint_as_float(s[1]), w, __uint_as_float(s[0])); };
  const float x01 = fold(__builtin_amdgcn_permlane32_swap(u(a[0]), u(a[1]), false, false), 0x1p-16f);
  const float x23 = fold(__builtin_amdgcn_permlane32_swap(u(a[2]), u(a[3]), false, false), 0x1p-16f);
  return fold(__builtin_amdgcn_permlane16_swap(u(x01), u(x23), false, false), 0x1p-8f);
}
__device__ inline floatx4 term_mma(const uintx4& state, const bf16x8& w, const floatx4& acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, state), w, acc, 0, 0, 0);
}
// Weights of a block of 32 k: column l % 16, k = 8 (l / 16) + 0..7; zero beyond H (a multiple of 8).
__device__ inline bf16x8 term_weights(const bf16_t* row, int k, int H) {
  const bf16x8 v = ldg8h(row + min(k, H - 8));
  return k < H ? v : __builtin_bit_cast(bf16x8, uintx4{0, 0, 0, 0});
}
// Whether a weight of the wave is infinite (the same answer in every lane): its product with a zero term,
// which most states have, is NaN, so terms cannot carry it, and fp32 MFMAs contract in their place.
template <int NB, int NQ>
__device__ inline bool term_weights_infinite(const bf16x8 (&w)[NB][NQ]) {
  bool inf = false;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const uintx4 v = __builtin_bit_cast(uintx4, w[b][q]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        inf |= (v[e] & 0x7fffu) == 0x7f80u || (v[e] & 0x7fff0000u) == 0x7f800000u;
    }
  return __any(inf);
}

__device__ inline void scan_store_agent(float* p, uintx4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}
// Row-block groups that have been given to XCDs, from the word that records them: four bits per XCD,
// 1 + the group, 0 not decided, XCD_CLOSED not to be used any more.
constexpr unsigned XCD_CLOSED = 15;
__device__ inline int xcd_groups(unsigned word) {
  int n = 0;
  for (int x = 0; x < SCAN_XCDS; ++x) {
    const unsigned v = (word >> (4 * x)) & 15;
    n += v != 0 && v != XCD_CLOSED;
  }
  return n;
}

// The new element of a state row from its sums over K.
//   s: recurrent sums (adjoint: one), p: projection row, kd: direct coefficient (adjoint), prev, prevc: the
//   element of the row the step starts from, g, gc: right-hand side (c: the LSTM's cell half)
template <int KIND, int NS, int NG>
__device__ inline void scan_element(const ScanArgs& a, const float (&s)[NS], const float (&p)[NG],
                                    const float (&bias)[NG], float kd, float prev, float prevc, float g,
                                    float gc, float& out, float& outc) {
  if constexpr (KIND == SCAN_GRU) {
    const float rg = sigmoidf_(p[0] + s[0] + bias[0]);
    const float zg = sigmoidf_(p[1] + s[1] + bias[1]);
    const float n = tanhf_(p[2] + rg * (s[2] + bias[2]));
    const float c = a.gamma * (1.0f - zg);
    out = a.implicit_ ? (prev + c * n) * fast_rcp(1.0f + c) : prev + c * (n - prev);
  } else if constexpr (KIND == SCAN_LSTM) {
    const float ig = sigmoidf_(s[0] + p[0] + bias[0]);
    const float fg = sigmoidf_(s[1] + p[1] + bias[1]);
    const float gg = tanhf_(s[2] + p[2] + bias[2]);
    const float og = sigmoidf_(s[3] + p[3] + bias[3]);
    if (a.implicit_) {
      outc = (prevc + a.gamma * ig * gg) * fast_rcp(1.0f + a.gamma * (1.0f - fg));
      out = (prev + a.gamma * og * tanhf_(outc)) * fast_rcp(1.0f + a.gamma);
    } else {
      outc = prevc + a.gamma * (ig * gg - (1.0f - fg) * prevc);
      out = prev + a.gamma * (og * tanhf_(outc) - prev);
    }
    outc += gc;
  } else if constexpr (KIND == SCAN_ODE) {
    out = prev + a.gamma * (sigmoidf_(s[0] + p[0]) - 0.5f * prev);
  } else {
    out = kd * prev + s[0];
  }
  out += g;
}

// The form with a row block per XCD; a.ring and a.ring4 are set.
hipError_t launch_scan_xcd(int kind, const ScanArgs& a, const ScanShape& s, hipStream_t st);

}  // namespace mg

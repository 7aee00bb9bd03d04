// Workgroup-tile product of fp32 VALUES on the 16-bit matrix pipe, for the step kernels and the input
// gradients (the weight gradients take their terms from here too): the "NT" tile product of gemm_core.h with each operand carried as two fp16 terms,
// a = a0 + a1 (22 mantissa bits), consumed by v_mfma_f32_16x16x32_f16 as a0*b0 + a1*b0 + a0*b1.
//
// Accuracy.  What the terms and the dropped a1*b1 leave out is about 6e-8 of a product, of either
// sign; the matrix pipe itself cuts off below the last bit of every sum it forms, so three products
// are closer to the exact sum than the six that three bf16 terms take, and than the fp32 MFMAs.
// Error against 64 bits, states against Xavier weights (two fp16 terms : three bf16 terms : fp32
// MFMA): 512 columns 2.6e-7 : 3.5e-7 : 2.9e-7, 1024 columns 3.6 : 4.9 : 4.1, 1536 columns
// 4.4 : 5.9 : 4.9.  (The projection keeps three bf16 terms with the lower products summed apart,
// gemm_core_bf16.h: 1.8e-7 over 1024 columns, 2.2e-7 with fp16 terms in that form.  Summed 128 columns
// at a time two fp16 terms reach 1.6e-7 there and half the time, but the states that follow end up
// further off, 2.07e-7 against 1.77e-7: few large errors become many small ones.)
//
// Range.  fp16 has five exponent bits, so every row of an operand is scaled by a power of two of its
// own and the sums back, exactly: the rows of B, split once per call, by their largest value; a row of
// A, split on its way to LDS, by the largest value of its first K-slice, which leaves the rest of the
// row a factor of 2^9.  A row whose first slice is zero is scaled by 2^127: rows of zeros (H0, zero
// guesses) and adjoints that have decayed to the smallest numbers are carried like that, anything else
// overflows.  The rows of a tile with a sum that is not finite are read through for their largest
// values; one that still has such a sum holds an operand that is not finite itself and is contracted
// in fp32.  (Reading through every row that starts with zeros took 35 us in one tile of ten of an
// adjoint over 2048 steps.)  Subnormal terms keep their bits on this pipe;
// what is below them is 2^-31 of the row's largest value.
//
// What is left out is thus bounded by 2^-22 of a value where it is within 2^9 of its row's largest and by 2^-31 of
// that largest below: an element of a product whose row of B is zero wherever the row of A is not small (two
// nets of different scale side by side in one layer) has fewer digits than in fp32.  Every row of a dense
// B sees the large elements too.
//
// Data path (16384 rows x 512, the level step: 145 us with three bf16 terms, 118 with two fp16 terms in
// the loop of gemm_core_bf16.h, 91 this way; 16384 LSTM rows 243, 157, 126).  With half the MFMAs the K loop is bound by what feeds them, LDS above all: 32x32 blocks
// of A and B fragments read by every wave cost 105 of the LDS's 128 bytes per clock at full matrix
// rate for the 128 x 64 (x3) tile.  So B does not pass through LDS: the split leaves it in the order in
// which lanes take it (term_pack.h), a wave owns its columns alone (the waves of a tile lie side by
// side) and loads its fragments straight into registers, one slice ahead.  A goes to LDS in fragment
// order too, in three slices taking turns, so that a slice costs one barrier, its conversion and writes
// go between the MFMAs of an earlier one, and its first fragments are read before the barrier.
#pragma once
#include "gemm_core_bf16.h"
#include "term_pack.h"

namespace mg {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Two floats rounded to fp16 (a in the low half); what their roundings leave.
__device__ inline unsigned round2_f16(float a, float b) {
  typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
  typedef float floatx2 __attribute__((ext_vector_type(2)));
  const floatx2 v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, f16x2));
}
// (one mixed-precision instruction each: the half is read as it is and negated)
__device__ inline void minus2_f16(float& a, float& b, unsigned r) {
  asm("v_fma_mix_f32 %0, %1, -1.0, %0 op_sel_hi:[1,0,0]" : "+v"(a) : "v"(r));
  asm("v_fma_mix_f32 %0, %1, -1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(b) : "v"(r));
}
// Terms of pair i (0..3) of eight values: t0 + t1 = v f up to 2^-22.
struct Words8 {
  unsigned t[3][4];                // eight values' terms, two to a word
};
__device__ inline void split_pair(const F32x8& v, int i, float f, Words8& w) {
  float a = (i < 2 ? v.lo4[2 * i] : v.hi4[2 * i - 4]) * f;
  float b = (i < 2 ? v.lo4[2 * i + 1] : v.hi4[2 * i - 3]) * f;
  w.t[0][i] = round2_f16(a, b);
  minus2_f16(a, b, w.t[0][i]);
  w.t[1][i] = round2_f16(a, b);
}
// The same in three bf16 terms, exactly (gemm_core_bf16.h).
__device__ inline void split_pair_bf16(const F32x8& v, int i, float f, Words8& w) {
  float a = (i < 2 ? v.lo4[2 * i] : v.hi4[2 * i - 4]) * f;
  float b = (i < 2 ? v.lo4[2 * i + 1] : v.hi4[2 * i - 3]) * f;
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    w.t[t][i] = round2_bf16(a, b);
    if (t < 2) minus2_bf16(a, b, w.t[t][i]);
  }
}
__device__ inline f16x8 words8(const unsigned (&w)[4]) {
  typedef unsigned uintx4_ __attribute__((ext_vector_type(4)));
  const uintx4_ v = {w[0], w[1], w[2], w[3]};
  return __builtin_bit_cast(f16x8, v);
}
__device__ inline float top8(float m, const F32x8& v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) m = fmaxf(m, fmaxf(fabsf(v.lo4[i]), fabsf(v.hi4[i])));
  return m;
}
// Exponent by which a row with the largest magnitude m is scaled: m lands in [2^top, 2^(top+1)).  (At
// most 2^127, the largest power of two there is: rows below 2^(top-127) end lower, a row of 2^-126 at
// 2, with 2^-26 of its largest value left out.)
__device__ inline int term_exponent(float m, int top) {
  return min(top + 127 - (int)(__float_as_uint(m) >> 23), 127);
}
__device__ inline float exp2_int(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }
constexpr int TERM_TOP_A = 6, TERM_TOP_B = 13;

__device__ inline const int* pack_exponents(const void* pack, long long rows, int K) {
  return reinterpret_cast<const int*>((const char*)pack + pack_exponents_at(rows, K));
}

// How the waves of configuration C (NP = 3) share a tile: WR x WC waves per K-split group, each RB x CB
// blocks of 16 x 16 (x NG).
template <class C>
struct TermGeom {
  static constexpr int NW = C::WM * C::WN;
  static constexpr int WR = NW > 4 && C::TN <= 128 ? 2 : 1, WC = NW / WR;
  static constexpr int RB = C::TM / 16 / WR, CB = C::TN / 16 / WC;
  static constexpr int NF = C::NG * CB;                   // B fragments per term and slice
  // terms per operand: with LOSUM three bf16 terms and six products, the lower five summed apart
  static constexpr bool X3 = C::LOSUM;
  static constexpr int NTM = X3 ? 3 : 2;
  static constexpr int GB = NF >= 3 || X3 ? 1 : 2;        // row blocks whose MFMAs alternate
  static constexpr int BLK = C::TM / 16;                  // row blocks of the tile
  static constexpr int BUF = C::KS * NTM * BLK * 64;        // 16-byte chunks of one slice of A
  static_assert(RB * WR * 16 == C::TM && CB * WC * 16 == C::TN, "waves must cover the tile");
  static_assert(C::TK == 32 * C::KS && RB % GB == 0, "");
};
template <class C>
struct TermAcc {
  typedef TermGeom<C> G;
  floatx4 v[G::RB][C::NG][G::CB];
  __device__ inline void zero() {
#pragma unroll
    for (int r = 0; r < G::RB; ++r)
#pragma unroll
      for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int c = 0; c < G::CB; ++c) v[r][g][c] = zero4();
  }
};
// Position of the calling wave and lane in a tile.
template <class C>
struct TermLane {
  typedef TermGeom<C> G;
  int ks, row0, col0, li, lq;      // first row and column of the wave; lane % 16, lane / 16
  __device__ inline TermLane() {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    ks = wave / G::NW;
    row0 = (wave % G::NW) / G::WC * G::RB * 16;
    col0 = (wave % G::NW) % G::WC * G::CB * 16;
    li = threadIdx.x & 15;
    lq = (threadIdx.x >> 4) & 3;
  }
};

// First k of slice i of a pass over K in memory order.
template <class C>
struct InOrder {
  __device__ inline int operator()(int i) const { return i * C::TK; }
};

// Largest m of the CPR lanes that share a row (neighbours).
template <class C>
__device__ inline float over_row(float m) {
#pragma unroll
  for (int o = 1; o < C::CPR; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  return m;
}
// Largest magnitude over the row behind chunk s of the calling thread: load(k), columns k..k+7 of the row, K of
// them.  Eight slices' loads at a time.
template <class C, class Load>
__device__ inline float row_top(int s, int K, Load load) {
  float m = 0.f;
  for (int k = (threadIdx.x + s * C::NT) % C::CPR * 8; k < K; k += 8 * C::TK) {
    F32x8 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = load(min(k + u * C::TK, K - 8));
#pragma unroll
    for (int u = 0; u < 8; ++u) m = top8(m, v[u]);
  }
  return over_row<C>(m);
}

// One pass over K (a multiple of 8).  loadA, finA: as in gemm_nt_tile_bf16, called slice after slice;
// order(i): first k of the i-th slice; top(s): row_top of the row behind chunk s; brow(g, c): packed row
// (g, column c of the tile) of B; rowexp: LDS, receives the exponents the tile rows of A are scaled
// by; through: find them from whole rows, not from first slices.
template <class C, class LoadA, class Top, class FinA, class Order, class BRow>
__device__ inline void gemm_nt_tile_terms(TermAcc<C>& acc, int K, LoadA loadA, Top top, FinA finA,
                                          Order order, const char* pack, BRow brow, f16x8* lds,
                                          int* rowexp, bool through) {
  typedef TermGeom<C> G;
  const int tid = threadIdx.x;
  const TermLane<C> me;
  decltype(loadA(0, 0)) ra[C::A_CHUNKS], ra1[C::A_CHUNKS];       // (ra1: prologue only)
  auto load_a = [&](int s, int k0) {
    return loadA(s, min(k0 + ((tid + s * C::NT) % C::CPR) * 8, K - 8));
  };
  // (32-bit offsets: launches on terms keep their packs below 4 GB)
  unsigned bo[C::NG][G::CB];
#pragma unroll
  for (int g = 0; g < C::NG; ++g)
#pragma unroll
    for (int c = 0; c < G::CB; ++c)
      bo[g][c] = (unsigned)pack_row(brow(g, me.col0 + c * 16 + me.li), K, G::NTM);
  f16x8 rb[2][G::NTM][C::NG][G::CB];                 // [slice % 2][term]
  constexpr int NLB = G::NTM * C::NG * G::CB, PACK_K8 = PACK_TERM * G::NTM;        // loads of B per slice
  auto fetch_b = [&](int d, int j, int k0) {
    const int g = j / G::NTM / G::CB, c = j / G::NTM % G::CB, t = j % G::NTM;
    // (columns beyond K, a whole K-split group of them in the last slice: those of the last k / 8)
    const int k8 = min(k0 / 8 + me.ks * 4, K / 8 - 1);
    const unsigned lane = (unsigned)min(me.lq, K / 8 - 1 - k8) * PACK_K8;
    rb[d][t][g][c] = *reinterpret_cast<const f16x8*>(pack + (long long)k8 * PACK_K8 +
                                                     t * PACK_TERM + (bo[g][c] + lane));
  };
  // scale of the row behind each chunk; odd tile rows enter with the opposite sign (see contract_terms)
  float rowscale[C::A_CHUNKS];
  auto scale_rows = [&]() {
#pragma unroll
    for (int s = 0; s < C::A_CHUNKS; ++s) {
      const int q = tid + s * C::NT;
      if constexpr (G::X3) {
        rowscale[s] = (q / C::CPR) & 1 ? -SPLIT3_SCALE : SPLIT3_SCALE;
        continue;
      }
      float m = over_row<C>(top8(0.f, finA(ra[s])));
      if (through) m = top(s);
      const int e = term_exponent(m, TERM_TOP_A);
      rowscale[s] = (q / C::CPR) & 1 ? -exp2_int(e) : exp2_int(e);
      if (q % C::CPR == 0) rowexp[q / C::CPR] = e;
    }
  };
  // A in LDS: [slice % 3][K-split group][term][row block][k / 8][row % 16], the rows of a k / 8 exchanged
  // by it and by the group, so that eight lanes (two rows, or one of both groups) write to different banks
  Words8 aw[C::A_CHUNKS];
  auto convert = [&](int j, int k0) {           // pair j of the thread's 4 A_CHUNKS
    const int s = j / 4, c = (tid + s * C::NT) % C::CPR;
    // (columns beyond K: zeros, or what makes the tile one that is not finite)
    const float f = k0 + c * 8 < K ? rowscale[s] : 0.f;
    if constexpr (G::X3)
      split_pair_bf16(finA(ra[s]), j % 4, f, aw[s]);
    else
      split_pair(finA(ra[s]), j % 4, f, aw[s]);
  };
  auto stash = [&](int p, int s) {
    const int q = tid + s * C::NT, row = q / C::CPR, c = q % C::CPR;
    const int at = p * G::BUF + (c / 4) * G::NTM * G::BLK * 64 + (row / 16) * 64 + (c % 4) * 16 +
                   ((row & 15) ^ (2 * (c % 4)) ^ (c / 4));
#pragma unroll
    for (int t = 0; t < G::NTM; ++t) lds[at + t * G::BLK * 64] = words8(aw[s].t[t]);
  };
  const int a_at = me.ks * G::NTM * G::BLK * 64 + (me.row0 / 16) * 64 + me.lq * 16 +
                   (me.li ^ (2 * me.lq) ^ me.ks);
  auto read_a = [&](int p, int r, int t) {
    return lds[p * G::BUF + a_at + t * G::BLK * 64 + r * 64];
  };
  typedef f16x8 Frags[G::NTM][G::GB];                // [term][row block]
  auto read_group = [&](int p, int r0, Frags& f) {
#pragma unroll
    for (int i = 0; i < G::GB; ++i)
#pragma unroll
      for (int t = 0; t < G::NTM; ++t) f[t][i] = read_a(p, r0 + i, t);
  };
  TermAcc<C> lo;                                // (X3: the lower products)
  if constexpr (G::X3) lo.zero();
  auto multiply = [&](int d, int r0, const Frags& f) {
    if constexpr (G::X3) {
      auto mm = [&](TermAcc<C>& sum, int t, int u) {
#pragma unroll
        for (int g = 0; g < C::NG; ++g)
#pragma unroll
          for (int c = 0; c < G::CB; ++c)
            sum.v[r0][g][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, f[t][0]), __builtin_bit_cast(bf16x8, rb[d][u][g][c]),
                sum.v[r0][g][c], 0, 0, 0);
      };
      mm(lo, 2, 0);
      mm(acc, 0, 0);
      mm(lo, 1, 0);
      mm(lo, 0, 1);
      mm(lo, 1, 1);
      mm(lo, 0, 2);
      return;
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)                // a0 b0, a1 b0, a0 b1
#pragma unroll
      for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int c = 0; c < G::CB; ++c)
#pragma unroll
          for (int i = 0; i < G::GB; ++i)
            acc.v[r0 + i][g][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                f[u == 1][i], rb[d][u == 2][g][c], acc.v[r0 + i][g][c], 0, 0, 0);
  };
  const int nkt = (K + C::TK - 1) / C::TK;
  // k of the slices kt + 1, kt + 2, kt + 3 (beyond the last slice: that one again, not used)
  int o1 = order(min(1, nkt - 1)), o2 = order(min(2, nkt - 1)), o3 = order(min(3, nkt - 1));
  const int o0 = order(0);
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) ra[s] = load_a(s, o0);
#pragma unroll
  for (int s = 0; s < C::A_CHUNKS; ++s) ra1[s] = load_a(s, o1);
#pragma unroll
  for (int j = 0; j < NLB; ++j) fetch_b(0, j, o0);
  __builtin_amdgcn_sched_barrier(0);            // (all of them in flight before the first is waited for)
  scale_rows();
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int s = 0; s < C::A_CHUNKS; ++s) {
#pragma unroll
      for (int i = 0; i < 4; ++i) convert(4 * s + i, n ? o1 : o0);
      stash(n, s);
      ra[s] = n ? load_a(s, o2) : ra1[s];
    }
  __syncthreads();
  // Slice kt.  The fragments of a group of row blocks are read while the group before is multiplied, across
  // the barrier too: slice kt + 1 has been in LDS since the barrier before this slice.  Everything
  // else is dealt out over the groups, since the waves of a workgroup come to the same point together:
  // the loads of B for the next slice over the first three quarters (they queue at the CU's one
  // address unit: all at once they held the waves up for 500 to 900 clocks), the conversion of
  // slice kt + 2, in registers since the slice before, pair by pair.
  Frags f[2];
  constexpr int NGRP = G::RB / G::GB, NPAIR = 4 * C::A_CHUNKS;
  constexpr int BGRP = NGRP * 3 / 4 > 0 ? NGRP * 3 / 4 : 1;
  static_assert(NGRP % 2 == 0, "a slice starts on the first set of fragments");
  int p = 0, p1 = 1, p2 = 2;                     // LDS buffers of slices kt, kt + 1, kt + 2
  auto slice = [&](auto d_tag, int kt) {
    constexpr int d = decltype(d_tag)::value;    // kt % 2
#pragma unroll
    for (int i = 0; i < NGRP; ++i) {
      if (i + 1 < NGRP)
        read_group(p, (i + 1) * G::GB, f[(i + 1) & 1]);
      else
        read_group(p1, 0, f[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NLB; ++j)
        if (j * BGRP / NLB == i) fetch_b(d ^ 1, j, o1);
      multiply(d, i * G::GB, f[i & 1]);
#pragma unroll
      for (int j = 0; j < NPAIR; ++j)
        if (j * NGRP / NPAIR == i) {
          convert(j, o2);
          if (j % 4 == 3) {
            stash(p2, j / 4);
            ra[j / 4] = load_a(j / 4, o3);
          }
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const int t = p;
    p = p1;
    p1 = p2;
    p2 = t;
    o1 = o2;
    o2 = o3;
    o3 = order(min(kt + 4, nkt - 1));
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  read_group(p, 0, f[0]);
  int kt = 0;
  for (; kt + 1 < nkt; kt += 2) {
    slice(even, kt);
    slice(odd, kt + 1);
  }
  if (kt < nkt) slice(even, kt);
  if constexpr (G::X3) {
#pragma unroll
    for (int r = 0; r < G::RB; ++r)
#pragma unroll
      for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int c = 0; c < G::CB; ++c) {
          acc.v[r][g][c] += lo.v[r][g][c];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc.v[r][g][c][e] *= e & 1 ? -SPLIT3_UNSCALE : SPLIT3_UNSCALE;
        }
  }
}

// Whether any sum of the workgroup's tile is not finite (the same answer in every thread).  A value
// that fp16 rounds to an infinity has a second term of the opposite sign, so a sum of terms shows any
// operand it cannot carry.
template <class C>
__device__ inline bool tile_not_finite(const TermAcc<C>& acc) {
  floatx4 t = zero4();                          // (four chains: one of 96 waits for each link)
#pragma unroll
  for (int r = 0; r < TermGeom<C>::RB; ++r)
#pragma unroll
    for (int g = 0; g < C::NG; ++g)
#pragma unroll
      for (int c = 0; c < TermGeom<C>::CB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = fmaf(acc.v[r][g][c][e], 0.f, t[e]);
  const float u = (t[0] + t[1]) + (t[2] + t[3]);
  return __syncthreads_or(u != u) != 0;
}
// acc = A * B^T in fp32, operands straight from memory (small rather than fast: only tiles with
// sums that are not finite come here).  load_a(r, k): columns k..k+3 of tile row r of A; frow(g, c): row
// (g, column c of the tile) of B.  K a multiple of 4.
template <class C, class LoadA4, class FRow>
__device__ inline void contract_f32(TermAcc<C>& acc, int K, LoadA4 load_a, FRow frow) {
  typedef TermGeom<C> G;
  const TermLane<C> me;
  acc.zero();
#pragma unroll 1
  for (int k0 = 16 * me.ks; k0 < K; k0 += 16 * C::KS) {
    const int k = k0 + 4 * me.lq, kc = k < K ? k : K - 4;
    floatx4 fb[C::NG][G::CB];
#pragma unroll
    for (int g = 0; g < C::NG; ++g)
#pragma unroll
      for (int c = 0; c < G::CB; ++c)
        fb[g][c] = k < K ? ldg4(frow(g, me.col0 + c * 16 + me.li) + kc) : zero4();
#pragma unroll
    for (int r = 0; r < G::RB; ++r) {
      const floatx4 fa = k < K ? load_a(me.row0 + r * 16 + me.li, kc) : zero4();
#pragma unroll
      for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int c = 0; c < G::CB; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc.v[r][g][c] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(fa[e], fb[g][c][e], acc.v[r][g][c], 0, 0, 0);
    }
  }
}

// acc = A * B^T on terms.  la, top, fa, order: as in gemm_nt_tile_terms; pack, rows: the packed terms of B
// (launch_split2) and its rows; brow(g, c): row of B behind column c of the tile, gate g; load_a, frow: as
// in contract_f32.  The MFMA rounds its sum down (towards minus infinity) below the last bit, the same
// way in every row: sums over rows (bias gradients, residual norms) would collect it, with the sign of
// the odd rows turned it alternates instead (bias gradients at 12800 rows x 1000, three bf16 terms:
// 4.3e-7 off with the signs as they are, 2.9e-7 with fp32 MFMAs).
template <class C, class LoadA, class Top, class FinA, class BRow, class LoadA4, class FRow,
          class Order = InOrder<C>>
__device__ inline void contract_terms(TermAcc<C>& acc, int K, LoadA la, Top top, FinA fa,
                                      const void* pack, long long rows, BRow brow, void* lds,
                                      LoadA4 load_a, FRow frow, Order order = InOrder<C>()) {
  typedef TermGeom<C> G;
  __shared__ __attribute__((aligned(16))) int rowexp[C::TM];
  const TermLane<C> me;
  int ce[C::NG][G::CB];
#pragma unroll
  for (int g = 0; g < C::NG; ++g)
#pragma unroll
    for (int c = 0; c < G::CB; ++c)
      ce[g][c] = pack_exponents(pack, rows, K)[brow(g, me.col0 + c * 16 + me.li)];
#pragma unroll 1
  for (int through = 0; through < 2; ++through) {
    acc.zero();
    gemm_nt_tile_terms<C>(acc, K, la, top, fa, order, (const char*)pack, brow, (f16x8*)lds,
                          rowexp, through != 0);
#pragma unroll
    for (int r = 0; r < G::RB; ++r) {
      typedef int intx4_ __attribute__((ext_vector_type(4)));
      const intx4_ re = *reinterpret_cast<const intx4_*>(&rowexp[me.row0 + r * 16 + 4 * me.lq]);
#pragma unroll
      for (int g = 0; g < C::NG; ++g)
#pragma unroll
        for (int c = 0; c < G::CB; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = acc.v[r][g][c][e];
            acc.v[r][g][c][e] = ldexpf(e & 1 ? -v : v, -re[e] - ce[g][c]);
          }
    }
    if (!tile_not_finite<C>(acc)) return;
  }
  contract_f32<C>(acc, K, load_a, frow);
}

// Staging for the epilogue (EpiStage::write) of sums in this layout.
template <class C>
__device__ inline void stage_write_terms(const TermAcc<C>& acc, int ba, float* stage) {
  typedef TermGeom<C> G;
  typedef EpiStage<C> E;
  const TermLane<C> me;
#pragma unroll
  for (int r = 0; r < G::RB; ++r) {
    // 32-row group of the tile; pass ba stages the groups ba, ba + BM, ...
    if constexpr (G::WR > 1) static_assert(C::BM == 1, "");
    if (G::WR == 1 && (r / 2) % C::BM != ba) continue;
    const int grp = (me.row0 / 16 + r) / 2;
    const int row = grp / C::BM * 32 + (r & 1) * 16 + 4 * me.lq;
#pragma unroll
    for (int g = 0; g < C::NG; ++g)
#pragma unroll
      for (int c = 0; c < G::CB; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          stage[me.ks * E::SLAB + (g * E::ROWS + row + e) * E::LD + me.col0 + c * 16 + me.li] =
              acc.v[r][g][c][e];
  }
}

// The same on three bf16 terms (LOSUM).
template <class C, class LoadA, class FinA, class BRow, class LoadA4, class FRow>
__device__ inline void contract_terms_x3(TermAcc<C>& acc, int K, LoadA la, FinA fa, const void* pack,
                                         BRow brow, void* lds, LoadA4 load_a, FRow frow) {
  acc.zero();
  gemm_nt_tile_terms<C>(acc, K, la, [](int) { return 0.f; }, fa, InOrder<C>(), (const char*)pack,
                        brow, (f16x8*)lds, nullptr, false);
  if (tile_not_finite<C>(acc)) contract_f32<C>(acc, K, load_a, frow);
}

// Stores the tile of a plain GEMM: out[m, n] + bias[n], leading dimension N.  A wave's two column blocks
// exchange every other quad of rows first, so that a store covers whole 128-byte lines of two rows (lines
// in halves: 559 MB written where 403 are the projection of 65536 x 1536).
template <class C>
__device__ inline void store_tile_terms(const TermAcc<C>& acc, float* out, const float* bias,
                                        long long m0, int n0, long long M, int N) {
  typedef TermGeom<C> G;
  static_assert(G::CB == 2 && C::NG == 1, "");
  const TermLane<C> me;
  const int n = n0 + me.col0 + (me.lq & 1) * 16 + me.li;
  const float b = bias && n < N ? bias[n] : 0.f;
#pragma unroll
  for (int r = 0; r < G::RB; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc.v[r][0][0][e]),
                                                      __float_as_uint(acc.v[r][0][1][e]), false, false);
      const long long m = m0 + me.row0 + r * 16 + 4 * (me.lq & 2) + e;
      if (n < N && m < M) out[m * N + n] = __uint_as_float(x[0]) + b;
      if (n < N && m + 4 < M) out[(m + 4) * N + n] = __uint_as_float(x[1]) + b;
    }
}

// Sums of the workgroup tile of a kernel of configuration C (TileCfg or TileCfgB).
template <class C, class = void>
struct InTerms : std::false_type {};
template <class C>
struct InTerms<C, typename std::enable_if<C::NP == 3 && !C::LOSUM>::type> : std::true_type {};
template <class C>
struct TileSums {
  typedef typename std::conditional<InTerms<C>::value, TermAcc<C>, Acc<C>>::type type;
};
template <class C>
__device__ inline void stage_write(const typename TileSums<C>::type& acc, int ba, float* stage) {
  if constexpr (InTerms<C>::value)
    stage_write_terms<C>(acc, ba, stage);
  else
    EpiStage<C>::write(acc, ba, stage);
}

}  // namespace mg

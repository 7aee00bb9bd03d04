// A whole serial propagation (coarsest-level solve, serial scan, serial back-propagation) of a
// few rows as one launch: see kernels_scan.hip.
#pragma once
#include "common.h"

namespace mg {

// Recurrence kinds.  GRU, ODE and LSTM take h_k = Phi(h_{k-1}) + g_k for k = 1..N; the adjoint
// takes w_{k-1} = (dPhi_k/dh)^T w_k + g_{k-1} for k = N..1.
enum ScanKind { SCAN_GRU = 0, SCAN_ADJOINT = 1, SCAN_LSTM = 2, SCAN_ODE = 3 };

struct ScanArgs {
  const void* Wt;      // recurrent weights, float or bf16: U[NG H, H] (forward), UT[H, 3H] (adjoint)
  const float* b_h;    // [NG H] (GRU, LSTM)
  const float* P;      // projection rows [*, B, NG H] (forward)
  const float* kap;    // coefficient rows [N + 1, B, kw] (adjoint)
  float* u;            // state array [N + 1, B, H] (LSTM: [N + 1, B, 2H])
  const float* g;      // right-hand side, laid out like u (may be null)
  int* ctl;            // device words: [0] workgroups that have arrived, [1] not all came in time (both for
                       // the exchange through memory), [2..3] (64 bits) next item, the rest in scan_exchange.h
  float* ring;         // scan_ring_floats(...) floats, or null: exchange through memory
  long long ring4;     // (set by launch_scan)
  int N, B, H, kw;
  long long pstep;     // forward: step k reads projection point k * pstep - 1
  float gamma;
  int implicit_;       // GRU / LSTM: implicit form of the step
  int bf16;            // 1: Wt is bf16
  int terms;           // GRU on bf16 weights: inside the XCDs, contract terms of the state (see
                       // kernels_scan_xcd.hip); more than 64 rows always do
  long long wait_ticks;   // limit of the wait for all workgroups to arrive (100 MHz ticks)
};

// True if a solve of N steps over B rows of hidden width H runs as one launch.
// terms: as in ScanArgs; ring: there is space for scan_ring_floats(...) floats.
bool scan_covers(int kind, long long N, int B, int H, bool terms, bool ring);
// Scratch with which the exchange runs inside the XCDs (0: this shape does not).
size_t scan_ring_floats(int kind, int B, int H, bool terms);
hipError_t launch_scan(int kind, const ScanArgs& a, hipStream_t s);

}  // namespace mg

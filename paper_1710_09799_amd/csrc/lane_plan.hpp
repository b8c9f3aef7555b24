// lane_plan.hpp -- when the one-wavefront tile kernel (fwd_lane.hpp) runs and
// with which tile.  Host code, no device calls.
#pragma once

#include <algorithm>
#include <cstdint>

namespace mln {

// Tiles of W cells on one wavefront (W / 64 cells per lane) or on W / 64
// wavefronts of the one-cell-per-thread kernel.  A lane's step is as long as
// its cells, so tiles of four cells per lane need about three wavefronts per
// compute unit to win (three-level FP64, 256 cells and 24 steps: 721 tiles
// 7.1e10 against 7.2e10 cell-updates/s, 289 tiles 2.9e10 against 3.5e10), and
// from there on they do (5042 tiles 1.46e11 against 9.2e10); tiles of one or
// two cells per lane always do (128 cells, 24 steps: 500 tiles 3.3e10 against
// 2.5e10; 64 cells, 12 steps: 1000 tiles 3.8e10 against 2.4e10).
inline bool lane_better(int W, int64_t ntiles, int cus) { return W <= 128 || ntiles >= 3 * (int64_t)cus; }

// Smallest grid that the automatic choice gives to the one-wavefront kernel
// (four lanes per cell below): where the measured times cross, us per step
// one wavefront / four lanes.  Two-level: FP64 22000 cells 0.65 / 0.64, 24000
// 0.66 / 0.74; compensated 20000 cells 0.70 / 0.62, 25000 0.72 / 0.85; FP32 23000
// cells 0.60 / 0.56, 25000 0.56 / 0.69 (and 32000 0.56 / 0.54).  Three-level:
// FP64 22500 cells 0.92 / 0.81, 24000 0.90 / 0.93; FP32 36000 cells 0.88 / 0.79,
// 40000 0.90 / 0.94; compensated (its product on the matrix cores) 40000 cells
// 1.19 / 1.12, 45000 1.33 / 1.16, 60000 1.46 / 1.38, 75000 1.49 / 1.72.
inline int64_t lane_min_cells(int N, bool fp32_plain, bool comp) {
  if (N == 2) return fp32_plain ? 24000 : 23000;
  return fp32_plain ? 38000 : (comp ? 45000 : 23000);
}

// Whether a solver may take `bytes` more for a second state buffer that it can
// do without: at most an eighth of the device memory that is free, so that
// what the caller allocates next still fits (several steps per launch are worth
// 1.7x on the 2-D grid; a state of that size fills 36 GB).
inline bool second_buffer_fits(uint64_t bytes, uint64_t free_bytes) { return bytes <= free_bytes / 8; }

struct LanePlan {
  int W, K;  // cells per tile, steps per launch
};

// Tile and steps per launch from a model of a launch: a fixed 2.3 us, K steps
// of the busiest SIMD (n wavefronts on it: the latency L of one wavefront's
// step, or n times its issue time I) and half of the launch's memory time
// (the other half overlaps).  L and I in us for 1, 2 and 4 cells per lane,
// fitted to runs of 4000 to 4 million cells; the choice is within a few
// percent of the best shape there.
inline LanePlan lane_plan(int N, bool fp32_plain, int state_bytes, int64_t nx, int cus) {
  static const double L[2][2][3] = {{{0.34, 0.47, 0.74}, {0.30, 0.40, 0.60}}, {{0.73, 1.09, 2.02}, {0.52, 0.90, 1.63}}};
  static const double I[2][2][3] = {{{0.15, 0.22, 0.40}, {0.10, 0.14, 0.27}}, {{0.56, 0.80, 1.50}, {0.28, 0.54, 1.07}}};
  static const int C[3] = {1, 2, 4};
  const int ni = N == 2 ? 0 : 1, pi = fp32_plain ? 1 : 0;
  LanePlan best{256, 24};
  double best_t = 0.0;
  for (int c = 0; c < 3; ++c) {
    const int W = 64 * C[c];
    for (int K = 8; K <= (W == 64 ? 28 : W * 3 / 8); K += 4) {
      const int64_t owned = W - 2 * K, tiles = (nx + owned - 1) / owned;
      const double n = (double)tiles / (4.0 * cus);
      // up to four wavefronts share a SIMD at once; beyond that they follow each other
      const double w = n <= 1.0 ? 1.0 : (n <= 4.0 ? (double)(int64_t)(n + 0.999999) : n + 0.4);
      const double step = std::max(L[ni][pi][c], n <= 1.0 ? 0.0 : w * I[ni][pi][c]);
      const double mem = (double)nx * (1.0 + (double)K / (double)owned) * 2.0 * state_bytes / 4.9e6;
      const double t = (2.3 + K * step + 0.5 * mem) / K;
      if (best_t == 0.0 || t < best_t) {
        best_t = t;
        best = {W, K};
      }
    }
  }
  return best;
}

// The same for the FP64 matrix-core kernel of N = 4, 6 (fwd_mfma64.hpp): a
// compute unit works off its tiles in rounds of as many as its registers hold
// (wavefronts per SIMD: two at N = 6, three at N = 4); a round costs 3 us of
// loads and stores and K steps of L[w] us with w wavefronts on the busiest
// SIMD, a launch F us.  Fitted to runs of 2000 to 200000 cells, us per step
// model / measured: six levels, 50000 cells, 256 cells and 24 steps 4.2 / 4.4,
// 128 and 30 6.4 / 6.1, 64 and 12 7.2 / 7.1; 2000 cells, 128 and 48 2.4 / 2.3;
// four levels, 200000 cells, 128 and 12 6.1 / 6.0.
inline LanePlan mfma64_plan(int N, int64_t nx, int cus) {
  static const double L[2][4] = {{0.0, 1.72, 2.1, 2.3}, {0.0, 2.15, 3.65, 3.65}};
  static const int waves[2] = {3, 2}, Ws[3] = {64, 128, 256};
  const int ni = N == 4 ? 0 : 1;
  const double F = N == 4 ? 3.0 : 9.0;
  LanePlan best{256, 24};
  double best_t = 0.0;
  for (int W : Ws) {
    const int share = waves[ni] * 256 / (2 * W);  // tiles a compute unit holds: W / 32 wavefronts each
    if (share < 1) continue;
    const int wmax = std::max(1, share * W / 128);  // wavefronts per SIMD of a full round
    for (int K = 4; 2 * K < W && K <= 60; K += 2) {
      const int64_t owned = W - 2 * K, tiles = (nx + owned - 1) / owned, per = (tiles + cus - 1) / cus;
      const int64_t full = per / share, rest = per % share;
      const double t = (F + full * (3.0 + K * L[ni][wmax]) +
                        (rest ? 3.0 + K * L[ni][std::max<int64_t>(1, (rest * W + 127) / 128)] : 0.0)) / K;
      if (best_t == 0.0 || t < best_t) {
        best_t = t;
        best = {W, K};
      }
    }
  }
  return best;
}

}  // namespace mln

// Decomposition of the few-column kernel (xorenc_spmm_f4.h).  Host arithmetic only: no HIP in this file, so that it can be
// checked without a GPU.
#ifndef XORENC_F4_PLAN_H
#define XORENC_F4_PLAN_H

#include <algorithm>
#include <cstdint>

#include "xorenc_split_plan.h"

constexpr int kF4MaxB = 8;                  // the 16 rows of the X operand: two terms of eight columns
constexpr int kF4MaxBOneRound = 2;          // beyond that the other kernels are faster on one round (measured) ...
constexpr int kF4MinRoundsWide = 4;         // ... and pays from this many rounds on (measured, 4096 columns of W)
constexpr int kF4Waves = 16;
constexpr int kF4XBytes = 64 * 1024 + 256;  // raw X, then the X operands, then the partial sums
constexpr int kF4MaxSpr = 256;              // 16 waves x 8 pairs x 2 words
constexpr int kF4SclBytes = 2304;           // two scale bytes per (half-word, column)

struct F4Plan {
  int PW, KS, RG, grid, rounds;
};

// pairs per wave: what fits 128 registers, without and with the words of a round requested ahead (more tables
// need more temporaries, a field that straddles two dwords a larger set of words per pair)
constexpr int f4_pmax(int Q) { return Q == 1 ? 8 : (Q == 2 ? 6 : (Q == 3 ? 4 : 2)); }
constexpr int f4_pmax_mr(int Q, int nibt) {
  return Q == 1 ? (nibt == 1 ? 6 : 4) : Q == 2 ? (nibt == 3 ? 3 : 4) : Q == 3 ? (nibt == 3 ? 2 : 3) : 2;
}

// Picks the decomposition for a layer of `nrb` row blocks and `spr` words per row (slices of one word, `nib` tables) and B
// columns: PW word pairs per wave, KS K ranges, RG granules per workgroup and round, and the number of rounds (at most
// one workgroup per CU); false when the kernel does not apply to the call.
inline bool f4_plan(int spr, int nrb, int q, int nib, int B, F4Plan *out) {
  const int PMAX = f4_pmax(q), PMAX_MR = f4_pmax_mr(q, nib);
  if (B < 1 || B > kF4MaxB || spr > kF4MaxSpr) return false;
  const int spr_pad = 2 * ((spr + 1) / 2);  // whole word pairs
  // raw X (with its column padding) and the operands of the whole K range share one area; scales next to it
  if ((int64_t)spr_pad * 128 * B + 256 > kF4XBytes || 4 * spr_pad * B + 16 > kF4SclBytes) return false;
  // one conversion item (half-word, column) per thread
  const int items = 2 * spr_pad * (B >= 5 ? 8 : (B >= 3 ? 4 : B));
  if (items > kF4Waves * 64) return false;
  const int pairs = (spr + 1) / 2;
  const int n_gran = 2 * nrb;
  int best_cost = 1 << 30;
  F4Plan best{};
  for (int pw = PMAX; pw >= 1; --pw) {
    const int ks = (pairs + pw - 1) / pw;
    if (ks > kF4Waves) break;
    const int rg = std::min(kF4Waves / ks, 8);  // at most 8 x 128 outputs per workgroup and round: one per thread
    const int wgs = (n_gran + rg - 1) / rg;
    const int grid = std::min(wgs, kSplitMaxGroups);
    const int rounds = (wgs + grid - 1) / grid;
    // the kernel variant that walks over rounds also serves more than two columns; its requests of the next round
    // need registers too
    if ((rounds > 1 || B > kF4MaxBOneRound) && pw > PMAX_MR) continue;
    // time of a wave: a fixed part, then per round its pairs and the exchange of the partial sums; among equals,
    // more workgroups
    const int cost = (4 + rounds * (pw + 2)) * 1024 - grid;
    if (cost < best_cost) {
      best_cost = cost;
      best = F4Plan{pw, ks, rg, grid, rounds};
    }
  }
  if (best_cost == (1 << 30)) return false;
  if (B > kF4MaxBOneRound && best.rounds < kF4MinRoundsWide) return false;
  *out = best;
  return true;
}

#endif

// Where the encoders keep their patch counts, and how the emission of the patch lists is cut into workgroups.  Host
// arithmetic only: no HIP in this file, so that it can be compiled and checked without a GPU.
#ifndef XORENC_ENCODE_PLAN_H
#define XORENC_ENCODE_PLAN_H

#include <algorithm>
#include <cmath>

#include "xorenc_internal.h"

constexpr int ENC_THREADS = 256;
constexpr int ENC_UNITS = ENC_THREADS / 32;  // 32-slice groups of a workgroup of the encoding kernels
constexpr int EMIT_UNITS = 128;              // most units of a workgroup of the emission
// Counting blocks up to which a workgroup of the emission adds up the totals before its own by itself (4 bytes per
// ENC_UNITS * J units and workgroup from the L2; 16384 x 4096, two planes: 64 KB at most); from there a scan is cheaper.
constexpr int kDirectBlocks = 32768;

// The counts lie in the workspace behind the patch bitmaps, where it has 4 bytes per unit and plane: 2 bytes per unit,
// then 4 per counting block (8 where the totals are scanned, which takes thousands of blocks).  A block has at least
// eight units or is the only one of its plane, so they fit from two units per plane on.  With one unit per plane the
// block's total is the unit's count, and there are no counts of units.
struct EncodePlan {
  int64_t unit_at;     // byte offset of uint16[q*n_units] behind the bitmaps, -1: the block totals are the counts
  int64_t block_at;    // of uint32[q*n_blocks]
  int64_t scanned_at;  // of uint32[q*n_blocks + 1], -1: not scanned
  int32_t n_blocks;    // counting blocks of a plane
  int32_t units_per_block;
  int32_t per;           // counting blocks of a workgroup of the emission
  uint32_t emit_groups;  // workgroups of the emission
};

inline EncodePlan encode_plan(const xorenc_sizes &sz, int32_t q, int32_t n_out) {
  EncodePlan P;
  const int64_t n_counts = (int64_t)q * sz.n_units;
  P.units_per_block = ENC_UNITS * (n_out / 64);
  P.n_blocks = (int32_t)((sz.n_eslots + ENC_THREADS - 1) / ENC_THREADS);
  const int32_t blocks = q * P.n_blocks;
  P.unit_at = sz.n_units > 1 ? 0 : -1;
  P.block_at = sz.n_units > 1 ? (2 * n_counts + 3) / 4 * 4 : 0;
  P.scanned_at = blocks > kDirectBlocks ? P.block_at + 4 * (int64_t)blocks : -1;
  // as many blocks as a workgroup has room for, fewer while there are not a thousand workgroups
  P.per = std::max(1, std::min(EMIT_UNITS / P.units_per_block, blocks / 1024));
  P.emit_groups = (uint32_t)((blocks + P.per - 1) / P.per);
  return P;
}

// The encoder with the fewest patches: most care bits of a slice that is tried by syndrome (sets of up to three care bits)
// before it is put on the list for the search over all inputs, in workgroups of the slices kernel that have few such
// slices (kSyndromeFew) and in those that have more.
//
// A few cost next to nothing, their waves run beside other workgroups', while the search of any slice at all takes a
// wave of every CU tens of microseconds.  Many have to be worth it: a slice takes about 4000 + 12 c^2 cycles of one SIMD by
// syndrome (c care bits) and 2^(n_in - 10) (100 + 90 J) by search, a third of that may be lost where no set matches, and
// fewer than four workgroups per CU leave SIMDs idle.  The sets reach a share of the 2^(c - n_in) syndromes.
// us a call, all slices of up to `few` care bits by syndrome / none / this rule: 16384 x 4096, S = 0.95, n_out = 192, n_in = 20
// 80 / 302 / 80; 4096 x 4096, S = 0.9, n_out = 192, n_in = 20 677 / 4650 / 685; S = 0.9, n_in = 12 70 / 108 / 72; 2048 x 2048,
// S = 0.8, n_in = 16 267 / 214 / 201; two planes, S = 0.5, n_in = 16 1890 / 814 / 814; 1024 x 1024, S = 0.5, n_in = 20 2565 /
// 1300 / 1244 (64 workgroups).
constexpr int kSyndromeFew = 16;

struct SyndromeCare {
  int few, many;
};

inline SyndromeCare syndrome_care(int n_in, int J, int64_t workgroups) {
  SyndromeCare care{std::min(32, n_in + 12), 0};
  const double idle = std::max(1.0, 1024.0 / (double)std::max<int64_t>(workgroups, 1));
  const double search = std::exp2(n_in - 10) * (100 + 90 * J);
  for (int c = 1; c <= care.few; ++c) {
    const double sets = c + c * (c - 1) / 2 + c * (c - 1) * (c - 2) / 6;
    const double match = std::min(1.0, sets / std::exp2(std::max(0, c - n_in)));
    if ((4000 + 12 * c * c) * idle > 0.7 * search * match) break;
    care.many = c;
  }
  return care;
}

#endif

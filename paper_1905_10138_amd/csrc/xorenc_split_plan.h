// Sizes of the scratch area in which workgroups that split the reduction of an output tile meet, and the few-column
// kernel's cut of the reduction.  Host arithmetic only: no HIP in this file, so that it can be checked without a GPU.
#ifndef XORENC_SPLIT_PLAN_H
#define XORENC_SPLIT_PLAN_H

#include <algorithm>
#include <cstdint>

constexpr int kSplitTileFloats = 4096;  // largest output tile of a split launch (64 x 64)
constexpr int kSplitMaxGroups = 256;    // workgroups of a split launch (one per CU), and tickets of a scratch area

constexpr int kSmallMaxB = 8;            // columns of the few-column kernel: rows 0..7 of its accumulators
constexpr int kSmallXBytes = 96 * 1024;  // LDS set aside for X^T (rows padded by 16 bytes)

// Cut of a reduction of `spr` words per row into `ks` ranges of `sps` words (whole words per wave) for `row_groups` row
// tiles: at most one workgroup per CU, and as many more as it takes that X^T of a range fits the LDS set aside for it.
// ks > 1 needs the scratch area: a ticket per row tile and kSmallMaxB columns of `rows` values per workgroup.
inline bool small_split(int row_groups, int rows, int spr, int B, int waves, bool scratch, int *ks_out, int *sps_out) {
  if (B > kSmallMaxB) return false;
  int ks = 1;
  if (row_groups < kSplitMaxGroups && scratch)
    ks = std::max(1, std::min((spr + waves - 1) / waves, kSplitMaxGroups / row_groups));
  int sps = (spr + ks - 1) / ks;
  sps = (sps + waves - 1) / waves * waves;
  auto x_bytes = [&] { return (int64_t)B * ((int64_t)std::min(sps, spr) * 128 + 16); };
  while (x_bytes() > kSmallXBytes && sps > waves) sps -= waves;
  if (x_bytes() > kSmallXBytes) return false;
  ks = (spr + sps - 1) / sps;
  if (ks > 1 && (!scratch || row_groups > kSplitMaxGroups ||
                 (int64_t)row_groups * ks * rows * kSmallMaxB > (int64_t)kSplitMaxGroups * kSplitTileFloats))
    return false;
  *ks_out = ks;
  *sps_out = sps;
  return true;
}

#endif

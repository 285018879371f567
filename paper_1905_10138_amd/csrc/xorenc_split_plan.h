// Sizes of the scratch area in which workgroups that split the reduction of an output tile meet, and the product kernels'
// cuts of the reduction.  Host arithmetic only: no HIP in this file, so that it can be checked without a GPU.
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

// Cut of a product's reduction: `ks` workgroups per output tile with `sps` words of the row each (whole words per wave).
// `us`: estimate of the time that the cut decides on, for choosing between kernel variants.
struct ReductionCut {
  int ks, sps;
  double us;
};

constexpr int kSplitMaxParts = 4;  // the workgroup that arrives last at a tile reads every part

// Variant of the kernel for `col_blocks` blocks of 32 columns and `row_blocks` of 32 rows per workgroup of `waves` waves.
struct CutVariant {
  int q, col_blocks, row_blocks, waves;
  bool one_word, split_x;  // slices of one word; X in memory as three terms per column
  bool by_entry;           // long patch lists are taken entry by entry
};

// Splitting a tile's reduction over workgroups shortens every wave's share and costs a meeting: parts stored to the
// coherent level, a ticket, the parts read back by the last, one after the other.  Filling the chip's CUs at any price, as
// was done before, paid 1.3 to 2.5 us for it to save a few slices of 0.3 to 0.7 us each (us, most workgroups / this rule:
// 2048 x 2048, B = 8 7.0 / 5.5; 4096 x 1024, B = 64 7.1 / 5.5; 2500 x 1500, two planes, B = 64 8.0 / 6.3).  The time of a
// word per wave and of a meeting were fitted to 500 products of 512 x 512 to 4096 x 9216, one to three planes, with few
// patches, n_in = 16 and 24 (one word per slice) or 16 and 20, all cuts timed on each: 0.5 % from the best cut in the mean
// over these very products.  Other widths, four planes and longer lists have the same estimate.
// Kernels that take lists entry by entry (X read element by element, or split on its way) have no such estimate: a word
// takes 0.3 us or, with the hundreds of entries of a narrow encrypted vector, 10, and the host does not know the lists.
// They fill the chip (us, so / by the estimate: 3877 x 1051, two planes, n_out = 128, n_in = 5, B = 9 33 / 64; fp32 X,
// 3094 x 316, four planes, S = 0.8, n_in = 7, B = 12 41 / 69; 2043 x 303, three planes, n_in = 11, B = 64 9.2 / 9.9; the
// other way 969 x 539, n_in = 14, B = 100 8.8 / 8.2).
inline ReductionCut cut_reduction(const CutVariant &v, int spr, int row_groups, int col_groups, bool scratch) {
  const int64_t tiles = (int64_t)row_groups * col_groups;
  double word = 0.1 + 0.2 * v.q;
  if (v.col_blocks > 1) word *= 1.4;
  if (v.row_blocks > 1) word *= 1.7;
  if (v.waves > 8) word *= 1.25;
  if (v.split_x) word *= 3.0;
  if (!v.one_word) word *= 1.75;
  // narrow tiles read W once per block of columns, and rows of X in halves of a cache line
  if (v.col_blocks == 1 && col_groups > 1) word = (word + 0.06 * (col_groups - 1)) * (spr > 64 ? 1.3 : 1.0);
  const bool large_tile = v.col_blocks * v.row_blocks > 1;
  double fixed = 0.0;
  if (v.waves > 8 && v.one_word) fixed += 0.1 + 0.15 * v.q;
  if (v.col_blocks == 2) fixed += 0.35 + 0.05 * v.q;
  int most = 1;
  if (scratch && tiles < kSplitMaxGroups && 1024 * v.row_blocks * v.col_blocks <= kSplitTileFloats)
    most = (int)std::max<int64_t>(1, std::min<int64_t>({(spr + v.waves - 1) / v.waves, kSplitMaxGroups / tiles, kSplitMaxParts}));
  ReductionCut best{1, 0, 0.0};
  for (int want = v.by_entry ? most : 1; want <= most; ++want) {
    int sps = (spr + want - 1) / want;
    sps = (sps + v.waves - 1) / v.waves * v.waves;
    const int ks = (spr + sps - 1) / sps;
    // (a last word that only some of the waves have costs about half)
    double us = fixed + 0.5 * word * (sps / v.waves + (double)spr / ((double)ks * v.waves));
    if (ks > 1) {
      const double full = std::min(1.0, (double)(tiles * ks) / kSplitMaxGroups);  // (the more workgroups, the longer they meet)
      us += (large_tile ? 0.65 + 0.48 * ks : 0.5 + 0.3 * ks + 0.6 * full) + (v.one_word ? 0.0 : 0.6);
    }
    if (best.sps == 0 || us < best.us) best = ReductionCut{ks, sps, us};
  }
  return best;
}

#endif

"""Host-side plans of the library (headers without HIP), compiled with g++ together with the host sources and checked on
the CPU for conditions that a run on the GPU would only break now and then."""
import os
import shutil
import subprocess

import pytest

from helpers import CUTS_IN_PARTS, FEW_COLUMNS_IN_ROUNDS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1905_10138_amd", "csrc")


def run_program(tmp_path, text, *sources, flags=()):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++ here")
    src, exe = str(tmp_path / "main.cpp"), str(tmp_path / "main")
    with open(src, "w") as f:
        f.write(text)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, *flags, src,
                    *[os.path.join(CSRC, s) for s in sources], "-o", exe], check=True, timeout=120)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:]


ENCODE_PLAN = r"""
#include <cstdio>
#include "xorenc_encode_plan.h"

#define CHECK(c) do { if (!(c)) { std::printf("m=%d n=%d q=%d n_out=%d: %s\n", m, n, q, n_out, #c); return false; } } while (0)

static bool check(int m, int n, int q, int n_out) {
  xorenc_sizes sz;
  CHECK(xorenc_get_sizes(m, n, 8, q, n_out, &sz) == XORENC_OK);
  const EncodePlan P = encode_plan(sz, q, n_out);
  // [0, end) of the workspace behind the bitmaps: units, blocks and scanned totals, one after the other
  const int64_t end = 4 * (int64_t)q * sz.n_units, blocks = (int64_t)q * P.n_blocks;
  int64_t at = 0;
  if (P.unit_at >= 0) {
    CHECK(P.unit_at >= at && P.unit_at % 2 == 0);
    at = P.unit_at + 2 * q * sz.n_units;
  } else {
    CHECK(sz.n_units == 1 && P.n_blocks == 1);  // a block's total stands for its unit's count
  }
  CHECK(P.block_at >= at && P.block_at % 4 == 0);
  at = P.block_at + 4 * blocks;
  CHECK((P.scanned_at >= 0) == (blocks > kDirectBlocks));
  if (P.scanned_at >= 0) {
    CHECK(P.scanned_at >= at && P.scanned_at % 4 == 0);
    at = P.scanned_at + 4 * (blocks + 1);
  }
  CHECK(at <= end);
  CHECK((int64_t)P.n_blocks * P.units_per_block >= sz.n_units && (int64_t)(P.n_blocks - 1) * P.units_per_block < sz.n_units);
  CHECK(P.per >= 1 && P.per * P.units_per_block <= EMIT_UNITS);
  CHECK((int64_t)P.emit_groups * P.per >= blocks && (int64_t)(P.emit_groups - 1) * P.per < blocks);
  return true;
}

int main() {
  for (int q = 1; q <= 4; ++q)
    for (int n_out = 64; n_out <= 256; n_out += 64) {
      for (int m = 1; m <= 700; m += 31)
        for (int n = 1; n <= 1400; n += 63)
          if (!check(m, n, q, n_out)) return 1;
      for (int m : {8191, 32768, 32800, 65536, 500000})
        for (int n : {1, 64, 65, 4096, 9216, 30000})
          if (!check(m, n, q, n_out)) return 1;
    }
  return 0;
}
"""


def test_patch_counts_lie_in_the_workspace(tmp_path):
    """The emission of the patch lists runs as many workgroups in any order, and each writes offsets as it goes: the
    counts that the others still read have to lie in the workspace, apart from each other and inside its stated size.
    (With one unit per plane they used to lie in the offsets: a late workgroup read what an early one had written.)"""
    run_program(tmp_path, ENCODE_PLAN, "xorenc_host.cpp")


SYNDROME = r"""
#include <cstdio>
#include "xorenc_encode_plan.h"

#define CHECK(c) do { if (!(c)) { std::printf("n_in=%d J=%d workgroups=%lld: %s\n", n_in, J, (long long)groups, #c); return 1; } } while (0)

int main() {
  for (int n_in = 11; n_in <= 24; ++n_in)
    for (int J = 1; J <= 4; ++J) {
      int before = 0;
      for (int64_t groups : {(int64_t)1, (int64_t)2, (int64_t)63, (int64_t)205, (int64_t)1024, (int64_t)100000, (int64_t)1 << 21}) {
        const SyndromeCare care = syndrome_care(n_in, J, groups);
        CHECK(care.few >= 1 && care.few <= 32);                // a lane and a bit of a dword per kept bit
        CHECK(care.many >= before && care.many <= care.few);   // the more workgroups, the more are worth it
        before = care.many;
      }
    }
  // the workgroups of test_gpu_encode.py's test_fewest_patches_by_syndrome
  struct { int n_in, J, groups, few, many; } const cases[] = {{11, 1, 1, 23, 0}, {13, 2, 1, 25, 0}, {16, 3, 1, 28, 0},
                                                              {16, 1, 3, 28, 0}, {16, 4, 205, 28, 3}, {16, 4, 1024, 28, 28},
                                                              {16, 1, 1024, 28, 19}};
  for (const auto &c : cases) {
    const int n_in = c.n_in, J = c.J;
    const int64_t groups = c.groups;
    const SyndromeCare care = syndrome_care(n_in, J, groups);
    CHECK(care.few == c.few && care.many == c.many);
  }
  return 0;
}
"""


def test_slices_tried_by_syndrome(tmp_path):
    run_program(tmp_path, SYNDROME)


SMALL_SPLIT = r"""
#include <cstdio>
#include "xorenc_split_plan.h"

#define CHECK(c) do { if (!(c)) { std::printf("groups=%d rows=%d spr=%d B=%d waves=%d scratch=%d ks=%d sps=%d: %s\n", \
                                              groups, rows, spr, B, waves, scratch, ks, sps, #c); return false; } } while (0)

static bool check(int groups, int rows, int spr, int B, int waves, bool scratch) {
  int ks = 0, sps = 0;
  if (!small_split(groups, rows, spr, B, waves, scratch, &ks, &sps)) return true;  // another kernel's
  CHECK(ks >= 1 && sps >= 1 && (int64_t)ks * sps >= spr && (int64_t)(ks - 1) * sps < spr);
  CHECK((int64_t)B * ((int64_t)(sps < spr ? sps : spr) * 128 + 16) <= kSmallXBytes);
  if (ks > 1) {
    CHECK(scratch);
    CHECK(groups <= kSplitMaxGroups);  // tickets
    CHECK((int64_t)groups * ks * rows * kSmallMaxB <= (int64_t)kSplitMaxGroups * kSplitTileFloats);
  }
  return true;
}

int main() {
  for (int waves : {8, 12, 16})
    for (int rows : {32, 64})
      for (int B = 1; B <= 9; ++B)
        for (int groups : {1, 2, 7, 64, 127, 128, 129, 200, 255, 256, 257, 300, 1024, 30000})
          for (int spr = 1; spr <= 3000; spr += spr < 400 ? 1 : 37)
            for (int scratch = 0; scratch < 2; ++scratch)
              if (!check(groups, rows, spr, B, waves, scratch)) return 1;
  return 0;
}
"""


def test_parts_of_the_few_column_kernel_fit_the_scratch_area(tmp_path):
    """The cut that makes X^T of a range fit LDS may take more workgroups than the chip has compute units: parts and tickets
    have to lie inside the scratch area all the same.  (They used to run over its end: 12800 x 16384, four columns with a
    leading dimension of four, 400 workgroups in the room of 256.)"""
    run_program(tmp_path, SMALL_SPLIT)


CUT = r"""
#include <cstdio>
#include "xorenc_split_plan.h"

#define CHECK(e) do { if (!(e)) { std::printf("q=%d cols=%d rows=%d waves=%d spr=%d groups=%d x %d scratch=%d ks=%d sps=%d: %s\n", \
    v.q, v.col_blocks, v.row_blocks, v.waves, spr, rg, cg, scratch, c.ks, c.sps, #e); return false; } } while (0)

static bool check(const CutVariant &v, int spr, int rg, int cg, bool scratch) {
  const ReductionCut c = cut_reduction(v, spr, rg, cg, scratch);
  CHECK(c.sps >= 1 && c.sps % v.waves == 0);  // whole words per wave
  CHECK((int64_t)c.ks * c.sps >= spr && (int64_t)(c.ks - 1) * c.sps < spr);  // every word once, no empty part
  CHECK(c.ks >= 1 && c.ks <= kSplitMaxParts && c.us > 0.0);
  if (c.ks > 1) {
    CHECK(scratch && (int64_t)rg * cg * c.ks <= kSplitMaxGroups);  // tickets and parts
    CHECK(32 * v.row_blocks * 32 * v.col_blocks <= kSplitTileFloats);
  }
  if (v.by_entry) {  // as many parts as there are CUs and whole words per wave for
    int most = 1;
    while (scratch && most < kSplitMaxParts && (int64_t)rg * cg * (most + 1) <= kSplitMaxGroups && most * v.waves < spr &&
           1024 * v.row_blocks * v.col_blocks <= kSplitTileFloats)
      ++most;
    const int sps = ((spr + most - 1) / most + v.waves - 1) / v.waves * v.waves;
    CHECK(c.sps == sps && c.ks == (spr + sps - 1) / sps);
  }
  return true;
}

int main() {
  for (int q = 1; q <= 4; ++q)
    for (int cols : {1, 2, 3})
      for (int rows : {1, 2, 4})
        for (int waves : {4, 8, 12, 16})
          for (int kind = 0; kind < 6; ++kind)
            for (int rg : {1, 2, 7, 63, 64, 65, 127, 128, 129, 255, 256, 257, 512, 30000})
              for (int cg : {1, 2, 4, 5, 33})
                for (int spr = 1; spr <= 2000; spr += spr < 100 ? 1 : 131)
                  for (int scratch = 0; scratch < 2; ++scratch)
                    if (!check(CutVariant{q, cols, rows, waves, kind % 2 == 0, kind / 2 == 1, kind / 2 == 2}, spr, rg, cg, scratch)) return 1;
  return 0;
}
"""


def test_cuts_of_the_reduction_cover_it_and_fit_the_scratch_area(tmp_path):
    run_program(tmp_path, CUT)


CUT_IN_PARTS = r"""
#include <cstdio>
#include "xorenc_split_plan.h"

int main() {
  struct { int q, m, n, B, col_blocks, waves, ks; } const cases[] = {CASES};
  for (const auto &c : cases) {
    const int rg = (c.m + 31) / 32, spr = (c.n + 63) / 64, blocks = (c.B + 31) / 32;
    // 32-row tiles: eight or twelve waves and one block of columns, or eight and two
    ReductionCut best{0, 0, 1e9};
    int cols = 0, waves = 0;
    for (const auto &v : {CutVariant{c.q, 1, 1, 8, true, false, false}, CutVariant{c.q, 1, 1, 12, true, false, false},
                          CutVariant{c.q, 2, 1, 8, true, false, false}}) {
      if (blocks > 1 ? v.waves > 8 : v.col_blocks > 1) continue;
      const int cg = (blocks + v.col_blocks - 1) / v.col_blocks;
      if (rg * cg > kSplitMaxGroups) continue;
      const ReductionCut cut = cut_reduction(v, spr, rg, cg, true);
      if (cut.us < best.us) best = cut, cols = v.col_blocks, waves = v.waves;
    }
    if (best.ks != c.ks || cols != c.col_blocks || waves != c.waves) {
      std::printf("q=%d %d x %d B=%d: %d parts, %d blocks of columns, %d waves\n", c.q, c.m, c.n, c.B, best.ks, cols, waves);
      return 1;
    }
  }
  return 0;
}
"""


def test_layers_in_two_and_three_parts(tmp_path):
    """The layers of test_gpu_spmm.py's test_two_and_three_workgroups_per_tile have as many parts as it says."""
    run_program(tmp_path, CUT_IN_PARTS.replace("CASES", ", ".join("{%d, %d, %d, %d, %d, %d, %d}" % c for c in CUTS_IN_PARTS)))


FEW_COLUMNS = r"""
#include <cstdio>
#include "xorenc_f4_plan.h"

int main() {
  struct { int q, m, n, n_in, pw, rounds; } const cases[] = {CASES};
  for (const auto &c : cases)
    for (int B = 1; B <= 2; ++B) {
      F4Plan P{};
      const bool taken = f4_plan((c.n + 63) / 64, (c.m + 31) / 32, c.q, (c.n_in + 7) / 8, B, &P);
      if (!taken || P.PW != c.pw || P.rounds != c.rounds) {
        std::printf("q=%d %d x %d n_in=%d B=%d: taken %d, %d pairs, %d rounds\n", c.q, c.m, c.n, c.n_in, B, taken, P.PW, P.rounds);
        return 1;
      }
    }
  return 0;
}
"""


def test_layers_whose_waves_end_inside_a_group(tmp_path):
    """The layers of test_gpu_spmm.py's test_long_patch_lists_of_few_columns have the word pairs per wave and the rounds
    that it says."""
    run_program(tmp_path, FEW_COLUMNS.replace("CASES", ", ".join("{%d, %d, %d, %d, %d, %d}" % c for c in FEW_COLUMNS_IN_ROUNDS)))


SCRATCH_OWNERS = r"""
#include <cstdio>
#include <set>
#include "xorenc_scratch.h"

#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static ScratchOwners owners, others;

int main() {
  auto at = [](uintptr_t p) { return reinterpret_cast<const void *>(p); };
  // streams, threads behind the handle that stands for a thread's stream, and captures on the same stream
  std::set<int> tickets, slots;
  int first_tickets = -1, first_slot = -1;
  for (int i = 0; i < 40; ++i) {
    const ScratchOwner o = i < 10 ? ScratchOwner{at(i < 2 ? i : 0x7f0000000000 + 0x500 * i), nullptr, 0}
                         : i < 20 ? ScratchOwner{at(2), at(0x600000 + 64 * i), 0} : ScratchOwner{at(0x7f0000000000), nullptr, (uint64_t)i};
    const ScratchShare none = owners.share(o, false, 0, 0), a = owners.share(o, true, 1, 1000);
    CHECK(none.slot == -1 && none.tickets == a.tickets && a.tickets >= 0 && a.tickets < kScratchOwners);
    CHECK(tickets.insert(a.tickets).second);                     // nobody else's
    CHECK((a.slot >= 0) == (i < kScratchSlots) && a.slot < kScratchSlots);
    if (a.slot >= 0) CHECK(slots.insert(a.slot).second);
    if (i == 0) first_tickets = a.tickets, first_slot = a.slot;
    for (int r = 0; r < 100; ++r) {                              // the calls of one owner keep their share
      const ScratchShare b = owners.share(o, true, 1, 100);
      CHECK(b.tickets == a.tickets && b.slot == a.slot && b.ring == 1024 + 256 * (uint32_t)r);
    }
  }
  const ScratchShare again = owners.share(ScratchOwner{at(0), nullptr, 0}, true, 0, 0);
  CHECK(again.tickets == first_tickets && again.slot == first_slot);
  // more captures than there are sets: the last ones get none, new streams still do, owners keep theirs
  int served = 0;
  for (uint64_t c = 1; c <= 3 * kScratchOwners; ++c) served += others.share(ScratchOwner{at(0x1000), nullptr, c}, false, 0, 0).tickets >= 0;
  CHECK(served == kScratchOwners - kScratchStreams);
  CHECK(others.share(ScratchOwner{at(0x1000), nullptr, 5}, false, 0, 0).tickets == 4);
  std::set<int> streams;
  for (int i = 0; i < kScratchStreams; ++i) streams.insert(others.share(ScratchOwner{at(0x2000 + 16 * i), nullptr, 0}, true, 0, 0).tickets);
  CHECK((int)streams.size() == kScratchStreams && *streams.begin() >= served && *streams.rbegin() < kScratchOwners);
  CHECK(others.share(ScratchOwner{at(0x9000000), nullptr, 0}, true, 0, 0).tickets == -1);
  // copies of X stay inside the ring
  uint32_t state = 12345, ring = 0;
  for (int i = 0; i < 100000; ++i) {
    state = state * 1664525u + 1013904223u;
    const size_t bytes = (i % 3 ? 16 * (1 + state % 5000) : state % 7 ? 16 * (1 + state % (kStageBytes / 16)) : kStageBytes);
    const uint32_t place = ring_place(ring, bytes);
    CHECK(place % 16 == 0 && place + bytes <= kRingBytes);
  }
  return 0;
}
"""


def test_tickets_and_slots_have_one_owner(tmp_path):
    """Two streams, or a stream and a captured graph, or two graphs, never share what a product keeps beside its arguments,
    however many calls are made in between (slots used to be handed out in turn at the time of the call).  The addresses
    that follow from a share are apart by construction."""
    run_program(tmp_path, SCRATCH_OWNERS)

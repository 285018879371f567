// Who may use which part of the memory that the library keeps on a GPU for products (host code without HIP, so that it can
// be checked without a GPU).
//
// A product may need tickets (one counter per output tile of a split reduction, zero between launches), and memory for
// partial tiles and for a copy of X.  Two calls whose kernels may run at the same time must not share any of it.  Calls
// on one stream run one after the other, and so do the kernels that one stream contributes to a captured graph; any
// other two may overlap, also long after the calls were made, when graphs are replayed.  So tickets belong to a stream,
// or to a stream's part of one capture, from its first call on and for good: a graph that is replayed later still holds
// them.  The first kScratchSlots of these owners that ask for it get memory too.
#ifndef XORENC_SCRATCH_H
#define XORENC_SCRATCH_H

#include <cstddef>
#include <cstdint>

#include "xorenc_split_plan.h"

constexpr int kScratchOwners = 4096;  // sets of tickets (1 KB each)
constexpr int kScratchStreams = 256;  // of them kept for streams, however many graphs a program captures
constexpr int kScratchSlots = 4;      // slots of memory (12 MiB each)
constexpr size_t kTicketBytes = (size_t)kSplitMaxGroups * sizeof(uint32_t);
constexpr size_t kPartBytes = (size_t)kSplitMaxGroups * kSplitTileFloats * sizeof(float);  // 4 MiB
constexpr size_t kStageBytes = (size_t)4 << 20;  // largest copy of X: 8192 rows of 256 bf16 columns
// Copies of X go round a ring: the lines of the copy that the product before has just read are still in the L2 caches of
// all XCDs (4 MiB each), and writing them again costs a call up to 3 us (4096 x 9216, two planes, fp32 X, B = 64: 31.0 us
// with one area, 28.1 with two and more; partial tiles, which bypass the L2, show no such difference).
constexpr size_t kRingBytes = 2 * kStageBytes;
constexpr size_t kSlotBytes = kPartBytes + kRingBytes;

// Place in the ring of a copy of `bytes` (at most kStageBytes); `at` moves behind it.
inline uint32_t ring_place(uint32_t &at, size_t bytes) {
  if (at + bytes > kRingBytes) at = 0;
  const uint32_t place = at;
  at += (uint32_t)((bytes + 255) / 256 * 256);
  return place;
}

struct ScratchOwner {
  const void *stream;
  const void *thread;  // tells the streams apart that share the handle of "this thread's default stream"; else null
  uint64_t capture;    // the capture's number, 0 outside of captures
};

struct ScratchShare {
  int tickets;  // -1: all sets belong to others
  int slot;     // -1: all slots belong to others, or none was asked for
  uint32_t ring;  // where the owner's last copy of X ends
};

// The owners on one GPU.  All zero is the empty table; the caller holds a lock.
class ScratchOwners {
 public:
  // The call is about to make `copies` copies of X, of at most `bytes` each (a bound for all of them).
  ScratchShare share(const ScratchOwner &o, bool want_slot, int copies, size_t bytes) {
    uint64_t h = ((uint64_t)reinterpret_cast<uintptr_t>(o.stream) >> 4) ^ (uint64_t)reinterpret_cast<uintptr_t>(o.thread) ^
                 (o.capture << 20);
    h *= 0x9E3779B97F4A7C15ull;
    for (uint32_t i = (uint32_t)(h >> 40) % kEntries;; i = (i + 1) % kEntries) {  // at least half of the entries are free
      Entry &e = entries_[i];
      if (e.number == 0) {
        if (n_owners_ >= kScratchOwners - (o.capture ? kScratchStreams : 0)) return {-1, -1, 0};
        e.owner = o;
        e.number = ++n_owners_;
      } else if (e.owner.stream != o.stream || e.owner.thread != o.thread || e.owner.capture != o.capture) {
        continue;
      }
      if (want_slot && e.slot == 0 && n_slots_ < kScratchSlots) e.slot = ++n_slots_;
      const uint32_t ring = e.ring;
      for (int i = 0; i < copies; ++i) ring_place(e.ring, bytes);
      return {e.number - 1, want_slot ? e.slot - 1 : -1, ring};
    }
  }

 private:
  static constexpr uint32_t kEntries = 2 * kScratchOwners;
  struct Entry {
    ScratchOwner owner;
    int32_t number, slot;  // from 1 on, 0: none
    uint32_t ring;
  };
  Entry entries_[kEntries];
  int32_t n_owners_, n_slots_;
};

#endif

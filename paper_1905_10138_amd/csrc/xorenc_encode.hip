// GPU encoder: Algorithm 1 (patch searching, Section 3.3 of arXiv 1905.10138) for every slice,
// one slice per lane.
//
// Per slice the accepted equations are kept in row-echelon form in LDS: basis[j] is the accepted
// (reduced) row whose lowest set coefficient is column j.  A new care-bit equation
// (M_i | w_i) is reduced against the basis in ascending pivot order; if its coefficients vanish
// it is either redundant (right-hand side 0) or contradicts the accepted ones (right-hand side
// 1): then it is dropped and position i becomes a patch.  Otherwise it joins the basis.  After
// the last care bit, back-substitution with every free variable 0 gives w^c, which is the
// solution the reduced row-echelon form of the accepted rows yields.
//
// Second encoder (Section 5.2, minimising n_patch for small n_in): the input with the fewest mismatched care bits,
// the smallest one read as an integer among equals.  A slice on which Algorithm 1 drops nothing has a solution
// without mismatches, and back-substitution gives the smallest such input: its pivots are the columns that are not
// sums of lower columns, so a free variable (a sum of lower columns) can be 0 whatever the higher variables are and
// a pivot variable is determined by the higher ones.  Only the other slices are searched.  Those with at most 32 care
// bits are tried by syndrome first (fewest_patches): sets of one, two, three care bits whose flips make the equations
// solvable.  The rest are listed, and every one of the 2^n_in inputs is tried on them as a matrix product on the matrix
// cores (exhaustive_search_kernel).
#include <hip/hip_runtime.h>

#include <mutex>

#include "xorenc_device.h"
#include "xorenc_encode_plan.h"

// Scratch area of xorenc_encode_static: device memory that every GPU holds from the time the library is loaded.
// In host code the array's name is only a handle for hipGetSymbolAddress; kernels get the looked-up address.
static __device__ __align__(256) unsigned char scratch[XORENC_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;

// Address of `scratch` on the current device, looked up once per device (with that device current).
int32_t static_scratch_address(void **out) {
  static std::mutex lock;
  static void *address[kMaxDevices] = {};
  int dev = -1;
  const hipError_t ed = hipGetDevice(&dev);
  if (ed != hipSuccess) return xorenc_internal_hip_status((int32_t)ed);
  if (dev < 0 || dev >= kMaxDevices) return XORENC_EUNSUPPORTED;
  std::lock_guard<std::mutex> guard(lock);
  if (!address[dev]) {
    void *p = nullptr;
    const hipError_t es = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (es != hipSuccess) return xorenc_internal_hip_status((int32_t)es);
    if (!p) return XORENC_EHIP;
    address[dev] = p;
  }
  *out = address[dev];
  return XORENC_OK;
}

// The patch counts that the slices leave for the offsets (encode_plan): 2-byte counts (a unit has at most 2048 patches),
// and totals per counting block, the ENC_UNITS * J units that a workgroup covers in one plane, in flattened (plane,
// block) order.
struct Counts {
  uint16_t *unit;     // [q*n_units], null with one unit per plane: its count is the total of its block
  uint32_t *block;    // [q*n_blocks]
  uint32_t *scanned;  // [q*n_blocks + 1]: exclusive sums of `block` (only when there are many blocks)
  int32_t n_units, n_blocks;
};

struct EncParams {
  const uint64_t *mask;
  const uint64_t *planes;
  uint8_t *enc;
  uint64_t *pbits;      // [q][n_slots] patch bitmaps (workspace); only units with patches are written and read
  Counts counts;
  int64_t n_slots, n_eslots;
  int32_t n_in, J;
  uint32_t M_rows[XORENC_MAX_N_OUT];
};

// First word of slice `eslot` = (rb*espr + S)*32 + rr of a plane: word w of it is slot ((rb*espr + S)*J + w)*32 + rr.
__device__ inline int64_t first_word(int64_t eslot, int J) { return (eslot >> 5) * J * 32 + (eslot & 31); }

// A pass over the slices [first, first + n) of every plane (n a multiple of 32, n*q < 2^32) numbers them plane by
// plane, entry = plane*n + slice - first; this is the first word of one in [q][n_slots].
__device__ inline int64_t entry_word(uint32_t entry, int64_t first, uint32_t n, int64_t n_slots, int J) {
  const uint32_t p = entry / n;
  return p * n_slots + first_word(first + (entry - p * n), J);
}

// Patches of the 32 slices of a unit (one per lane of a half wave): count for the unit and its block, bitmaps if there
// are any.  Every lane of the wave calls this with the same w; `block_total` is LDS.  The slices' counts are added up bit by
// bit with scalar instructions (most are 0 or 1).
__device__ inline void put_patches(uint64_t *pbits, const Counts &c, int p, int64_t slot, uint64_t patches, bool valid,
                                   uint32_t *block_total) {
  const uint32_t mine = (uint32_t)__builtin_popcountll(patches);
  uint32_t low = 0, high = 0;  // uniform: of the wave's two units
  for (int k = 0; k < 7; ++k) {
    const uint64_t have = __ballot((mine >> k) & 1u);
    low += (uint32_t)__builtin_popcount((uint32_t)have) << k;
    high += (uint32_t)__builtin_popcount((uint32_t)(have >> 32)) << k;
    if (!__ballot(mine >> (k + 1))) break;  // uniform
  }
  const uint32_t cnt = threadIdx.x & 32 ? high : low;
  if (valid && cnt) pbits[slot] = patches;
  if (valid && c.unit && (threadIdx.x & 31) == 0)
    c.unit[(int64_t)p * c.n_units + (slot - (int64_t)p * c.n_units * 32) / 32] = (uint16_t)cnt;
  if (low + high && (threadIdx.x & 63) == 0) atomicAdd(block_total, low + high);
}

// Fewest patches of one slice by syndrome: a wave, a care bit per lane, at most 32 of them (the equation of a lane's care
// bit in `row`, the wanted bit on top; 0 beyond the last).  The rows are brought to reduced echelon form, pivots in ascending
// columns; `sums` are the equations a reduced row is the sum of.  Where the coefficients of a reduced row vanish, its right-hand
// side has to be 0: the flips of a set of care bits must change exactly those that are 1 (the syndrome), and change the
// solution with free variables 0, the smallest one for this set, by the sum of the bits' columns.  The sets of one care bit
// are tried, then of two and of three; the first size with a match is the minimum and its smallest solution the answer.
// Returns false, for the whole wave, when no set of three or fewer matches.
//
// Bound: the chain of cross-lane reads, about 2 us a slice.  A search takes 2^n_in inputs: the 1500 of 360000 slices of
// 16384 x 4096, S = 0.95, n_out = 192, n_in = 20 that need patches took 220 us of matrix instructions, now the pass over all
// slices, which hides these waves behind its others, is 0.5 us longer and the search kernel returns after 4.5 us.
__device__ bool fewest_patches(uint32_t row, int n_care, int n_in, uint32_t *x_out) {
  const int lane = threadIdx.x & 63;
  uint32_t sums = lane < n_care ? 1u << lane : 0u;
  uint64_t pivots = 0;  // lanes whose row is a pivot row
  uint32_t pivot_bit = 0;
  for (int j = 0; j < n_in; ++j) {  // uniform
    const bool set = (row >> j) & 1u;
    const uint64_t from = __ballot(set) & ~pivots;
    if (!from) continue;
    const int k = __builtin_ctzll(from);
    pivots |= 1ull << k;
    const uint32_t pivot_row = __builtin_amdgcn_readlane(row, k), pivot_sums = __builtin_amdgcn_readlane(sums, k);
    if (lane == k) {
      pivot_bit = 1u << j;
    } else if (set) {
      row ^= pivot_row;
      sums ^= pivot_sums;
    }
  }
  // columns: what flipping this lane's care bit changes, in the vanished rows (numbered) and in the solution
  uint32_t change = 0, change_x = 0, syndrome = 0, x0 = 0, number = 1;
  for (int k = 0; k < n_care; ++k) {  // uniform
    const uint32_t in = ((uint32_t)__builtin_amdgcn_readlane(sums, k) >> (lane & 31)) & 1u;
    const uint32_t rhs = (uint32_t)__builtin_amdgcn_readlane(row, k) >> 31;
    const uint32_t bit = __builtin_amdgcn_readlane(pivot_bit, k);
    if (bit) {
      change_x |= in * bit;
      x0 |= rhs * bit;
    } else {
      change |= in * number;
      syndrome |= rhs * number;
      number <<= 1;
    }
  }
  uint32_t best = 0xffffffffu;
  if (lane < n_care && change == syndrome) best = x0 ^ change_x;
  if (!__ballot(best != 0xffffffffu)) {
    for (int i = 0; i < n_care; ++i) {
      const uint32_t want = syndrome ^ __builtin_amdgcn_readlane(change, i);
      if (lane < n_care && change == want) best = min(best, x0 ^ change_x ^ __builtin_amdgcn_readlane(change_x, i));
    }
  }
  if (!__ballot(best != 0xffffffffu)) {
    for (int i = 0; i < n_care; ++i) {
      const uint32_t want_i = syndrome ^ __builtin_amdgcn_readlane(change, i);
      const uint32_t x_i = x0 ^ __builtin_amdgcn_readlane(change_x, i);
      for (int k = i + 1; k < n_care; ++k) {
        const uint32_t want = want_i ^ __builtin_amdgcn_readlane(change, k);
        if (lane < n_care && change == want) best = min(best, x_i ^ change_x ^ __builtin_amdgcn_readlane(change_x, k));
      }
    }
  }
  if (!__ballot(best != 0xffffffffu)) return false;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) best = min(best, (uint32_t)__shfl_xor((int)best, o, 64));
  *x_out = best;
  return true;
}

// Algorithm 1 on slices with at most kFewCare care bits, a lane each (n_in + Q <= 27).  Slot t holds what the t-th equation
// of the lane's slice became, or 0 if it was dropped or redundant: from bit 5 on its coefficients and above them the planes'
// right-hand sides, in the lowest five bits the place of its pivot, the lowest coefficient.  An equation is reduced against
// the slots before it in their order: a slot has no bit at the pivots of those before it, so a cleared pivot stays cleared,
// and what remains is the one equation of its kind without bits at pivots, as in the other order.  All slots are registers
// and a reduction step is two instructions (the bit at the pivot spread over a word, of whose shift the instruction takes
// the lowest five bits, and and-xor), where a chain of LDS reads took about 300 cycles.
//
// Bound: instructions, about 34 and two per slot before it for an equation, of the slice with the most care bits in the
// wave; with few waves the latency of the words' and the network's loads, which travel together.  us for the kernels of a call,
// all in LDS / so: 2048 x 2048, S = 0.91, n_in = 16 14.9 / 10.0; 4096 x 4096, three planes, S = 0.8, n_in = 24 33.2 / 26.0;
// 16384 x 4096, two planes, S = 0.95, n_in = 8 33.2 / 31.6.  Slices with more than 32 care bits would need more registers than
// eight waves have (24 slots: 38 us for the second, a few slices had more); what they cost beside the others stands below.
constexpr int kFewCare = 32;
constexpr int kPivotBits = 5;
constexpr bool has_few_care(int Q, int J) { return J * (1 + 2 * Q) <= 10; }  // (the words of wider ones fill the registers)

template <int Q, int J, bool LISTS>
struct FewCare {
  uint64_t kept[J], bits[J][Q];         // in: care bits, wanted bits
  uint64_t patches[LISTS ? J : 1][Q];   // out, LISTS: the dropped equations
  uint32_t dropped;                     // out, else: bit p: plane p has any
  uint32_t x[Q];                        // out: the solution with free variables 0

  // rows: the network's, in LDS; n_care: of the lane's slice; steps: most care bits of a slice of the wave (uniform)
  __device__ inline void solve(const uint32_t *rows, int n_in, uint32_t coefs, int n_care, int steps) {
    uint32_t slot[kFewCare];
    coefs <<= kPivotBits;
    n_in += kPivotBits;
    int word = 0;          // the lane's word of the slice (J > 1)
    uint64_t left = kept[0], now[Q];
#pragma unroll
    for (int p = 0; p < Q; ++p) now[p] = bits[0][p];
    dropped = 0;
#pragma unroll
    for (int w = 0; w < (LISTS ? J : 0); ++w)
#pragma unroll
      for (int p = 0; p < Q; ++p) patches[w][p] = 0;
    auto next_word = [&] {
      if constexpr (J > 1) {
#pragma unroll
        for (int k = 1; k < J; ++k) {  // (an empty word may follow)
          if (!__ballot(left == 0 && word < J - 1)) break;  // uniform
          const bool go = left == 0 && word < J - 1;
          word += go ? 1 : 0;
#pragma unroll
          for (int w = 1; w < J; ++w)
            if (go && word == w) {
              left = kept[w];
#pragma unroll
              for (int p = 0; p < Q; ++p) now[p] = bits[w][p];
            }
        }
      }
    };
    // the next equation: its row of the network and right-hand sides (whatever it is behind the lane's last one)
    int at = 0, at_word = 0;
    uint32_t row = 0;
    auto fetch = [&] {
      next_word();
      at = (int)__builtin_ctzll(left | 1ull << 63);
      asm volatile("" : "+v"(at));  // (compared as 32 bits)
      at_word = word;
      left &= left - 1;
      row = rows[(J > 1 ? 64 * word : 0) + at] << kPivotBits;
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t half = at < 32 ? (uint32_t)now[p] : (uint32_t)(now[p] >> 32);
        row |= __builtin_amdgcn_ubfe(half, (uint32_t)at, 1u) << (n_in + p);
      }
    };
    fetch();
#pragma unroll
    for (int t = 0; t < kFewCare; ++t) {
      if (t < steps) {  // uniform
        uint32_t r = t < n_care ? row : 0u;
        const int i = at, w_i = at_word;
        if (t + 1 < kFewCare) fetch();
#pragma unroll
        for (int k = 0; k < t; ++k) r ^= (uint32_t)__builtin_amdgcn_sbfe((int)r, slot[k], 1u) & slot[k];
        const bool gone = (r & coefs) == 0;
        if (__ballot(gone && r >> kPivotBits)) {  // uniform: the equation is dropped where its right-hand side is 1
          const uint32_t rhs = gone ? r >> n_in : 0u;
          if constexpr (LISTS) {
#pragma unroll
            for (int w = 0; w < J; ++w)
#pragma unroll
              for (int p = 0; p < Q; ++p)
                if (J == 1 || w == w_i) patches[w][p] |= (uint64_t)((rhs >> p) & 1u) << i;
          } else {
            dropped |= rhs;
          }
        }
        const uint32_t pivots = 0xffffffffu >> (32 - kPivotBits);
        slot[t] = gone ? 0u : (r & ~pivots) | (uint32_t)__builtin_ctz((r & ~pivots) | 1u << 31);
      }
    }
    // back-substitution, last slot first: a slot's other bits are free columns and pivots of later slots
#pragma unroll
    for (int p = 0; p < Q; ++p) x[p] = 0;
#pragma unroll
    for (int t = kFewCare - 1; t >= 0; --t) {
      if (t < steps) {  // uniform
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t sum = (uint32_t)__builtin_popcount(slot[t] & coefs & x[p]) + (slot[t] >> (n_in + p));
          x[p] |= (sum & 1u) << (slot[t] & 31u);
        }
      }
    }
#pragma unroll
    for (int p = 0; p < Q; ++p) x[p] >>= kPivotBits;
  }
};

// Algorithm 1.  The planes share the mask, so the coefficients of a slice's equations, which of them join the basis
// and the pivots are the same for all planes: one elimination with Q right-hand sides, which travel in the bits above
// the n_in coefficients of a row (PACKED: n_in + Q <= 32) or as bits per pivot in a register per plane.
//
// Waves whose slices have few care bits keep everything in registers (FewCare).  The others' bound is the chain of dependent
// LDS reads of a reduction (one per set pivot) and the longest of 64 slices in a wave.  The network's rows are read from LDS
// (they used to be fetched from the kernel arguments with a vector load per equation), and the basis takes n_in KB of
// LDS instead of 32.  JT: words per slice in the kernels that have the registers (one word with any number of planes, two with
// one and two, three with one, see has_few_care, and n_in + Q <= 27); 0: any number of words, everything in LDS.
//
// SEARCH: first pass of the encoder with the fewest patches, over the slices [first, first + n).  The low half of a
// slice's first patch word becomes its key: the solution x (below 2^24) when nothing was dropped, x with the lowest bit of
// the mismatch count set when syndromes gave the fewest patches, otherwise all ones, and the slice joins the list, whose
// entry i is the high half of the first patch word of slice i of the pass's numbering; *list_len counts them.  The
// workgroup's waves take turns at the slices that are tried by syndrome (syndrome_care says which).
// The first pass for one and two words is kept to eight waves a SIMD: beyond 100 scalar or 64 vector registers a SIMD has room for
// seven, and a launch of eight workgroups per CU ran in two rounds (us for the kernels of a search, as many registers as it
// takes / eight waves: 16384 x 4096, two planes, n_out = 128, n_in = 16, S = 0.91 228 / 213, S = 0.85 1803 / 1703).  With three
// words it takes 86 million weights to have so many workgroups, and fewer registers cost 0.6 us (one
// plane, n_out = 192, n_in = 20 41.5 / 42.2).
constexpr bool at_eight_waves(bool search, int JT) { return search && (JT == 1 || JT == 2); }

template <int Q, bool PACKED, bool SEARCH, int JT>
__global__ __launch_bounds__(ENC_THREADS, at_eight_waves(SEARCH, JT) ? 8 : 1) void encode_slices_kernel(
    EncParams P, int64_t first, int64_t n, uint32_t *list_len, SyndromeCare care) {
  extern __shared__ uint32_t enc_lds[];  // [n_in][ENC_THREADS] basis, then the 64 J rows of the network
  __shared__ uint32_t block_total[Q];
  uint32_t *const rows = enc_lds + P.n_in * ENC_THREADS;
  const int tid = threadIdx.x;
  if (tid < Q) block_total[tid] = 0;
  const int64_t rel = (int64_t)blockIdx.x * ENC_THREADS + tid;
  const bool valid = rel < n;
  const int64_t eslot = first + (valid ? rel : 0);
  const int l_J = JT ? JT : P.J;
  const int64_t slot0 = first_word(eslot, l_J);
  const int n_in = P.n_in;
  const uint32_t coefs = n_in < 32 ? (1u << n_in) - 1u : 0xffffffffu;
  uint32_t *const basis = enc_lds + tid;  // row with pivot j at basis[j * ENC_THREADS]
  // the slice's words are requested before the network's rows are staged: they travel together
  uint64_t kept_all[JT ? JT : 1], bits_all[JT ? JT : 1][Q];
  int n_care = 0;
#pragma unroll
  for (int w = 0; w < JT; ++w) {
    kept_all[w] = valid ? P.mask[slot0 + 32 * w] : 0ull;
#pragma unroll
    for (int p = 0; p < Q; ++p) bits_all[w][p] = valid ? P.planes[p * P.n_slots + slot0 + 32 * w] : 0ull;
  }
  for (int i = tid; i < 64 * l_J; i += ENC_THREADS) rows[i] = P.M_rows[i];
  __syncthreads();

  bool dropped[Q] = {};
  uint32_t x[Q] = {};
#pragma unroll
  for (int w = 0; w < JT; ++w) n_care += __builtin_popcountll(kept_all[w]);
  asm volatile("" : "+v"(n_care));  // (compared as 32 bits)
  if (JT && !__ballot(n_care > kFewCare)) {  // uniform
    if constexpr (JT != 0) {
      constexpr bool LISTS = !at_eight_waves(SEARCH, JT);
      FewCare<Q, JT, LISTS> few;
#pragma unroll
      for (int w = 0; w < JT; ++w) {
        few.kept[w] = kept_all[w];
#pragma unroll
        for (int p = 0; p < Q; ++p) few.bits[w][p] = bits_all[w][p];
      }
      int steps = 0;  // the largest n_care
      for (int s = 32; s > 0; s >>= 1) steps += __ballot(n_care >= steps + s) ? s : 0;
      few.solve(rows, n_in, coefs, n_care, steps);
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        x[p] = few.x[p];
        if constexpr (!LISTS) dropped[p] = (few.dropped >> p) & 1u;
      }
      if constexpr (LISTS) {
#pragma unroll
        for (int w = 0; w < JT; ++w) {
#pragma unroll
          for (int p = 0; p < Q; ++p) {
            dropped[p] = dropped[p] || few.patches[w][p] != 0;
            if constexpr (!SEARCH)
              put_patches(P.pbits, P.counts, p, p * P.n_slots + slot0 + 32 * w, few.patches[w][p], valid, block_total + p);
          }
        }
      }
    }
  } else {
    // These waves take the longest and mostly wait: beside waves that solve in registers they issue first (us for the kernels
    // of a call, without / with the registers, the last with the words read twice and no priority: 16384 x 4096, n_out = 192,
    // S = 0.91, n_in = 20 47.6 / 40.8 / 56.3; 4096 x 4096, S = 0.7, n_in = 24 36.8 / 34.0 / 45.1; 8192 x 4096, two planes,
    // n_out = 128, S = 0.85, n_in = 24 48.3 / 44.8 / 54.2; where no wave is such, S = 0.9 and n_in = 16, nothing changes).
    if constexpr (JT != 0) __builtin_amdgcn_s_setprio(3);
    uint32_t have = 0;         // bit j: a basis row with pivot j exists
    uint32_t rhsbits[Q] = {};  // !PACKED: bit j = right-hand side of that row
    for (int w = 0; w < l_J; ++w) {  // uniform; care bits in ascending position over the whole slice
      const int64_t slot = slot0 + 32 * w;
      uint64_t kept, bits[Q], patches[Q] = {};  // kept: care bits
      if constexpr (JT == 0) {
        kept = valid ? P.mask[slot] : 0ull;
        if constexpr (SEARCH) n_care += __builtin_popcountll(kept);
#pragma unroll
        for (int p = 0; p < Q; ++p) bits[p] = valid ? P.planes[p * P.n_slots + slot] : 0ull;
      } else {
        kept = kept_all[0];
#pragma unroll
        for (int p = 0; p < Q; ++p) bits[p] = bits_all[0][p];
#pragma unroll
        for (int k = 1; k < JT; ++k)
          if (w == k) {  // uniform
            kept = kept_all[k];
#pragma unroll
            for (int p = 0; p < Q; ++p) bits[p] = bits_all[k][p];
          }
      }
      while (kept) {
        const int i = __builtin_ctzll(kept);
        kept &= kept - 1;
        uint32_t row = rows[64 * w + i];
        uint32_t rhs = 0;  // bit p: plane p
#pragma unroll
        for (int p = 0; p < Q; ++p) rhs |= (uint32_t)((bits[p] >> i) & 1) << p;
        if constexpr (PACKED) row |= rhs << n_in;
        uint32_t t = row & have;
        while (t) {  // reduce, ascending pivots (a basis row has no bit below its pivot)
          const int j = __builtin_ctz(t);
          row ^= basis[j * ENC_THREADS];
          if constexpr (!PACKED) {
#pragma unroll
            for (int p = 0; p < Q; ++p) rhs ^= ((rhsbits[p] >> j) & 1u) << p;
          }
          t = row & have;
        }
        if ((row & coefs) == 0) {  // 0 ... 0 | rhs: the equation is dropped where that is 1
          if constexpr (PACKED) rhs = row >> n_in;
#pragma unroll
          for (int p = 0; p < Q; ++p) patches[p] |= (uint64_t)((rhs >> p) & 1u) << i;
          continue;
        }
        const int piv = __builtin_ctz(row);
        basis[piv * ENC_THREADS] = row;
        have |= 1u << piv;
        if constexpr (!PACKED) {
#pragma unroll
          for (int p = 0; p < Q; ++p) rhsbits[p] |= ((rhs >> p) & 1u) << piv;
        }
      }
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        dropped[p] = dropped[p] || patches[p] != 0;
        if constexpr (!SEARCH)
          put_patches(P.pbits, P.counts, p, p * P.n_slots + slot, patches[p], valid, block_total + p);
      }
    }
    // back-substitution, free variables = 0, highest pivot first
    uint32_t t = have;
    while (t) {
      const int j = 31 - __builtin_clz(t);
      t &= ~(1u << j);
      const uint32_t row = basis[j * ENC_THREADS];
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t others = row & coefs & x[p];  // pivots above j already solved; free ones are 0
        const uint32_t rhs = PACKED ? row >> (n_in + p) : rhsbits[p] >> j;
        x[p] |= ((rhs ^ (uint32_t)__builtin_popcount(others)) & 1u) << j;
      }
    }
    if constexpr (JT != 0) __builtin_amdgcn_s_setprio(0);
  }
#pragma unroll
  for (int p = 0; p < Q; ++p) store_enc_unit(P.enc, p * P.n_eslots + eslot, n_in, x[p], valid);
  if constexpr (SEARCH) {
    uint32_t *const halves = reinterpret_cast<uint32_t *>(P.pbits);
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The basis is not needed any more: its place takes the slices to be tried by syndrome (tid << 8 | care bits << 2 |
    // plane) and a slice's equations per wave.  (n_in KB; the queue takes 1 KB per plane at most, and n_in is above ten.)
    uint32_t *const queue = enc_lds + 32 * (ENC_THREADS / 64);
    uint32_t *const queued = &block_total[0];  // (no counts are made in this pass)
    auto put_on_list = [&](bool put, int p, int64_t entry_rel) {
      const uint64_t listed = __ballot(put);
      if (!listed) return;  // uniform
      const int leader = __builtin_ctzll(listed);
      uint32_t base = 0;
      if (lane == leader) base = atomicAdd(list_len, (uint32_t)__builtin_popcountll(listed));
      base = (uint32_t)__shfl((int)base, leader, 64);
      if (put) {
        const uint32_t at = base + (uint32_t)__builtin_popcountll(listed & ((1ull << lane) - 1ull));
        halves[2 * entry_word(at, first, (uint32_t)n, P.n_slots, P.J) + 1] = (uint32_t)(p * n + entry_rel);
      }
    };
    __syncthreads();
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const bool search = valid && dropped[p];
      if (valid) halves[2 * (p * P.n_slots + slot0)] = search ? 0xffffffffu : x[p];
      const bool by_syndrome = search && n_care <= care.few;
      if (by_syndrome) queue[atomicAdd(queued, 1u)] = (uint32_t)tid << 8 | (uint32_t)n_care << 2 | (uint32_t)p;
      put_on_list(search && !by_syndrome, p, rel);
    }
    __syncthreads();
    const uint32_t n_queued = __builtin_amdgcn_readfirstlane(*queued);
    const int most_care = n_queued <= (uint32_t)kSyndromeFew ? care.few : care.many;  // uniform for the workgroup
    if (most_care < care.few) {
      for (uint32_t i0 = 0; i0 < n_queued; i0 += ENC_THREADS) {  // uniform
        const uint32_t e = i0 + tid < n_queued ? queue[i0 + tid] : 0u;
        put_on_list((int)((e >> 2) & 63u) > most_care, (int)(e & 3u), (int64_t)blockIdx.x * ENC_THREADS + (e >> 8));
      }
    }
    uint32_t *const eqs = enc_lds + 32 * wave;
    for (uint32_t i = wave; i < n_queued; i += ENC_THREADS / 64) {  // uniform per wave
      const uint32_t e = __builtin_amdgcn_readfirstlane(queue[i]);
      if ((int)((e >> 2) & 63u) > most_care) continue;
      const int p = (int)(e & 3u);
      const int64_t r = (int64_t)blockIdx.x * ENC_THREADS + (e >> 8);
      const int64_t word = first_word(first + r, P.J);
      // lane = bit position; the care bits' equations move to lanes 0, 1, ...
      int n_eqs = 0;
      for (int w = 0; w < P.J; ++w) {  // uniform
        const uint64_t kept = P.mask[word + 32 * w], bits = P.planes[p * P.n_slots + word + 32 * w];
        if ((kept >> lane) & 1)
          eqs[n_eqs + __builtin_popcountll(kept & ((1ull << lane) - 1ull))] =
              rows[64 * w + lane] | (uint32_t)((bits >> lane) & 1) << 31;
        n_eqs += __builtin_popcountll(kept);
      }
      n_eqs = __builtin_amdgcn_readfirstlane(n_eqs);
      __builtin_amdgcn_wave_barrier();  // (LDS operations of a wave execute in order)
      uint32_t xs = 0;
      const bool found = fewest_patches(lane < n_eqs ? eqs[lane] : 0u, n_eqs, n_in, &xs);
      __builtin_amdgcn_wave_barrier();
      if (found) {  // uniform
        if (lane == 0) halves[2 * (p * P.n_slots + word)] = 1u << 24 | xs;
      } else {
        put_on_list(lane == 0, p, r);
      }
    }
  } else {
    __syncthreads();
    if (tid < Q) P.counts.block[tid * P.counts.n_blocks + blockIdx.x] = block_total[tid];
  }
}

struct ExhParams {
  const uint64_t *mask;
  const uint64_t *planes;
  uint8_t *enc;
  uint64_t *pbits;
  Counts counts;
  int64_t n_slots, n_eslots;
  int32_t n_in, q;
  uint64_t Mcol[XORENC_MAX_J][XORENC_EXH_MAX_N_IN];  // [w][j]: bit i = M[64 w + i][j]
  uint64_t used[XORENC_MAX_J];                       // [w]: bit i = row 64 w + i of M is not zero
};

typedef __attribute__((ext_vector_type(8))) int32_t i32x8;

__global__ void exhaustive_reset_kernel(uint32_t *list_len) { *list_len = 0; }

// All 2^n_in inputs on the listed slices, 128 slices and 2^c consecutive inputs per item of work of a wave.
//
// With A[x][i] = (-1)^(output bit i of the network for input x) and B[i][s] = -(-1)^(wanted bit i of slice s) on care
// bits, 0 elsewhere, (A B)[x][s] = 2 mismatches - care bits: a product on the matrix cores in FP4, 32 inputs x 32
// slices x 64 bits per instruction.  A's block scale is 2^14 and the accumulator starts at the input's number in its
// tile (and the shift that keeps it positive), so a result plus 32 * tile is a float that holds the pair (mismatches,
// input) exactly (2 * 2^14 * 256 + 2^15 < 2^24; all terms are integers) and its minimum is the answer: half a v_min3_u32
// on the bit patterns per input and slice.  Rows of M that are zero mismatch or match whatever
// the input is and stay out, so that at most half of the care bits can be mismatched at the minimum over all inputs and
// its key (mismatches + 1) << 24 | input fits 32 bits; the minimum over one item's inputs can mismatch all 256, but not win, and its key is held at 255 << 24.  Tiles are visited in Gray
// code order: one column of M flips the signs of A (4 XORs per 64 bits, shared by the four slice tiles).
//
// Bound: VALU issue beside the matrix instructions.  Every slice of 16384 x 4096, n_out = 192, n_in = 20 used to be
// searched, one slice per lane, at 2J AND, 2J XOR and 2J population counts per input: 219 ms for the call, 0.30 ms with the
// slices that need patches in this kernel, 0.09 ms since syndromes leave it those they do not solve (16384 x 4096 with half
// of the weights kept, n_out = 64, n_in = 16, where nearly every slice is searched here: 14 and 5 ms).
// The width of an item falls from 2^15 to 2^10 inputs when there are too few slices to give every wave eight items.
// ALL: every slice of the pass is searched, in one item each and without a list.  With few inputs that is cheaper than
// the elimination that would sort out the slices that need no search, however few these are, and than joining the list
// (kAllMaxNIn; us for the kernels of a call, all slices / with the list: 16384 x 4096, S = 0.95, n_in = 8 34 / 199, n_in =
// 10 55 / 124, with n_out = 192 47 / 117; S = 0.8, n_in = 10 60 / 254; 1024 x 1024, S = 0.9, n_in = 8 13 / 26).
constexpr int kAllMaxNIn = 10;
static_assert(32 * (ENC_THREADS / 64) + XORENC_MAX_Q * ENC_THREADS <= (kAllMaxNIn + 1) * ENC_THREADS,
              "equations and queue of the slices tried by syndrome take the place of the basis");

template <int J, bool ALL>
__global__ __launch_bounds__(ENC_THREADS, 2) void exhaustive_search_kernel(ExhParams P, int64_t first, int64_t n,
                                                                          const uint32_t *list_len) {
  constexpr int NS = 4;                                   // slice tiles of a wave
  constexpr int COLS = XORENC_EXH_MAX_N_IN - 5;           // columns that change from tile to tile
  constexpr int kShift = J * 64 << 14;                    // keeps the accumulators positive
  __shared__ uint4 flip_s[COLS][J][2];                    // sign bits of column 5 + c, per half of a word
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, rl = lane & 31;
  auto sign_bits = [](uint32_t y, int d) { return ((y >> d) & 0x11111111u) << 3; };
  for (int i = tid; i < COLS * J * 2; i += ENC_THREADS) {
    const int c = i / (2 * J), w = (i >> 1) % J, h = i & 1;
    const uint32_t y = (uint32_t)(P.Mcol[w][5 + c] >> (32 * h));
    flip_s[c][w][h] = make_uint4(sign_bits(y, 0), sign_bits(y, 1), sign_bits(y, 2), sign_bits(y, 3));
  }
  __syncthreads();
  const uint32_t n_list = ALL ? (uint32_t)P.q * (uint32_t)n : *list_len;
  const int64_t groups = ((int64_t)n_list + 32 * NS - 1) / (32 * NS);
  const int64_t waves = (int64_t)gridDim.x * (ENC_THREADS / 64);
  int c = P.n_in < 15 ? (P.n_in > 5 ? P.n_in : 5) : 15;
  while (!ALL && c > 10 && (groups << (P.n_in - c)) < 8 * waves) --c;
  const int chunk_bits = P.n_in > c ? P.n_in - c : 0;
  const uint32_t tiles = 1u << (c - 5);

  const uint32_t *const halves = reinterpret_cast<const uint32_t *>(P.pbits);
  uint32_t *const keys = reinterpret_cast<uint32_t *>(P.pbits);
  // row rl of A for the inputs 0..31 (columns beyond n_in are zero: with n_in = 4 the inputs 16..31 repeat 0..15)
  uint32_t base[J];
#pragma unroll
  for (int w = 0; w < J; ++w) {
    base[w] = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j)
      base[w] ^= ((rl >> j) & 1) ? (uint32_t)(P.Mcol[w][j] >> (32 * g)) : 0u;
  }
  f32x16 number;
#pragma unroll
  for (int i = 0; i < 16; ++i) number[i] = (float)(kShift + 8 * (i / 4) + 4 * g + i % 4);

  for (int64_t item = (int64_t)blockIdx.x * (ENC_THREADS / 64) + (tid >> 6); item < (groups << chunk_bits);
       item += waves) {  // uniform per wave
    const int64_t group = item >> chunk_bits;
    const uint32_t chunk = (uint32_t)(item & ((1 << chunk_bits) - 1));
    // ---- the four slice tiles: column rl of tile t is list entry group*128 + 32 t + rl
    i32x8 b[NS][J];
    uint32_t care_bits[NS];
    int64_t word[NS];                                     // first word of the slice in [q][n_slots]
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int64_t li = group * (32 * NS) + 32 * t + rl;
      const bool valid = li < n_list;
      uint32_t entry = 0u;
      if (valid) entry = ALL ? (uint32_t)li : halves[2 * entry_word((uint32_t)li, first, (uint32_t)n, P.n_slots, J) + 1];
      word[t] = entry_word(entry, first, (uint32_t)n, P.n_slots, J);
      const int64_t mask_word = word[t] - entry / (uint32_t)n * P.n_slots;
      care_bits[t] = 0;
#pragma unroll
      for (int w = 0; w < J; ++w) {
        uint32_t care = reinterpret_cast<const uint32_t *>(P.mask)[2 * (mask_word + 32 * w) + g];
        const uint32_t want = reinterpret_cast<const uint32_t *>(P.planes)[2 * (word[t] + 32 * w) + g];
        care &= (uint32_t)(P.used[w] >> (32 * g));
        if (!valid) care = 0;
        care_bits[t] += __builtin_popcount(care);
        const uint32_t minus = care & ~want;
#pragma unroll
        for (int d = 0; d < 4; ++d) b[t][w][d] = (int32_t)((((care >> d) & 0x11111111u) << 1) | sign_bits(minus, d));
#pragma unroll
        for (int d = 4; d < 8; ++d) b[t][w][d] = 0;
      }
      care_bits[t] += (uint32_t)__shfl_xor((int)care_bits[t], 32, 64);
    }
    // ---- A of the chunk's first tile
    const uint32_t tile0 = chunk << (c - 5);
    i32x8 a[J];
#pragma unroll
    for (int w = 0; w < J; ++w) {
#pragma unroll
      for (int d = 0; d < 4; ++d) a[w][d] = (int32_t)(0x22222222u | sign_bits(base[w], d));
#pragma unroll
      for (int d = 4; d < 8; ++d) a[w][d] = 0;
    }
    auto flip = [&](int col) {
#pragma unroll
      for (int w = 0; w < J; ++w) {
        const uint4 f = flip_s[col][w][g];
        a[w][0] ^= (int32_t)f.x;
        a[w][1] ^= (int32_t)f.y;
        a[w][2] ^= (int32_t)f.z;
        a[w][3] ^= (int32_t)f.w;
      }
    };
    for (uint32_t bits = tile0; bits; bits &= bits - 1) flip(__builtin_ctz(bits));  // uniform
    uint32_t best[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) best[t] = 0xffffffffu;
    for (uint32_t i = 0; i < tiles; ++i) {          // uniform
      const float offset = (float)(32u * (i ^ (i >> 1)));
      f32x16 d[NS];
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        d[t] = number;
#pragma unroll
        for (int w = 0; w < J; ++w)
          d[t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[w], b[t][w], d[t], 4, 4, 0, 127 + 14, 0, 127);
      }
      if (i + 1 < tiles) flip(__builtin_ctz(i + 1));
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        // (positive floats order like their bit patterns; integer minima need no NaN handling)
        uint32_t v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = __float_as_uint(d[t][k]);
        const uint32_t m0 = min(min(v[0], v[1]), v[2]), m1 = min(min(v[3], v[4]), v[5]),
                       m2 = min(min(v[6], v[7]), v[8]), m3 = min(min(v[9], v[10]), v[11]),
                       m4 = min(min(v[12], v[13]), v[14]);
        const uint32_t m = min(min(min(m0, m1), m2), min(min(m3, m4), v[15]));
        best[t] = min(best[t], __float_as_uint(__uint_as_float(m) + offset));
      }
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const float v = __uint_as_float(min(best[t], (uint32_t)__shfl_xor((int)best[t], 32, 64))) - (float)kShift;
      const int64_t li = group * (32 * NS) + 32 * t + rl;
      if (g == 0 && li < n_list) {
        const int32_t pair = (int32_t)v + (int32_t)(care_bits[t] << 14);  // mismatches << 15 | input inside the chunk
        const uint32_t x = (chunk << c) | (uint32_t)(pair & 0x7fff);
        const uint32_t key = (uint32_t)(min(pair >> 15, 254) + 1) << 24 | x;  // (a chunk's minimum may be up to 256)
        if (ALL)
          keys[2 * word[t]] = key;
        else
          atomicMin(keys + 2 * word[t], key);
      }
    }
  }
}

// Keys -> patches, their counts, and the encrypted bits of the slices that were searched.  One plane per grid row.
template <int J>
__global__ __launch_bounds__(ENC_THREADS) void exhaustive_finish_kernel(ExhParams P, int64_t first, int64_t n) {
  __shared__ uint32_t block_total;
  if (threadIdx.x == 0) block_total = 0;
  const int64_t rel = (int64_t)blockIdx.x * ENC_THREADS + threadIdx.x;
  const int p = blockIdx.y;
  const bool valid = rel < n;
  const int64_t eslot = first + (valid ? rel : 0);
  const int64_t slot = first_word(eslot, J), word = p * P.n_slots + slot;
  const uint32_t key = valid ? (uint32_t)P.pbits[word] : 0u;
  const uint32_t x = key & 0xffffffu;
  const bool searched = key >= 1u << 24;
  const bool any = __ballot(searched) != 0ull;  // uniform
  uint64_t wanted[J], kept[J];  // requested together
#pragma unroll
  for (int w = 0; w < J; ++w) {
    wanted[w] = searched ? P.planes[word + 32 * w] : 0ull;
    kept[w] = searched ? P.mask[slot + 32 * w] : 0ull;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < J; ++w) {
    uint64_t patches = 0;
    if (any) {
      uint64_t y = 0;
      // (eight columns at a time: in a loop over the n_in each column was a scalar load to wait for, 9.3 us of kernel for
      // 16384 x 4096, n_out = 192, n_in = 20, now 7.1; two planes, n_out = 128, n_in = 16 16.2 and 11.5; columns beyond
      // n_in are zero)
#pragma unroll
      for (int j0 = 0; j0 < XORENC_EXH_MAX_N_IN; j0 += 8) {
        if (j0 >= P.n_in) break;  // uniform
#pragma unroll
        for (int j = j0; j < j0 + 8; ++j) y ^= ((x >> j) & 1u) ? P.Mcol[w][j] : 0ull;
      }
      patches = (y ^ wanted[w]) & kept[w];
    }
    put_patches(P.pbits, P.counts, p, word + 32 * w, patches, valid, &block_total);
  }
  if (any) store_enc_unit(P.enc, p * P.n_eslots + eslot, P.n_in, x, valid);
  __syncthreads();
  if (threadIdx.x == 0) P.counts.block[p * P.counts.n_blocks + (int)(first / ENC_THREADS) + blockIdx.x] = block_total;
}

// Exclusive scan of counts[0..n) into off[0..n] in three launches and without extra memory.  A block
// covers SCAN_BLOCK consecutive items, SCAN_PER per thread.
//   1. scan_local_kernel: prefix inside each block.  The first item of a block would be 0: that slot of
//      the NEXT block (off[n] for the last block) takes this block's total instead.
//   2. scan_blocks_kernel: one workgroup turns the totals parked in those slots into block offsets,
//      off[b * SCAN_BLOCK] = offset of block b, off[n] = grand total.
//   3. scan_add_kernel: every other item of a block adds the block's offset.
constexpr int SCAN_THREADS = 256, SCAN_PER = 16, SCAN_BLOCK = SCAN_THREADS * SCAN_PER;

__global__ __launch_bounds__(SCAN_THREADS) void scan_local_kernel(const uint32_t *counts, uint32_t *off, int n) {
  __shared__ uint32_t wsum[SCAN_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t first = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)tid * SCAN_PER;
  uint32_t v[SCAN_PER];
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < SCAN_PER; ++i) {
    v[i] = (first + i < n) ? counts[first + i] : 0u;
    sum += v[i];
  }
  // inclusive scan of the thread sums over the wave, then over the block's waves
  uint32_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < SCAN_THREADS / 64; ++w) {
    if (w < wave) before += wsum[w];
    total += wsum[w];
  }
  uint32_t run = before + incl - sum;  // exclusive prefix of this thread's first item inside the block
#pragma unroll
  for (int i = 0; i < SCAN_PER; ++i) {
    if (first + i < n && !(tid == 0 && i == 0)) off[first + i] = run;
    run += v[i];
  }
  if (tid == 0) {
    const int64_t next = ((int64_t)blockIdx.x + 1) * SCAN_BLOCK;
    off[next < n ? next : n] = total;
  }
}

__global__ __launch_bounds__(1024) void scan_blocks_kernel(uint32_t *off, int n, int nblocks) {
  __shared__ uint32_t part[1024];
  const int tid = threadIdx.x;
  // block b's total sits in slot (b+1)*SCAN_BLOCK (or n); thread t owns blocks [a, e)
  const int per = (nblocks + 1023) / 1024;
  const int a = min(nblocks, tid * per), e = min(nblocks, a + per);
  auto slot = [&](int b) {
    const int64_t next = ((int64_t)b + 1) * SCAN_BLOCK;
    return next < n ? next : (int64_t)n;
  };
  uint32_t s = 0;
  for (int b = a; b < e; ++b) s += off[slot(b)];
  part[tid] = s;
  __syncthreads();
  for (int d = 1; d < 1024; d <<= 1) {
    const uint32_t v = (tid >= d) ? part[tid - d] : 0u;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  uint32_t run = part[tid] - s;  // offset of block a
  for (int b = a; b < e; ++b) {
    const uint32_t t = off[slot(b)];
    run += t;
    off[slot(b)] = run;  // = offset of block b+1, or the grand total in off[n]
  }
  if (tid == 0) off[0] = 0u;
}

__global__ __launch_bounds__(SCAN_THREADS) void scan_add_kernel(uint32_t *off, int n) {
  if (blockIdx.x == 0) return;  // block 0's offset is 0
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK;
  const uint32_t add = off[base];
  const int64_t first = base + (int64_t)tid * SCAN_PER;
#pragma unroll
  for (int i = 0; i < SCAN_PER; ++i)
    if (first + i < n && !(tid == 0 && i == 0)) off[first + i] += add;
}

// Offsets of the units' patch lists and the lists themselves.  A workgroup covers `per` counting blocks (at most
// EMIT_UNITS units); where its lists start is the sum of the blocks before it, which it adds up itself instead of three
// scan launches (SCANNED: reads from the scanned totals).  Workgroups run in any order and `off` is written as they
// go: nothing that another one still reads may lie there.
template <bool SCANNED>
__global__ __launch_bounds__(ENC_THREADS) void emit_patches_kernel(const uint64_t *pbits, Counts C, int q, int64_t n_slots,
                                                                  int units_per_block, int per, uint32_t *off,
                                                                  uint16_t *patch, int64_t capacity, uint32_t *total) {
  __shared__ uint32_t wsum[ENC_THREADS / 64], start_s[EMIT_UNITS];
  __shared__ int64_t slot_s[EMIT_UNITS];  // first bitmap of a unit with patches, -1 for the others
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_all = q * C.n_blocks;
  const int block0 = blockIdx.x * per;
  // unit of this thread (tid < EMIT_UNITS): flattened block, plane, unit of the plane
  const int blk = block0 + tid / units_per_block;
  const int p = min(blk, n_all - 1) / C.n_blocks;
  const int64_t u = (int64_t)(blk - p * C.n_blocks) * units_per_block + tid % units_per_block;
  const bool mine = tid < per * units_per_block && blk < n_all && u < C.n_units;
  const uint32_t cnt = !mine ? 0u : C.unit ? C.unit[(int64_t)p * C.n_units + u] : C.block[blk];
  uint32_t before = 0;  // patches of earlier workgroups
  if constexpr (SCANNED) {
    before = C.scanned[block0];
  } else {
    int i = tid;
    for (; i + 7 * ENC_THREADS < block0; i += 8 * ENC_THREADS) {
      uint32_t v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = C.block[i + k * ENC_THREADS];
#pragma unroll
      for (int k = 0; k < 8; ++k) before += v[k];
    }
    for (; i < block0; i += ENC_THREADS) before += C.block[i];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) before += (uint32_t)__shfl_xor((int)before, o, 64);
    if (lane == 0) wsum[wave] = before;
    __syncthreads();
    before = 0;
#pragma unroll
    for (int w = 0; w < ENC_THREADS / 64; ++w) before += wsum[w];
    __syncthreads();
  }
  uint32_t incl = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  if (wave == 1) incl += wsum[0];  // (the units sit in the first two waves)
  const uint32_t start = before + incl - cnt;
  if (tid < EMIT_UNITS) {
    start_s[tid] = start;
    slot_s[tid] = cnt ? p * n_slots + u * 32 : -1;
  }
  if (mine) {
    off[(int64_t)p * C.n_units + u] = start;
    if (p == q - 1 && u == C.n_units - 1) {
      off[(int64_t)q * C.n_units] = start + cnt;
      if (total) __hip_atomic_store(total, start + cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  __syncthreads();
  // a half wave per unit; the bitmaps of its units are requested together
  const int rr = tid & 31, t0 = tid >> 5;
  uint64_t bits[EMIT_UNITS / ENC_UNITS];
#pragma unroll
  for (int k = 0; k < EMIT_UNITS / ENC_UNITS; ++k) {
    const int64_t slot = slot_s[t0 + k * ENC_UNITS];
    bits[k] = slot >= 0 ? pbits[slot + rr] : 0ull;
  }
#pragma unroll
  for (int k = 0; k < EMIT_UNITS / ENC_UNITS; ++k) {
    uint64_t w = bits[k];
    if (!__ballot(w != 0)) continue;  // uniform
    const int c = __builtin_popcountll(w);
    int inc = c;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const int v = __shfl_up(inc, o, 32);
      if (rr >= o) inc += v;
    }
    int64_t pos = (int64_t)start_s[t0 + k * ENC_UNITS] + (inc - c);
    while (w) {
      const int bit = __builtin_ctzll(w);
      w &= w - 1;
      if (pos < capacity) patch[pos] = (uint16_t)((rr << 6) | bit);
      ++pos;
    }
  }
}

template <int Q, bool SEARCH>
void launch_slices(const EncParams &P, int64_t first, int64_t n, uint32_t *list_len, SyndromeCare care, hipStream_t st) {
  const dim3 grid((unsigned)((n + ENC_THREADS - 1) / ENC_THREADS)), block(ENC_THREADS);
  const size_t lds = ((size_t)P.n_in * ENC_THREADS + 64 * P.J) * sizeof(uint32_t);
  const bool packed = P.n_in + Q <= 32, in_slots = P.n_in + Q + kPivotBits <= 32;
  if (in_slots && P.J == 1)
    hipLaunchKernelGGL((encode_slices_kernel<Q, true, SEARCH, 1>), grid, block, lds, st, P, first, n, list_len, care);
  else if (in_slots && P.J == 2 && has_few_care(Q, 2))
    hipLaunchKernelGGL((encode_slices_kernel<Q, true, SEARCH, has_few_care(Q, 2) ? 2 : 0>), grid, block, lds, st, P, first, n, list_len, care);
  else if (in_slots && P.J == 3 && has_few_care(Q, 3))
    hipLaunchKernelGGL((encode_slices_kernel<Q, true, SEARCH, has_few_care(Q, 3) ? 3 : 0>), grid, block, lds, st, P, first, n, list_len, care);
  else if (packed)
    hipLaunchKernelGGL((encode_slices_kernel<Q, true, SEARCH, 0>), grid, block, lds, st, P, first, n, list_len, care);
  else
    hipLaunchKernelGGL((encode_slices_kernel<Q, false, SEARCH, 0>), grid, block, lds, st, P, first, n, list_len, care);
}

template <int J>
void launch_search(bool all, dim3 search_grid, dim3 finish_grid, const ExhParams &E, int64_t first, int64_t n,
                   const uint32_t *list_len, hipStream_t st) {
  if (all)
    hipLaunchKernelGGL((exhaustive_search_kernel<J, true>), search_grid, dim3(ENC_THREADS), 0, st, E, first, n, list_len);
  else
    hipLaunchKernelGGL((exhaustive_search_kernel<J, false>), search_grid, dim3(ENC_THREADS), 0, st, E, first, n, list_len);
  hipLaunchKernelGGL(exhaustive_finish_kernel<J>, finish_grid, dim3(ENC_THREADS), 0, st, E, first, n);
}

template <bool SEARCH>
void launch_slices_q(int q, const EncParams &P, int64_t first, int64_t n, uint32_t *list_len, SyndromeCare care, hipStream_t st) {
  switch (q) {
    case 1: launch_slices<1, SEARCH>(P, first, n, list_len, care, st); break;
    case 2: launch_slices<2, SEARCH>(P, first, n, list_len, care, st); break;
    case 3: launch_slices<3, SEARCH>(P, first, n, list_len, care, st); break;
    default: launch_slices<4, SEARCH>(P, first, n, list_len, care, st); break;
  }
}

}  // namespace

namespace {

Counts counts_in(const EncodePlan &plan, const xorenc_sizes &sz, int32_t q, uint64_t *pbits) {
  unsigned char *const area = reinterpret_cast<unsigned char *>(pbits + (int64_t)q * sz.n_slots);
  Counts C;
  C.n_units = (int32_t)sz.n_units;
  C.n_blocks = plan.n_blocks;
  C.unit = plan.unit_at >= 0 ? reinterpret_cast<uint16_t *>(area + plan.unit_at) : nullptr;
  C.block = reinterpret_cast<uint32_t *>(area + plan.block_at);
  C.scanned = plan.scanned_at >= 0 ? reinterpret_cast<uint32_t *>(area + plan.scanned_at) : nullptr;
  return C;
}

void launch_emit(const EncodePlan &plan, const uint64_t *pbits, const Counts &C, int32_t q, const xorenc_sizes &sz,
                 uint32_t *patch_off_out, uint16_t *patch_out, int64_t patch_capacity, uint32_t *total_out, hipStream_t st) {
  const dim3 grid(plan.emit_groups), block(ENC_THREADS);
  if (C.scanned)
    hipLaunchKernelGGL(emit_patches_kernel<true>, grid, block, 0, st, pbits, C, q, sz.n_slots, plan.units_per_block,
                       plan.per, patch_off_out, patch_out, patch_capacity, total_out);
  else
    hipLaunchKernelGGL(emit_patches_kernel<false>, grid, block, 0, st, pbits, C, q, sz.n_slots, plan.units_per_block,
                       plan.per, patch_off_out, patch_out, patch_capacity, total_out);
}

int32_t encode_common(bool exhaustive, int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out,
                      const uint32_t *M_rows, const uint64_t *mask, const uint64_t *planes, uint8_t *enc_out,
                      uint32_t *patch_off_out, uint16_t *patch_out, int64_t patch_capacity, void *workspace,
                      int64_t workspace_bytes, uint32_t *total_out, void *hip_stream) {
  xorenc_sizes sz;
  const int32_t rc = xorenc_get_sizes(m, n, n_in, q, n_out, &sz);
  if (rc != XORENC_OK) return rc;
  if (!M_rows || !mask || !planes || !enc_out || !patch_off_out || !workspace || patch_capacity < 0)
    return XORENC_EINVAL;
  xorenc_internal_begin_call();
  if (patch_capacity > 0 && !patch_out) return XORENC_EINVAL;
  if (exhaustive && n_in > XORENC_EXH_MAX_N_IN) return XORENC_EUNSUPPORTED;
  const int64_t total = (int64_t)q * sz.n_slots;
  const int64_t n_counts = (int64_t)q * sz.n_units;
  if (workspace_bytes < total * 8 + n_counts * 4) return XORENC_EINVAL;
  if (n_counts > (int64_t)1 << 30) return XORENC_EUNSUPPORTED;
  if (((uintptr_t)mask & 7) || ((uintptr_t)planes & 7) || ((uintptr_t)workspace & 7) ||
      ((uintptr_t)patch_off_out & 3) || ((uintptr_t)patch_out & 1) || ((uintptr_t)enc_out & 3))
    return XORENC_EALIGN;
  for (int i = 0; i < n_out; ++i)
    if (n_in < 32 && (M_rows[i] >> n_in)) return XORENC_EINVAL;
  uint64_t *pbits = static_cast<uint64_t *>(workspace);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int J = n_out / 64;
  const EncodePlan plan = encode_plan(sz, q, n_out);
  const int n_blocks = q * plan.n_blocks;
  const Counts C = counts_in(plan, sz, q, pbits);
  EncParams P;
  P.mask = mask;
  P.planes = planes;
  P.enc = enc_out;
  P.pbits = pbits;
  P.counts = C;
  P.n_slots = sz.n_slots;
  P.n_eslots = sz.n_eslots;
  P.n_in = n_in;
  P.J = J;
  for (int i = 0; i < XORENC_MAX_N_OUT; ++i) P.M_rows[i] = i < n_out ? M_rows[i] : 0u;
  if (!exhaustive) {
    launch_slices_q<false>(q, P, 0, sz.n_eslots, nullptr, SyndromeCare{}, st);
  } else {
    ExhParams E;
    E.mask = mask;
    E.planes = planes;
    E.enc = enc_out;
    E.pbits = pbits;
    E.counts = C;
    E.n_slots = sz.n_slots;
    E.n_eslots = sz.n_eslots;
    E.n_in = n_in;
    E.q = q;
    for (int w = 0; w < XORENC_MAX_J; ++w) {
      E.used[w] = 0;
      for (int i = 0; i < 64; ++i) E.used[w] |= (uint64_t)(P.M_rows[64 * w + i] != 0) << i;
      for (int j = 0; j < XORENC_EXH_MAX_N_IN; ++j) {
        uint64_t col = 0;
        for (int i = 0; i < 64; ++i) col |= (uint64_t)((P.M_rows[64 * w + i] >> j) & 1u) << i;
        E.Mcol[w][j] = col;
      }
    }
    // free until the last kernel overwrites every entry
    uint32_t *const list_len = patch_off_out + q * sz.n_units;
    const int64_t range = (int64_t)1 << 29;  // slices of a pass: list entries are 32-bit numbers
    for (int64_t first = 0; first < sz.n_eslots; first += range) {
      const int64_t n_pass = sz.n_eslots - first < range ? sz.n_eslots - first : range;
      const dim3 fg((unsigned)((n_pass + ENC_THREADS - 1) / ENC_THREADS), (unsigned)q);
      const dim3 sg(J == 1 ? 1024 : J == 2 ? 768 : 512);  // search: the workgroups that are resident walk over the items
      const bool all = n_in <= kAllMaxNIn;
      if (!all) {
        hipLaunchKernelGGL(exhaustive_reset_kernel, dim3(1), dim3(1), 0, st, list_len);
        launch_slices_q<true>(q, P, first, n_pass, list_len, syndrome_care(n_in, J, (n_pass + ENC_THREADS - 1) / ENC_THREADS), st);
      }
      switch (J) {
        case 1: launch_search<1>(all, sg, fg, E, first, n_pass, list_len, st); break;
        case 2: launch_search<2>(all, sg, fg, E, first, n_pass, list_len, st); break;
        case 3: launch_search<3>(all, sg, fg, E, first, n_pass, list_len, st); break;
        default: launch_search<4>(all, sg, fg, E, first, n_pass, list_len, st); break;
      }
    }
  }
  if (C.scanned) {
    const int nscan = (n_blocks + SCAN_BLOCK - 1) / SCAN_BLOCK;
    hipLaunchKernelGGL(scan_local_kernel, dim3(nscan), dim3(SCAN_THREADS), 0, st, C.block, C.scanned, n_blocks);
    hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(1024), 0, st, C.scanned, n_blocks, nscan);
    hipLaunchKernelGGL(scan_add_kernel, dim3(nscan), dim3(SCAN_THREADS), 0, st, C.scanned, n_blocks);
  }
  launch_emit(plan, pbits, C, q, sz, patch_off_out, patch_out, patch_capacity, total_out, st);
  return xorenc_internal_check_launch();
}

}  // namespace

extern "C" int32_t xorenc_encode(int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out, const uint32_t *M_rows,
                                 const uint64_t *mask, const uint64_t *planes, uint8_t *enc_out,
                                 uint32_t *patch_off_out, uint16_t *patch_out, int64_t patch_capacity,
                                 void *workspace, int64_t workspace_bytes, void *hip_stream) {
  return encode_common(false, m, n, n_in, q, n_out, M_rows, mask, planes, enc_out, patch_off_out, patch_out,
                       patch_capacity, workspace, workspace_bytes, nullptr, hip_stream);
}

extern "C" int32_t xorenc_encode_static(int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out,
                                        const uint32_t *M_rows, const uint64_t *mask, const uint64_t *planes,
                                        uint8_t *enc_out, uint32_t *patch_off_out, uint16_t *patch_out,
                                        int64_t patch_capacity, void *hip_stream) {
  xorenc_sizes sz;
  const int32_t rc = xorenc_get_sizes(m, n, n_in, q, n_out, &sz);
  if (rc != XORENC_OK) return rc;
  const int64_t need = (int64_t)q * sz.n_slots * 8 + (int64_t)q * sz.n_units * 4;
  if (need > (int64_t)XORENC_STATIC_SCRATCH_BYTES) return XORENC_ELIMIT;
  void *area = nullptr;
  const int32_t rs = static_scratch_address(&area);
  if (rs != XORENC_OK) return rs;
  return encode_common(false, m, n, n_in, q, n_out, M_rows, mask, planes, enc_out, patch_off_out, patch_out,
                       patch_capacity, area, XORENC_STATIC_SCRATCH_BYTES, nullptr, hip_stream);
}

extern "C" int32_t xorenc_encode_exhaustive(int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out,
                                            const uint32_t *M_rows, const uint64_t *mask, const uint64_t *planes,
                                            uint8_t *enc_out, uint32_t *patch_off_out, uint16_t *patch_out,
                                            int64_t patch_capacity, void *workspace, int64_t workspace_bytes,
                                            void *hip_stream) {
  return encode_common(true, m, n, n_in, q, n_out, M_rows, mask, planes, enc_out, patch_off_out, patch_out,
                       patch_capacity, workspace, workspace_bytes, nullptr, hip_stream);
}

extern "C" int32_t xorenc_encode_total(int32_t fewest_patches, int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out,
                                       const uint32_t *M_rows, const uint64_t *mask, const uint64_t *planes,
                                       uint8_t *enc_out, uint32_t *patch_off_out, uint16_t *patch_out,
                                       int64_t patch_capacity, void *workspace, int64_t workspace_bytes,
                                       uint32_t *total_out, void *hip_stream) {
  if (!total_out) return XORENC_EINVAL;
  if ((uintptr_t)total_out & 3) return XORENC_EALIGN;
  const int32_t rc = encode_common(fewest_patches != 0, m, n, n_in, q, n_out, M_rows, mask, planes, enc_out, patch_off_out,
                                   patch_out, patch_capacity, workspace, workspace_bytes, total_out, hip_stream);
  if (rc != XORENC_OK) return rc;
  return xorenc_internal_hip_status((int32_t)hipStreamSynchronize(static_cast<hipStream_t>(hip_stream)));
}

extern "C" int32_t xorenc_encode_patches(int32_t m, int32_t n, int32_t n_in, int32_t q, int32_t n_out,
                                         uint32_t *patch_off_out, uint16_t *patch_out, int64_t patch_capacity,
                                         void *workspace, int64_t workspace_bytes, uint32_t *total_out, void *hip_stream) {
  xorenc_sizes sz;
  const int32_t rc = xorenc_get_sizes(m, n, n_in, q, n_out, &sz);
  if (rc != XORENC_OK) return rc;
  if (!patch_off_out || !workspace || !total_out || patch_capacity < 0 || (patch_capacity > 0 && !patch_out))
    return XORENC_EINVAL;
  const int64_t n_counts = (int64_t)q * sz.n_units;
  if (workspace_bytes < (int64_t)q * sz.n_slots * 8 + n_counts * 4) return XORENC_EINVAL;
  if (n_counts > (int64_t)1 << 30) return XORENC_EUNSUPPORTED;
  if (((uintptr_t)workspace & 7) || ((uintptr_t)patch_off_out & 3) || ((uintptr_t)patch_out & 1) || ((uintptr_t)total_out & 3))
    return XORENC_EALIGN;
  xorenc_internal_begin_call();
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  uint64_t *const pbits = static_cast<uint64_t *>(workspace);
  const EncodePlan plan = encode_plan(sz, q, n_out);
  launch_emit(plan, pbits, counts_in(plan, sz, q, pbits), q, sz, patch_off_out, patch_out, patch_capacity, total_out, st);
  const int32_t rl = xorenc_internal_check_launch();
  if (rl != XORENC_OK) return rl;
  return xorenc_internal_hip_status((int32_t)hipStreamSynchronize(st));
}

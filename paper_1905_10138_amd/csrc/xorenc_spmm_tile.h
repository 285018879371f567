// Fused decrypt + patch + mask + dequantise + W X for many columns of bf16 X (arXiv 1905.10138, Sections 3.1-3.2 for the
// decode, Fig. 1 for the product).  Included by the per-Q instantiation units next to xorenc_spmm_kernel.h, whose operand
// synthesis (weights as FP4 codes converted to bf16 +-2/0), operand order and LDS layout of X it shares.
//
// What differs is who shares what.  There every wave streams its own slices of X and all waves of a workgroup split
// the reduction.  Here WR waves stand on top of each other: they multiply different rows by the same slice of X, which
// they fetch together, each a part, into one of two slice buffers.  A slice of X is then fetched once for
// 32 RB WR rows and one barrier per slice keeps the waves together.  A wave's tile is 32 RB rows x 32 NCB columns
// with NCB up to 4, so that a converted weight operand feeds four matrix instructions instead of two, and decoding a
// slice is spread over 4 Q RB NCB of them.  KG > 1: KG such groups split the reduction in halves and add up at the end.
//
// Bound: the matrix instructions as long as about four other instructions or fewer go with each (a 32-cycle
// instruction leaves the SIMD free to issue others for half of its time), which is what the wide tile is for; the
// LDS reads of the X operands (1 KB per RB Q matrix instructions) use half of the LDS bandwidth.
#ifndef XORENC_SPMM_TILE_H
#define XORENC_SPMM_TILE_H

#include "xorenc_spmm_kernel.h"

namespace xorenc_spmm_detail {

constexpr int kTileGroup = 4;   // slices whose compressed words are staged, and whose patches are scattered, together
constexpr int kTileChunk = 16;  // slices whose patch offsets and entries are staged together

// Bytes of LDS of a workgroup, in this order: two slices of X per reduction group; then per wave two groups of
// compressed words (mask halves of four slices, encrypted dwords), the patch lists of a chunk (offsets of two chunks,
// entries of one), flip words of a group; XOR tables; scales.
template <int Q, int RB, int NCB, int WR, int KG>
struct TileLds {
  static constexpr int X = KG * 2 * (NCB * 4096);
  static constexpr int COMP = RB * 1024 + RB * Q * 512;   // one group
  static constexpr int PATCH = 3 * RB * Q * 256;
  static constexpr int FLIPS = kTileGroup * RB * Q * 256;
  static constexpr int WAVE = 2 * COMP + PATCH + FLIPS;
  static constexpr int LUT = X + WR * KG * WAVE;
  static constexpr int ALPHA = Q * WR * RB * 128;
  static int total(int J, int nib) { return LUT + J * nib * 2048 + ALPHA; }
};

// Results go past the L2: the lines that a launch leaves dirty there are written back after its last store, when nothing else
// runs (16384 x 4096, one plane, B = 1024 100.7 -> 99.2 us; two planes, n_out = 192, n_in = 20, B = 250 with the copy of X 61.7 ->
// 61.1; in the kernels with smaller tiles it makes no difference).
__device__ inline void store_past_l2(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int Q, int RB, int NCB, int WR, int KG, int NIBT>
__global__ __launch_bounds__(WR *KG * 64, 2) void spmm_tile_kernel(DevLayer L, const uint16_t *__restrict__ X, int64_t ldx,
                                                                   int B, float *__restrict__ Y, int64_t ldy,
                                                                   int row_tiles, int tiles) {
  constexpr int NW = WR * KG, ROWS = 32 * RB * WR;
  constexpr int PANELS = NCB / 2;         // panels of 64 columns (128-byte rows)
  constexpr int XSL = PANELS * 8192;      // one slice buffer
  constexpr int PERX = PANELS * 8 / WR;   // direct loads of X per wave and slice
  static_assert(NCB % 2 == 0 && PERX >= 1 && PERX <= 8 && 8 % PERX == 0, "a wave's loads stay inside one panel");
  static_assert(KG == 1 || (KG == 2 && NCB % 2 == 0), "the groups exchange halves of their columns");
  extern __shared__ __attribute__((aligned(16))) uint8_t tile_lds_area[];

  // tiles go to the XCDs in runs (workgroup i runs on XCD i % 8), rows first: the workgroups of an XCD share X in its L2
  const int per_xcd = gridDim.x >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= tiles) return;
  const int tile_c = tile / row_tiles, tile_r = tile - tile_c * row_tiles;

  const int l_n = L.n, l_m = L.m, l_spr = L.spr, l_n_units = L.n_units, n_in = L.n_in, l_J = L.J;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, rl = lane & 31;
  const int wr = wave % WR, kg = wave / WR;
  const int row0 = tile_r * ROWS, col0 = tile_c * (32 * NCB);
  const int rb0 = tile_r * (RB * WR) + wr * RB;  // first row block of the wave
  typedef TileLds<Q, RB, NCB, WR, KG> Lds;
  uint8_t *const xbufs = tile_lds_area + kg * (2 * XSL);
  uint8_t *const wave_lds = tile_lds_area + Lds::X + wave * Lds::WAVE;
  uint32_t *const comp = reinterpret_cast<uint32_t *>(wave_lds);
  uint32_t *const pstage = reinterpret_cast<uint32_t *>(wave_lds + 2 * Lds::COMP);
  uint32_t *const flip_area = reinterpret_cast<uint32_t *>(wave_lds + 2 * Lds::COMP + Lds::PATCH);
  uint32_t *const lut = reinterpret_cast<uint32_t *>(tile_lds_area + Lds::LUT);
  float *const alpha_s = reinterpret_cast<float *>(tile_lds_area + Lds::LUT + l_J * NIBT * 2048);

  // ---- slices [k0, k0 + cnt) of this group; every group goes through the same number of barriers
  const int base_cnt = l_spr / KG, extra = l_spr % KG;
  const int k0 = kg * base_cnt + min(kg, extra), cnt = base_cnt + (kg < extra ? 1 : 0);
  const int iters = base_cnt + (extra ? 1 : 0);

  // ---- descriptors and per-lane offsets (see spmm_kernel)
  const int64_t row_bytes = ldx * 2;
  const uint32_t x_extent = ((uint32_t)((int64_t)(l_n - 1) * row_bytes + (int64_t)(B - col0) * 2) + 3u) & ~3u;
  const uint64_t x_base = reinterpret_cast<uint64_t>(X + col0);
  const u32x4 xdesc = {(uint32_t)x_base, (uint32_t)(x_base >> 32) & 0xffffu, x_extent, kRsrcFlags};
  const u32x4 mdesc = {(uint32_t)reinterpret_cast<uint64_t>(L.mask32),
                       (uint32_t)(reinterpret_cast<uint64_t>(L.mask32) >> 32) & 0xffffu, (uint32_t)(L.n_slots * 8),
                       kRsrcFlags};
  const u32x4 edesc = {(uint32_t)reinterpret_cast<uint64_t>(L.enc),
                       (uint32_t)(reinterpret_cast<uint64_t>(L.enc) >> 32) & 0xffffu,
                       (uint32_t)((L.n_eslots >> 3) * L.q * n_in), kRsrcFlags};
  auto row_of_pos = [](int pos) {
    return ((pos & 1) << 2) | (((pos >> 1) & 1) << 3) | ((pos >> 2) & 1) | (((pos >> 3) & 1) << 1) |
           (((pos >> 4) & 1) << 4) | (((pos >> 5) & 1) << 5);
  };
  const int first_load = wr * PERX, panel = first_load / 8;  // this wave's part of a slice
  const int xch = (lane & 7) ^ (((lane >> 3) & 3) << 1);
  const uint32_t x_lane_off = (uint32_t)(row_of_pos(lane >> 3) * row_bytes) +
                              ((col0 + panel * 64 + xch * 8 < B) ? (uint32_t)(panel * 128 + xch * 16) : 0u);
  const uint32_t xbufs_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)(xbufs));
  uint32_t x_row[PERX];  // byte offset of each load's first row inside a slice (uniform)
#pragma unroll
  for (int i = 0; i < PERX; ++i)
    x_row[i] = __builtin_amdgcn_readfirstlane((uint32_t)(row_of_pos(((first_load + i) & 7) << 3) * row_bytes));
  const uint32_t x_dst = __builtin_amdgcn_readfirstlane(xbufs_lds + (uint32_t)(first_load * 1024));
  uint32_t x_next = __builtin_amdgcn_readfirstlane((uint32_t)(k0 * 64 * row_bytes));  // the slice to be fetched next
  const uint32_t x_step = __builtin_amdgcn_readfirstlane((uint32_t)(64 * row_bytes));
  auto dma_x = [&](uint32_t buf_off) {  // the next slice of X, this wave's part
#pragma unroll
    for (int i = 0; i < PERX; ++i)
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(x_dst + buf_off + i * 1024),
                   "v"(x_lane_off), "s"(xdesc), "s"(x_next + x_row[i])
                   : "memory");
    x_next += x_step;
  };
  const uint32_t e_bit = (uint32_t)(rl * n_in);
  const uint32_t e_lane_dw = e_bit >> 5, e_shift = e_bit & 31u;  // the field's first dword in its unit, and bit in that
  const uint32_t e_plane_units = (uint32_t)(L.n_eslots >> 5), e_unit_bytes = (uint32_t)(n_in * 4);
  const uint32_t j_magic = l_J == 4 ? 0x40000000u : l_J == 3 ? 0x55555556u : 0x80000000u;
  const int j_shift = l_J == 1 ? 1 : 0;
  auto slice_of_word = [&](int s) { return (int)__umulhi((uint32_t)s << j_shift, j_magic); };  // s / J (s < 2^26)
  const uint32_t comp_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(__attribute__((address_space(3))) uint32_t *)(comp));
  auto dma_dword = [&](uint32_t lds_addr, const u32x4 &desc, uint32_t so) {  // 64 consecutive dwords
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(
                     __builtin_amdgcn_readfirstlane(lds_addr)),
                 "v"(lane * 4), "s"(desc), "s"(__builtin_amdgcn_readfirstlane(so))
                 : "memory");
  };
  // The compressed words of the group's four slices lie one after the other: 1 KB of masks per row block, fetched with
  // one load, and 4 n_in dwords of encrypted bits (fewer with wide slices) per row block and plane, one load per 64.
  // What is fetched beyond the range belongs to other units; a row block beyond the matrix reads zero masks (range check).
  const bool enc2 = n_in * (l_J == 1 ? 4 : l_J == 2 ? 3 : 2) > 64;  // (four words touch that many slices)
  auto load_comp = [&](int gi) {
    const int s = k0 + gi * kTileGroup, es = slice_of_word(s);
    const uint32_t dst = comp_lds + (gi & 1) * Lds::COMP;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(
                       __builtin_amdgcn_readfirstlane(dst + rb * 1024)),
                   "v"(lane * 16), "s"(mdesc),
                   "s"(__builtin_amdgcn_readfirstlane((uint32_t)((rb0 + rb) * l_spr + s) * 256u))
                   : "memory");
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t so = ((uint32_t)p * e_plane_units + (uint32_t)((rb0 + rb) * L.espr + es)) * e_unit_bytes;
        dma_dword(dst + RB * 1024 + (rb * Q + p) * 512, edesc, so);
        if (enc2) dma_dword(dst + RB * 1024 + (rb * Q + p) * 512 + 256, edesc, so + 256u);
      }
    }
  };
  struct Words {
    uint32_t mw[RB], e0[RB][Q], e1[RB][Q], flips[RB][Q];
  };
  auto read_comp = [&](int i, Words &c) {  // words and flips of slice k0 + i; the flip words are zero again afterwards
    const int gi = i / kTileGroup, t = i % kTileGroup;
    const uint32_t *const src = comp + (gi & 1) * (Lds::COMP / 4);
    const uint32_t eo = (uint32_t)(slice_of_word(k0 + i) - slice_of_word(k0 + gi * kTileGroup)) * (uint32_t)n_in + e_lane_dw;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      c.mw[rb] = src[rb * 256 + t * 64 + 2 * rl + g];
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t *const e = src + RB * 256 + (rb * Q + p) * 128 + eo;
        c.e0[rb][p] = e[0];
        c.e1[rb][p] = e[1];  // (in the LDS of the workgroup; used only where the field straddles)
        uint32_t *const f = flip_area + (t * RB * Q + rb * Q + p) * 64 + lane;
        c.flips[rb][p] = *f;
        *f = 0u;
      }
    }
  };

  // ---- first loads
  if (cnt > 0) {
    load_comp(0);
    dma_x(0);
  }

  // ---- patch lists, kTileChunk slices at a time: lane i holds the offset of unit i of the chunk, lane j its entries 2j
  // and 2j + 1.  They take the road of the compressed words (no load of the loop returns into a register, so the
  // compiler places no wait of its own): chunk c + 1's entries and chunk c + 2's offsets are requested when chunk c begins.
  // Past the range the staged values are those of other units, which nothing uses; past the arrays they are zero.
  const uint16_t *const l_patch = L.patch;
  const uint32_t pstage_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(__attribute__((address_space(3))) uint32_t *)(pstage));
  const u32x4 odesc = {(uint32_t)reinterpret_cast<uint64_t>(L.patch_off),
                       (uint32_t)(reinterpret_cast<uint64_t>(L.patch_off) >> 32) & 0xffffu,
                       (uint32_t)(((int64_t)L.q * l_n_units + 1) * 4), kRsrcFlags};
  const uint32_t p_skew = (uint32_t)(reinterpret_cast<uint64_t>(l_patch) >> 1) & 1u;  // entries are 2-byte aligned
  const uint64_t p_base = reinterpret_cast<uint64_t>(l_patch) & ~3ull;
  const uint32_t p_total = __builtin_amdgcn_readfirstlane(L.patch_off[(int64_t)L.q * l_n_units]);
  const u32x4 pdesc = {(uint32_t)p_base, (uint32_t)(p_base >> 32) & 0xffffu, (2u * (p_skew + p_total) + 3u) & ~3u,
                       kRsrcFlags};
  auto load_off = [&](int c) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p)
        dma_dword(pstage_lds + ((c & 1) * RB * Q + rb * Q + p) * 256, odesc, (uint32_t)(p * l_n_units + (rb0 + rb) * l_spr + k0 + c * kTileChunk) * 4u);
  };
  auto load_ent = [&](int c) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t base = __builtin_amdgcn_readfirstlane(pstage[((c & 1) * RB * Q + rb * Q + p) * 64]);
        dma_dword(pstage_lds + (2 * RB * Q + rb * Q + p) * 256, pdesc, (2u * (base + p_skew)) & ~3u);
      }
  };
  // group gi is the next to be decoded; what was requested for it has landed.  Its patches are scattered into the flip
  // words of its four slices, all lists of the wave at once: each has LPL lanes, lane j of them takes entry j of the
  // group's list, whose unit it finds by counting list ends.
  constexpr int NL = RB * Q, LPL = NL <= 2 ? 32 : 16;  // lists (a row block and plane each), lanes per list
  const int ln = min(lane / LPL, NL - 1), jl = lane % LPL;
  const uint16_t *const ent_half = reinterpret_cast<const uint16_t *>(pstage + 2 * NL * 64) + ln * 128;
  auto group_begin = [&](int gi) {
    constexpr int PER_CHUNK = kTileChunk / kTileGroup;
    const int gc = gi % PER_CHUNK, c = gi / PER_CHUNK;
    const uint32_t *const offs = pstage + ((c & 1) * NL + ln) * 64;
    const uint32_t base = offs[0];
    const uint4 o4 = *reinterpret_cast<const uint4 *>(offs + kTileGroup * gc);
    // (offsets past the end of the array arrive as zero)
    const uint32_t e1 = max(o4.x, o4.y), e2 = max(e1, o4.z), e3 = max(e2, o4.w);
    const uint32_t e4 = NL * LPL == 64 || lane < NL * LPL ? max(e3, offs[kTileGroup * gc + 4]) : 0u;
    uint32_t j = o4.x + (uint32_t)jl;
    while (__ballot(j < e4)) {  // uniform; one trip unless the lists are long
      if (j < e4) {
        const uint32_t h = j - base + ((base + p_skew) & 1u);  // halfword of the staged ones
        uint32_t v = ent_half[min(h, 127u)];
        asm volatile("" : "+v"(v));  // (keeps the two loads apart: one through a selected pointer would be a flat load)
        if (h >= 128u) v = l_patch[j];
        const uint32_t t = (j >= e1 ? 1u : 0u) + (j >= e2 ? 1u : 0u) + (j >= e3 ? 1u : 0u);
        // entry = (row%32) << 6 | bit: the word half is bit 5
        atomicXor(flip_area + (t * NL + ln) * 64 + ((v >> 6) | (v & 32u)), 1u << (v & 31u));
      }
      j += LPL;
    }
    if (gc == PER_CHUNK - 1) {  // the chunk's entries have all been read
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      load_ent(c + 1);
      load_off(c + 2);
    }
    load_comp(gi + 1);
  };
  load_off(0);
  load_off(1);

  // ---- XOR tables and scales, shared by the workgroup
  build_shared_tables(L, wave, NW, lane, l_J, NIBT, lut, NIBT * 512);
  for (int i = tid; i < Q * ROWS; i += NW * 64) {
    const int p = i / ROWS, r = row0 + i % ROWS;
    alpha_s[i] = (r < l_m) ? -0.5f * L.alpha[(int64_t)p * l_m + r] : 0.f;
  }
  for (int i = lane; i < kTileGroup * RB * Q * 64; i += 64) flip_area[i] = 0u;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  load_ent(0);

  f32x16 acc[Q][RB][NCB];
#pragma unroll
  for (int p = 0; p < Q; ++p)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[p][rb][cb][i] = 0.f;

  // per-lane offset of the transposing reads inside a slice buffer, for the two column blocks of a panel
  const int jj = (lane >> 2) & 3, c4 = lane & 3;
  const int pos_lane = jj | (g << 5);
  uint32_t tr_off[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const int c = 4 * cb + 2 * ((lane >> 4) & 1) + (c4 >> 1);
    tr_off[cb] = (uint32_t)(pos_lane * 128 + ((c ^ ((pos_lane & 3) << 1)) * 16) + 8 * (c4 & 1));
  }
  auto lookup = [&](const Words &c, uint32_t(&S)[RB][Q], int s) {
    const uint32_t *const lut_g = lut + g + (s - slice_of_word(s) * l_J) * (NIBT * 512);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t x = __builtin_amdgcn_alignbit(c.e1[rb][p], c.e0[rb][p], e_shift);
        // (columns of M beyond n_in are zero: index bits beyond n_in choose among equal entries)
        uint32_t v = lut_g[2 * (x & 255u)];
        if constexpr (NIBT >= 2) v ^= lut_g[2 * (256 + ((x >> 8) & 255u))];
        if constexpr (NIBT >= 3) v ^= lut_g[2 * (512 + ((x >> 16) & 255u))];
        if constexpr (NIBT >= 4) v ^= lut_g[2 * (768 + (x >> 24))];
        S[rb][p] = v;
      }
  };
  // code pairs of a half-word: I_par holds (mask, sign) of its bits 2k + par
  uint32_t I0[RB][Q], I1[RB][Q];
  auto interleave = [&](const Words &c, const uint32_t(&S)[RB][Q]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t v = S[rb][p] ^ c.flips[rb][p];
        I0[rb][p] = (c.mw[rb] & 0x55555555u) | ((v << 1) & 0xAAAAAAAAu);
        I1[rb][p] = ((c.mw[rb] >> 1) & 0x55555555u) | (v & 0xAAAAAAAAu);
      }
  };
  bf16x8 bfrag[2][NCB];
  auto read_bfrag = [&](const uint8_t *buf, int t, bf16x8(&bf)[NCB]) {
    const int par = t >> 1, e = t & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const uint8_t *src = buf + tr_off[cb & 1] + (cb >> 1) * 8192 + (4 * par + 8 * e) * 128;
      const s16x4 lo = lds_read_tr16(src), hi = lds_read_tr16(src + 16 * 128);
      bf[cb] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  auto mfma_step = [&](int t, const bf16x8(&bf)[NCB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t I = t < 2 ? I0[rb][p] : I1[rb][p];
        const bf16x8 a = __builtin_bit_cast(bf16x8, expand_fp4_codes(((t & 1) ? I : I << 2) & 0xCCCCCCCCu));
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[p][rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bf[cb], acc[p][rb][cb], 0, 0, 0);
      }
  };

  // ---- slice 0's operands
  Words cw;
  uint32_t S[RB][Q];
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (cnt > 0) {
    group_begin(0);
    read_comp(0, cw);
    lookup(cw, S, k0);
    interleave(cw, S);
  }
  for (int i = 0; i < iters; ++i) {
    // X of slice i and the words of slice i + 1 have landed, and every wave is done with the buffer of slice i - 1
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (i >= cnt) continue;  // uniform
    // (first: the read of a long list from memory brings a wait of the compiler's for everything in flight)
    if ((i + 1) % kTileGroup == 0) group_begin((i + 1) / kTileGroup);
    if (i + 1 < cnt) dma_x((i + 1) & 1 ? (uint32_t)XSL : 0u);
    // one straight run of instructions: multiply slice i, decode slice i + 1 (behind the last slice: whatever the
    // staging area holds, for nobody)
    const uint8_t *const buf = xbufs + (i & 1 ? XSL : 0);
    read_bfrag(buf, 0, bfrag[0]);
    read_comp(i + 1, cw);
    read_bfrag(buf, 1, bfrag[1]);
    mfma_step(0, bfrag[0]);
    // (left alone, the compiler moves all operand reads of the slice in front of the first product)
    __builtin_amdgcn_sched_barrier(0);
    lookup(cw, S, k0 + i + 1);
    read_bfrag(buf, 2, bfrag[0]);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(1, bfrag[1]);
    __builtin_amdgcn_sched_barrier(0);
    read_bfrag(buf, 3, bfrag[1]);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(2, bfrag[0]);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(3, bfrag[1]);
    interleave(cw, S);
  }

  // ---- epilogue.  acc element i of a lane is row 8*(i/4) + 4*g + i%4, column rl of its 32x32 block.
  const float *const al = alpha_s + wr * RB * 32;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
      f32x4 a4[Q];
#pragma unroll
      for (int p = 0; p < Q; ++p) a4[p] = *reinterpret_cast<const f32x4 *>(al + p * ROWS + rb * 32 + 8 * j4 + 4 * g);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float v = a4[0][k] * acc[0][rb][cb][4 * j4 + k];
#pragma unroll
          for (int p = 1; p < Q; ++p) v += a4[p][k] * acc[p][rb][cb][4 * j4 + k];
          acc[0][rb][cb][4 * j4 + k] = v;
        }
    }
  auto store = [&](int cb) {
    const int gc = col0 + cb * 32 + rl;
    if (gc >= B) return;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int gr = (rb0 + rb) * 32 + 8 * (j >> 2) + 4 * g + (j & 3);
        if (gr < l_m) store_past_l2(Y + (int64_t)gr * ldy + gc, acc[0][rb][cb][j]);
      }
  };
  if constexpr (KG == 1) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) store(cb);
  } else {
    // group 0 stores the first half of the columns, group 1 the second; the other half of each goes through LDS (the
    // X ring is idle after the barrier): [wave][column block][element][lane]
    __syncthreads();
    float *const ex = reinterpret_cast<float *>(tile_lds_area);
    constexpr int HALF = NCB / 2;
#pragma unroll
    for (int h = 0; h < HALF; ++h)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          ex[(((wave * HALF + h) * RB + rb) * 16 + j) * 64 + lane] = kg == 0 ? acc[0][rb][HALF + h][j] : acc[0][rb][h][j];
    __syncthreads();
    const int other = wr + (1 - kg) * WR;
#pragma unroll
    for (int h = 0; h < HALF; ++h)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const float o = ex[(((other * HALF + h) * RB + rb) * 16 + j) * 64 + lane];
          if (kg == 0)
            acc[0][rb][h][j] += o;
          else
            acc[0][rb][HALF + h][j] += o;
        }
    if (kg == 0) {
#pragma unroll
      for (int h = 0; h < HALF; ++h) store(h);
    } else {
#pragma unroll
      for (int h = 0; h < HALF; ++h) store(HALF + h);
    }
  }
}

template <int Q, int RB, int NCB, int WR, int KG>
int32_t launch_tile(const DevLayer &D, const void *X, int64_t ldx, int B, float *Y, int64_t ldy, hipStream_t st) {
  const int row_tiles = (D.nrb + RB * WR - 1) / (RB * WR), col_tiles = (B + 32 * NCB - 1) / (32 * NCB);
  const int tiles = row_tiles * col_tiles;
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8)), block(WR * KG * 64);
  const int exchange = KG == 2 ? WR * KG * (NCB / 2) * RB * 4096 : 0;
  const int lds = max(TileLds<Q, RB, NCB, WR, KG>::total(D.J, D.nib), exchange);
  const uint16_t *Xh = static_cast<const uint16_t *>(X);
  switch (D.nib) {
    case 1: hipLaunchKernelGGL((spmm_tile_kernel<Q, RB, NCB, WR, KG, 1>), grid, block, lds, st, D, Xh, ldx, B, Y, ldy, row_tiles, tiles); break;
    case 2: hipLaunchKernelGGL((spmm_tile_kernel<Q, RB, NCB, WR, KG, 2>), grid, block, lds, st, D, Xh, ldx, B, Y, ldy, row_tiles, tiles); break;
    case 3: hipLaunchKernelGGL((spmm_tile_kernel<Q, RB, NCB, WR, KG, 3>), grid, block, lds, st, D, Xh, ldx, B, Y, ldy, row_tiles, tiles); break;
    default: hipLaunchKernelGGL((spmm_tile_kernel<Q, RB, NCB, WR, KG, 4>), grid, block, lds, st, D, Xh, ldx, B, Y, ldy, row_tiles, tiles); break;
  }
  return xorenc_internal_check_launch();
}

// Share of the chip's time that useful outputs fill with tiles of `area` outputs.  Workgroups of one reduction group run
// two per CU when `paired`; a round that gives every CU one of them takes 0.6 of the time of a round with two.
inline double tile_fill(int64_t outputs, int64_t tiles, int area, bool paired) {
  const int64_t pairs = paired ? tiles / 512 : 0, rest = tiles - 512 * pairs;
  const double rounds = (double)pairs + (paired && rest > 256 ? 1.0 : 0.6 * (double)((rest + 255) / 256));
  return (double)outputs / (rounds * 512.0 * area);
}

// Aligned bf16 X with enough columns and rows to keep the chip's matrix cores busy with whole tiles.  The tile is as
// wide as the accumulators of Q planes allow.  Measured against the kernels that serve the call otherwise (us, n = 4096
// unless stated): one plane, 16384 rows, B = 1024 124 -> 105, B = 512 68 against 68 (fill 0.83: stays there), 4096 rows,
// B = 1024 40 against 64 (0.42: stays); two planes, 16384 rows, B = 1024 219 -> 188, B = 256 62 -> 55, n_out = 192
// 105 -> 57, 4096 x 9216 at B = 1024 121 -> 112 and at B = 512 63 against 106 (0.5: stays); three planes, 6000 x 3000,
// B = 256 43 -> 35 (0.73), B = 1024 145 -> 98; four planes 56 -> 43 and 218 -> 120.  Slices of several words have no
// other kernel with tiles above 64 x 64.
template <int Q>
bool dispatch_tile_q(const DevLayer &D, const void *X, int32_t x_dtype, int64_t ldx, int B, float *Y, int64_t ldy,
                     int x_fast, hipStream_t st, int32_t *rc) {
  constexpr int RB = Q == 1 ? 2 : 1, NCB = Q <= 2 ? 4 : 2, WR = 4;
  constexpr int AREA = 32 * RB * WR * 32 * NCB;
  // (the masks of four slices are fetched 16 bytes at a time)
  if (x_dtype != XORENC_X_BF16 || !x_fast || ((uintptr_t)D.mask32 & 15)) return false;
  const int64_t tiles = (int64_t)((D.nrb + RB * WR - 1) / (RB * WR)) * ((B + 32 * NCB - 1) / (32 * NCB));
  const int64_t outputs = (int64_t)D.m * B;
  if (tiles > (1 << 30)) return false;
  const double least = D.J > 1 ? 0.55 : Q == 1 ? 0.9 : Q == 2 ? 0.85 : Q == 3 ? 0.65 : 0.55;
  const int lds1 = TileLds<Q, RB, NCB, WR, 1>::total(D.J, D.nib);
  const bool paired = lds1 <= 80 * 1024;
  const double fill1 = lds1 <= 160 * 1024 ? tile_fill(outputs, tiles, AREA, paired) : 0.0;
  double fill2 = 0.0;  // two reduction groups: a workgroup has the CU to itself
  if (Q >= 2 && TileLds<Q, RB, NCB, WR, 2>::total(D.J, D.nib) <= 160 * 1024)
    fill2 = 0.95 * (double)outputs / ((double)((tiles + 255) / 256) * 256.0 * AREA);
  if (fill1 < least && fill2 < least) return false;
  if constexpr (Q >= 2) {
    if (fill2 > fill1) {
      *rc = launch_tile<Q, RB, NCB, WR, 2>(D, X, ldx, B, Y, ldy, st);
      return true;
    }
  }
  *rc = launch_tile<Q, RB, NCB, WR, 1>(D, X, ldx, B, Y, ldy, st);
  return true;
}

}  // namespace xorenc_spmm_detail

#endif

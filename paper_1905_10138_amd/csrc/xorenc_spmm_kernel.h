// Fused decrypt + patch + mask + dequantise + W X kernel for the gfx950 matrix cores
// (arXiv 1905.10138: Sections 3.1-3.2 for the decode, Fig. 1 for the product it feeds).
// Included by the per-Q instantiation units xorenc_spmm_q*.hip.
//
// Operand synthesis.  The MFMA A operand is built in registers as bf16 values -2*t, t in
// {-1,0,+1} the ternary weight of one bit-plane: bit 15 = quantised bit, bit 14 = mask bit, all
// other bits 0 (0xC000 = -2, 0x4000 = +2, 0x0000 / 0x8000 = +-0).  The factor -1/2 is folded into
// alpha in the fp32 epilogue, so the scales are never rounded to bf16.  These patterns are what the
// FP4 (e2m1) codes 1100, 0100, 0000, 1000 convert to, and gfx950 converts two codes to two bf16
// values in one instruction: the (mask, sign) bit pairs are arranged as the top two bits of 4-bit
// codes (two instructions per eight weights) and each operand dword then costs one conversion.
//
// Work decomposition.  A workgroup of NW waves owns RB row blocks of 32 rows and CW = 32*NCB
// columns of X.  The waves split the reduction dimension into contiguous slice ranges and are
// fully independent until the final reduction: each wave streams the 64 rows of X that belong to
// its current slice through private LDS buffers and gathers its B operands from them with the
// transposing LDS read, so the main loop has no workgroup barrier.  Aligned bf16 X goes from global
// memory straight into LDS (one slice buffer per wave, requested a slice ahead); any
// other X passes through registers (one buffer).  Lane (rl = lane%32, g = lane/32) holds the
// 32-bit half g of the slice of row rl of each row block.
//
// One 32-bit half feeds 4 MFMA steps t = 2*par + e.  I_par is the word whose bit pairs
// (2k, 2k+1) hold (mask, sign) of half-word bit 2k+par; code word (par, e) keeps the pairs with
// k%2 = e, pair k in the top bits of code k/2.  Byte d of that word is operand dword d, so operand
// slot j = 2d + (high code) of step t of half g is the W column (X row)
//     64 s + 32 g + 8 (j>>1) + 4 (j&1) + 2 e + par
// and the B operand is gathered from exactly those X rows.
//
// Addressing.  Every global load in the loop is a buffer load: (descriptor) + (per-lane 32-bit
// offset fixed for the whole kernel) + (uniform scalar offset), so the loop spends no vector
// instructions on addresses, and loads beyond the end of X return zero (rows of the padded last
// slice) instead of needing a branch.
#ifndef XORENC_SPMM_KERNEL_H
#define XORENC_SPMM_KERNEL_H

#include "xorenc_device.h"

namespace xorenc_spmm_detail {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr uint32_t kRsrcFlags = 0x00020000u;  // raw buffer, 32-bit data format

// Transposing LDS read: within each group of 16 lanes, lane i receives element i%4 of the 8 bytes
// addressed by lanes 4j + i/4, j = 0..3.
__device__ inline s16x4 lds_read_tr16(const uint8_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p));
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// Eight FP4 (e2m1) codes -> eight bf16 values, one conversion per pair: code 0100 is +2, 1100 is -2,
// 0000 / 1000 are +-0; byte d of w becomes operand dword d (low code in the low half).
__device__ inline u32x4 expand_fp4_codes(uint32_t w) {
  u32x4 a;
  a[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 0));
  a[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 1));
  a[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 2));
  a[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, 1.0f, 3));
  return a;
}

// Partial sums of a split launch travel between workgroups that may sit on different XCDs, whose L2 caches are
// not coherent with each other for ordinary accesses: relaxed device-scope atomic accesses go to the coherent
// level directly, without the cache write-back and invalidation a fence would bring.
__device__ inline void split_store(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float split_load(const float *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the same for 16 bytes at a time: buffer accesses with the sc0 and sc1 bits set (coherent at device scope)
constexpr int kCoherentAux = 0x11;
__device__ inline __amdgpu_buffer_rsrc_t split_rsrc(float *base) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000u);
}
__device__ inline void split_store4(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, byte_off, 0, kCoherentAux);
}
__device__ inline u32x4 split_load4(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, kCoherentAux);
}

// One XOR table by one wave: entry v = XOR of the eight columns selected by the bits of v, lower and upper 32 rows next to
// each other.  A lane builds the entries lane, lane + 64, lane + 128 and lane + 192.
__device__ inline void build_xor_table(int lane, const uint32_t *col_lo, const uint32_t *col_hi, uint32_t *table) {
  uint32_t lo = 0, hi = 0;
#pragma unroll
  for (int t = 0; t < 6; ++t)
    if ((lane >> t) & 1) {
      lo ^= col_lo[t];
      hi ^= col_hi[t];
    }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t klo = ((k & 1) ? col_lo[6] : 0u) ^ ((k & 2) ? col_lo[7] : 0u);
    const uint32_t khi = ((k & 1) ? col_hi[6] : 0u) ^ ((k & 2) ? col_hi[7] : 0u);
    *reinterpret_cast<uint2 *>(table + 2 * (64 * k + lane)) = make_uint2(lo ^ klo, hi ^ khi);
  }
}

// The tables of every word of a slice, shared by a workgroup of `waves` waves.  Bound: the scalar loads of the columns, which
// have to travel before anything is built.  A wave takes a table at a time, so that the waves' loads travel together; one
// table after the other by all waves, each behind its own loads, took 1.5 us of every product with six tables (192-bit
// slices, n_in = 16: 4096 x 4096, B = 32 8.2 -> 6.7 us) and 1.1 us with nine in spmm_tile_kernel.
template <int JT>
__device__ inline void build_shared_tables(const DevLayerFor<JT> &L, int wave, int waves, int lane, int J, int nib, uint32_t *lut,
                                           int word_stride) {
  for (int i = wave; i < J * nib; i += waves) {  // uniform
    const int w = i / nib, b = i - w * nib;
    build_xor_table(lane, L.Mcol_lo + w * XORENC_MAX_N_IN + 8 * b, L.Mcol_hi + w * XORENC_MAX_N_IN + 8 * b,
                    lut + w * word_stride + 512 * b);
  }
}

constexpr int largest_divisor_at_most(int n, int cap) {
  int best = 1;
  for (int d = 1; d <= n && d <= cap; ++d)
    if (n % d == 0) best = d;
  return best;
}

constexpr int32_t kXSplit = 2;  // x_dtype of X that has been split into three bf16 matrices (inside the library only)

template <bool V>
struct BoolC {
  static constexpr bool value = V;
};

// NIBV: the layer's nib_variant (number of byte-indexed tables, one or two dwords per field; nib_variant_of), or 0:
// any n_in, read from the layer at run time (only for X that has to be fetched element by element).
// JT = most 64-bit words per slice the variant has table space for: 1 (n_out = 64) or 4 (n_out up to 256).
// NARROW: at most eight columns of X (one 16-byte chunk per row): a slice of X is 1 KB and arrives with a
// single direct load; the operand lanes of the 24 padding columns read the same chunk again.
// TERMS = 3: fp32 X that a kernel before this one has split into three bf16 matrices (hi, mid, lo, one after the other,
// each of 64 rows per word of a row of W).  The wave walks over the three slices of X of every slice of W with the same
// operands; hi has accumulators of its own, so that the sums of the large terms are rounded as they would be alone.
template <int NCB, int Q, int RB, bool XF32, int NW, bool XFAST, int NIBV, int JT, bool NARROW = false, int TERMS = 1>
__global__ __launch_bounds__(NW * 64, (NW == 4 && XFAST && !XF32) ? 2 : 1) void spmm_kernel(DevLayerFor<JT> L, const void *__restrict__ Xv, int64_t ldx, int B,
                                                      float *__restrict__ Y, int64_t ldy, int slices_per_split,
                                                      int n_splits) {
  constexpr int CW = 32 * NCB;                 // bf16 columns held in LDS per X row
  // XDIR: bf16 X with 16-byte aligned rows goes from global memory straight into LDS (no register
  // staging); the wave then owns one unpadded, swizzled slice buffer.  Otherwise X passes through
  // registers into one padded buffer.
  constexpr bool XDIR = XFAST && !XF32;
  static_assert(!NARROW || (XDIR && NCB == 1), "narrow rows of X exist on the direct path with one column block");
  constexpr int RSB = NARROW ? 16 : XDIR ? CW * 2 : CW * 2 + 16;  // LDS row stride in bytes
  constexpr int XSL = 64 * RSB;                     // the 64 X rows of one slice
  constexpr int NIBT = tables_of_variant(NIBV);
  constexpr int KC = RB * (1 + Q * (two_dwords_of_variant(NIBV) ? 2 : 1));  // compressed dwords per lane and slice (XDIR)
  // The staging area also takes the patch offsets of the wave's range (one dword
  // per lane, row block and plane), fetched ahead of everything else.
  constexpr bool OFF_DMA = XDIR;
  constexpr int KO = OFF_DMA ? RB * Q : 0;
  constexpr int CSL = (KC + KO) * 256;                    // staging area of one slice (XDIR)
  constexpr int XBUF0 = XDIR ? XSL + CSL : XSL;  // one wave's LDS share
  constexpr int ROWS = 32 * RB;
  constexpr int NR = XF32 ? CW / 3 : CW;       // real X columns per workgroup
  constexpr int NCH = NARROW ? 1 : XF32 ? NR / 4 : CW / 8;  // 16-byte chunks per X row in global memory
  constexpr int RPI = 64 / NCH;                // rows covered by one load instruction of the wave (XFAST)
  constexpr int EPC = XF32 ? 4 : 8;            // X elements per chunk
  constexpr int ESZ = XF32 ? 4 : 2;            // bytes per X element
  constexpr int NIBMAX = NIBT ? NIBT : 4;
  constexpr int TS = ROWS + 4;                 // stride (floats) between columns of a reduction tile
  constexpr int TILE = CW * TS;                // a tile is stored column-major: [column][row]
  // The epilogue keeps NREG reduction tiles in LDS (over the then idle X buffers): as many as fit
  // next to the tables, at most one per wave, and a divisor of NW so that the rounds are even.
  // (four-wave workgroups are meant to run two per CU: half of the LDS each)
  constexpr int TILE_BUDGET = (NW == 4 && XDIR && JT == 1) ? 80 * 1024 - 1024 - NW * NIBMAX * 2048
                              : (JT == 1)                ? 148 * 1024
                                                         : 160 * 1024 - 2048 - JT * NIBMAX * 2048;
  constexpr int FIT = TILE_BUDGET / (TILE * 4);
  constexpr int NREG = largest_divisor_at_most(NW, FIT);
  constexpr int LDSB0 = (NW * XBUF0 > NREG * TILE * 4) ? NW * XBUF0 : NREG * TILE * 4;
  // Flip words of GS slices (long patch lists), [slice][row block and plane][lane], zero between groups: they lie behind
  // the slice buffers, mostly where the reduction tiles will be.  Four slices if they fit without taking the room of the
  // tables per wave, else two or one.  Where these tables leave no room at all, four lists per wave share one set of tables
  // (four planes, twelve waves, odd n_in up to 24: 1280 x 6144, S = 0.9, n_in = 5, B = 88 63.9 us entry by entry, 16.4 so;
  // S = 0.91, n_in = 24, lists of few entries: 13.1 and 13.2), and fewer lists are applied entry by entry (n_in = 32 in
  // slices of one word, which hardly need patches).  So they are with more than four lists per wave of twelve waves, whose
  // state spilled 50 registers.
  constexpr int FLIP1 = RB * Q * 256;                          // one slice
  constexpr int LDS_REST = JT * NIBMAX * 2048 + Q * ROWS * 4;  // shared tables, scales
  constexpr int LDS_PRIV = NW * NIBMAX * 2048 + Q * ROWS * 4;  // tables per wave, scales
  auto lds_with = [](int gs) { return LDSB0 > NW * (XBUF0 + gs * FLIP1) ? LDSB0 : NW * (XBUF0 + gs * FLIP1); };
  auto fits = [lds_with](int gs, bool keep_priv) {
    return XDIR && (RB * Q <= 4 || NW <= 8) && lds_with(gs) + LDS_REST <= 160 * 1024 &&
           (!keep_priv || JT > 1 || LDSB0 + LDS_PRIV > 160 * 1024 || lds_with(gs) + LDS_PRIV <= 160 * 1024) &&
           (NW != 4 || lds_with(gs) + (JT == 1 ? LDS_PRIV : LDS_REST) <= 80 * 1024);
  };
  constexpr bool PRIV_FIRST = RB * Q < 4 || fits(1, true);
  constexpr int GS = fits(4, PRIV_FIRST) ? 4 : fits(2, PRIV_FIRST) ? 2 : fits(1, PRIV_FIRST) ? 1 : 0;
  static_assert(GS > 0 || !XDIR || (RB * Q > 4 && NW > 8) || (Q == 2 && NIBV == 4),
                "kernels for aligned X scatter long patch lists, but for the two stated above");
  constexpr bool SCATTER = GS > 0;
  constexpr int XBUF = XBUF0 + GS * FLIP1;
  constexpr int LDSB = lds_with(GS);
  static_assert(!XF32 || NCB % 3 == 0, "fp32 X uses three bf16 terms per column");
  static_assert(FIT >= 1, "a reduction tile must fit in the X buffers");
  static_assert(NW % NREG == 0, "waves must split evenly over the reduction tiles");
  __shared__ __attribute__((aligned(16))) uint8_t xbuf_all[LDSB];
  // Small tables are kept once per wave (no workgroup barrier before the first look-up); larger
  // ones are shared by the workgroup.
  constexpr bool PRIV_LUT = JT == 1 && NIBT >= 1 && LDSB + NW * NIBT * 2048 + Q * ROWS * 4 <= 160 * 1024;
  constexpr int LUT_WORD = NIBMAX * 512;  // dwords of the tables of one 64-bit word of a slice
  __shared__ __attribute__((aligned(16))) uint32_t lut_all[(PRIV_LUT ? NW : 1) * JT * LUT_WORD];
  uint32_t *const lut = lut_all + (PRIV_LUT ? (threadIdx.x >> 6) * LUT_WORD : 0);
  static_assert(LDSB + (PRIV_LUT ? NW : 1) * JT * LUT_WORD * 4 + Q * ROWS * 4 <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(16))) float alpha_s[Q * ROWS];

  // Every kernel argument the kernel uses is fetched up front in one batch of scalar loads (one
  // round trip to the argument segment instead of one per first use).
  const uint8_t *const l_enc = L.enc;
  const uint32_t *const l_mask32 = L.mask32;
  const uint32_t *const l_patch_off = L.patch_off;
  const uint16_t *const l_patch = L.patch;
  const float *const l_alpha = L.alpha;
  const int l_m = L.m, l_n = L.n, l_spr = L.spr, l_nrb = L.nrb, l_n_units = L.n_units, l_nib = L.nib, l_q = L.q,
            l_n_in = L.n_in;
  const int64_t l_n_slots = L.n_slots;
  const int l_J = (JT > 1) ? L.J : 1, l_espr = (JT > 1) ? L.espr : L.spr;
  const int64_t l_n_eslots = (JT > 1) ? L.n_eslots : L.n_slots;
  asm volatile("" ::"s"(l_enc), "s"(l_mask32), "s"(l_patch_off), "s"(l_patch), "s"(l_alpha), "s"(l_m), "s"(l_n),
               "s"(l_spr), "s"(l_nrb), "s"(l_n_units), "s"(l_nib), "s"(l_n_in), "s"(l_q), "s"(l_n_slots), "s"(Xv), "s"(ldx), "s"(B),
               "s"(Y), "s"(ldy), "s"(slices_per_split), "s"(n_splits));
  // a wave that has not sent its first loads yet goes before the waves that already have
  __builtin_amdgcn_s_setprio(3);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, rl = lane & 31;
  const int row0 = blockIdx.x * ROWS;
  const int col0 = blockIdx.y * NR;  // first real X column of this workgroup
  const int nib = NIBT ? NIBT : l_nib;
  const int n_in = l_n_in;
  const uint32_t enc_bytes = (uint32_t)((l_n_eslots >> 3) * l_q * n_in);  // n_eslots is a multiple of 32
  uint8_t *xbuf = xbuf_all + wave * XBUF;

  // ---- this wave's contiguous slice range [w0, w1) inside the workgroup's [s_begin, s_end)
  const int s_begin = blockIdx.z * slices_per_split;
  const int s_end = min(l_spr, s_begin + slices_per_split);
  const int total = max(0, s_end - s_begin);
  const int base_cnt = total / NW, extra = total % NW;  // the first `extra` waves take one more
  const int w0 = s_begin + wave * base_cnt + min(wave, extra);
  const int cnt = base_cnt + (wave < extra ? 1 : 0);
  const int w1 = w0 + cnt;

  // ---- buffer descriptors
  const int64_t row_bytes = ldx * ESZ;
  // (16-byte fetches are range-checked dword by dword: an odd number of bf16 columns ends in the middle of a dword,
  // which still has to count as inside; the two bytes behind it lie in the same aligned dword as the last element)
  const uint32_t term_bytes = (uint32_t)((int64_t)l_spr * 64 * row_bytes);
  const uint32_t x_extent =
      TERMS > 1 ? TERMS * term_bytes - (uint32_t)(col0 * ESZ)
                : ((uint32_t)((int64_t)(l_n - 1) * row_bytes + (int64_t)(B - col0) * ESZ) + (XFAST ? 3u : 0u)) &
                      (XFAST ? ~3u : ~0u);
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t *>(static_cast<const uint8_t *>(Xv) + (int64_t)col0 * ESZ), 0, x_extent, kRsrcFlags);
  const __amdgpu_buffer_rsrc_t mrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t *>(l_mask32), 0, (uint32_t)(l_n_slots * 8), kRsrcFlags);
  const __amdgpu_buffer_rsrc_t ersrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t *>(l_enc), 0, enc_bytes, kRsrcFlags);

  // ---- X loader.  One slice = 64 rows of X.  Chunk = 16 bytes of a row (8 bf16 / 4 fp32 columns).
  // XFAST: chunk i of a lane is (row i*RPI + lane/NCH, chunk lane%NCH), 16-byte loads.
  // otherwise: lane = row, chunk i is walked element by element (any B, ldx, alignment).
  // Chunks that lie beyond column B are redirected to chunk 0 (in bounds); what they put into the
  // padded X columns only reaches output columns that are never stored.
  // Register-light variants fetch the first two slices at once; the others fetch the second
  // slice only after the first has been copied to LDS.
  constexpr bool PRO2 = (NCH <= 8) && !XF32 && NW <= 8;
  uint4 xr[NCH];                // X rows of the slice after the one in LDS
  uint4 xr0[PRO2 ? NCH : 1];    // prologue only: X rows of the first slice
  // XDIR layout of a slice buffer: X row r sits at row position pos(r), whose bits 0..5 are bits
  // 2,3,0,1,4,5 of r, and 16-byte chunk c of that row at chunk c ^ swz(pos), swz = (pos&3)<<1 for
  // 8-chunk rows and ((pos>>1)&1)<<1 for 4-chunk rows.  The four X rows one transposing read
  // touches (r, r+4, r+8, r+12) are then four consecutive positions whose 32-byte pieces fall
  // into four different groups of eight banks.  A direct load writes lane l's 16 bytes at
  // (instruction base) + 16 l, so lane l fetches the chunk that belongs there.
  constexpr int LB = (RPI == 8) ? 3 : 4;  // position bits supplied by the lane (XDIR)
  auto row_of_pos = [](int pos) {
    return ((pos & 1) << 2) | (((pos >> 1) & 1) << 3) | ((pos >> 2) & 1) | (((pos >> 3) & 1) << 1) |
           (((pos >> 4) & 1) << 4) | (((pos >> 5) & 1) << 5);
  };
  auto swz_of_pos = [](int pos) { return NARROW ? 0 : (NCH == 8) ? ((pos & 3) << 1) : (((pos >> 1) & 1) << 1); };
  const int xrow = XDIR ? row_of_pos(lane / NCH) : (XFAST ? lane / NCH : lane);
  const int xch = XDIR ? ((lane % NCH) ^ swz_of_pos(lane / NCH)) : (XFAST ? lane % NCH : 0);
  const uint32_t x_lane_off = (uint32_t)(xrow * row_bytes) + ((col0 + xch * EPC < B) ? xch * 16 : 0);
  const uint32_t x_lds_off = XFAST ? (uint32_t)(xrow * RSB + xch * 16) : (uint32_t)(lane * RSB);
  // direct global -> LDS copy of slice s into this wave's slice buffer (XDIR)
  const uint64_t x_base = reinterpret_cast<uint64_t>(static_cast<const uint8_t *>(Xv) + (int64_t)col0 * ESZ);
  const u32x4 xdesc = {(uint32_t)x_base, (uint32_t)(x_base >> 32) & 0xffffu, x_extent, kRsrcFlags};
  const uint32_t xbuf_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)(xbuf));
  auto dma_x = [&](int s, int term = 0) {
    const uint32_t sbase = (uint32_t)(s * 64 * row_bytes) + (TERMS > 1 ? (uint32_t)term * term_bytes : 0u);  // uniform
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const uint32_t so = __builtin_amdgcn_readfirstlane(sbase + (uint32_t)(row_of_pos(i << LB) * row_bytes));
      const uint32_t dst = __builtin_amdgcn_readfirstlane(xbuf_lds + (uint32_t)(i * 1024));
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(x_lane_off),
                   "s"(xdesc), "s"(so)
                   : "memory");
    }
  };
  auto load_x = [&](int s, uint4(&xr)[NCH]) {
    const uint32_t sbase = (uint32_t)(s * 64 * row_bytes);  // uniform
    if constexpr (XFAST) {
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const u32x4 v =
            __builtin_amdgcn_raw_buffer_load_b128(xrsrc, x_lane_off, sbase + (uint32_t)(i * RPI * row_bytes), 0);
        xr[i] = make_uint4(v[0], v[1], v[2], v[3]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        uint32_t h[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
          h[e] = 0u;
          if (col0 + i * EPC + e < B) {  // uniform
            const uint32_t so = sbase + (uint32_t)((i * EPC + e) * ESZ);
            if constexpr (XF32)
              h[e] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, x_lane_off, so, 0);
            else
              h[e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(xrsrc, x_lane_off, so, 0);
          }
        }
        if constexpr (XF32)
          xr[i] = make_uint4(h[0], h[1], h[2], h[3]);
        else
          xr[i] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
      }
    }
  };
  auto store_x = [&](const uint4(&xr)[NCH]) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      // XFAST: row advances by RPI per i, chunk fixed; otherwise row fixed, chunk = i
      const int ch = XFAST ? xch : i;
      uint8_t *dst_row = xbuf + x_lds_off + (XFAST ? i * RPI * RSB : 0);
      if constexpr (!XF32) {
        *reinterpret_cast<uint4 *>(dst_row + (XFAST ? 0 : i * 16)) = xr[i];
      } else {
        // exact split of each fp32 value into three bf16 terms: hi + mid + lo
        const uint32_t f[4] = {xr[i].x, xr[i].y, xr[i].z, xr[i].w};
        uint32_t part[3][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v0 = __uint_as_float(f[e]);
          const uint32_t h0 = f32_to_bf16_rne(v0);
          const float r1 = v0 - __uint_as_float(h0 << 16);
          const uint32_t h1 = f32_to_bf16_rne(r1);
          const float r2 = r1 - __uint_as_float(h1 << 16);
          part[0][e] = h0;
          part[1][e] = h1;
          part[2][e] = f32_to_bf16_rne(r2);
        }
        // real column 4*ch+e of the tile -> LDS column part*32 + 4*ch + e (NR = 32 real columns)
        uint8_t *row_base = XFAST ? dst_row - xch * 16 : dst_row;
#pragma unroll
        for (int pt = 0; pt < 3; ++pt) {
          const uint2 w2 = make_uint2(part[pt][0] | (part[pt][1] << 16), part[pt][2] | (part[pt][3] << 16));
          *reinterpret_cast<uint2 *>(row_base + (pt * 32 + 4 * ch) * 2) = w2;
        }
      }
    }
  };

  // ---- compressed words of one slice for this lane: mask half and the dword(s) holding its
  // encrypted bits (the n_in bits of slot rl start at bit rl*n_in of the unit's run of n_in dwords)
  struct Comp {
    uint32_t mw[RB];
    uint32_t e0[RB][Q];
    uint32_t e1[RB][Q];  // second dword, only needed when a 3-byte field straddles two dwords
  };
  const bool two_dw = NIBV ? two_dwords_of_variant(NIBV) : ((n_in & (n_in - 1)) != 0);
  const uint32_t m_lane_off = (uint32_t)(rl * 8 + g * 4);
  const uint32_t e_bit = (uint32_t)(rl * n_in);
  const uint32_t e_lane_off = (e_bit >> 5) << 2;
  const uint32_t e_shift = e_bit & 31u;
  const uint32_t e_plane_units = (uint32_t)(l_n_eslots >> 5), e_unit_bytes = (uint32_t)(n_in * 4);
  auto load_comp = [&](int s, Comp &c) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int rbg = blockIdx.x * RB + rb;
      c.mw[rb] = 0u;
#pragma unroll
      for (int p = 0; p < Q; ++p) c.e0[rb][p] = c.e1[rb][p] = 0u;
      if (rbg < l_nrb) {  // uniform
        const uint32_t u = (uint32_t)(rbg * l_spr + s);  // uniform
        const uint32_t eu = (JT > 1) ? (uint32_t)(rbg * l_espr + s / l_J) : u;  // the unit's slices
        c.mw[rb] = __builtin_amdgcn_raw_buffer_load_b32(mrsrc, m_lane_off, u * 256u, 0);
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t so = ((uint32_t)p * e_plane_units + eu) * e_unit_bytes;
          c.e0[rb][p] = __builtin_amdgcn_raw_buffer_load_b32(ersrc, e_lane_off, so, 0);
          if (two_dw) c.e1[rb][p] = __builtin_amdgcn_raw_buffer_load_b32(ersrc, e_lane_off, so + 4u, 0);
        }
      }
    }
  };

  // XDIR: the compressed words take the same road as X, global memory -> LDS without a register in
  // between, one dword per lane and stream, unconditionally (a row block beyond the matrix reads a
  // zero mask through the descriptor's range check, which makes its operand +-0 whatever the
  // encrypted bits are).  No load of the loop returns into a register, so the compiler has nothing
  // to wait for and the loop's only waits on memory are the explicit ones below; the words are
  // picked up from LDS with ordinary reads after such a wait.
  const u32x4 mdesc = {(uint32_t)reinterpret_cast<uint64_t>(l_mask32),
                       (uint32_t)(reinterpret_cast<uint64_t>(l_mask32) >> 32) & 0xffffu, (uint32_t)(l_n_slots * 8),
                       kRsrcFlags};
  const u32x4 edesc = {(uint32_t)reinterpret_cast<uint64_t>(l_enc),
                       (uint32_t)(reinterpret_cast<uint64_t>(l_enc) >> 32) & 0xffffu,
                       enc_bytes, kRsrcFlags};
  constexpr int NGRP = NCH + KC;  // loads per slice
  uint32_t *const cbuf = reinterpret_cast<uint32_t *>(xbuf + (XDIR ? XSL : 0));  // after the X slice
  const uint32_t cbuf_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(size_t)(__attribute__((address_space(3))) uint32_t *)(cbuf));
  auto dma_dword = [&](uint32_t lds_addr, uint32_t lane_off, const u32x4 &desc, uint32_t so) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(
                     __builtin_amdgcn_readfirstlane(lds_addr)),
                 "v"(lane_off), "s"(desc), "s"(__builtin_amdgcn_readfirstlane(so))
                 : "memory");
  };
  auto load_comp_hidden = [&](int s) {
    int k = 0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const uint32_t u = (uint32_t)((blockIdx.x * RB + rb) * l_spr + s);  // uniform
      const uint32_t eu = (JT > 1) ? (uint32_t)((blockIdx.x * RB + rb) * l_espr + s / l_J) : u;
      dma_dword(cbuf_lds + (k++) * 256, m_lane_off, mdesc, u * 256u);
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const uint32_t so = ((uint32_t)p * e_plane_units + eu) * e_unit_bytes;
        dma_dword(cbuf_lds + (k++) * 256, e_lane_off, edesc, so);
        if (two_dw) dma_dword(cbuf_lds + (k++) * 256, e_lane_off, edesc, so + 4u);
      }
    }
  };
  auto read_comp = [&](Comp &c) {
    int k = 0;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      c.mw[rb] = cbuf[(k++) * 64 + lane];
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        c.e0[rb][p] = cbuf[(k++) * 64 + lane];
        c.e1[rb][p] = two_dw ? cbuf[(k++) * 64 + lane] : 0u;
      }
    }
  };
  auto wait_loads = [&] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

  // ---- first loads go out before anything else so that they overlap the table build
  Comp ring[2];
  const bool pre_ok = cnt <= 63;  // uniform: lane i can hold the patch offset of unit i of the range
  if constexpr (OFF_DMA) {
    // The patch offsets go first: their answer starts the only dependent read of the prologue (the patch
    // entries), which then overlaps the arrival of the first slice instead of following it.
    if (cnt > 0 && pre_ok) {
      const u32x4 odesc = {(uint32_t)reinterpret_cast<uint64_t>(l_patch_off),
                           (uint32_t)(reinterpret_cast<uint64_t>(l_patch_off) >> 32) & 0xffffu,
                           (uint32_t)(((int64_t)l_q * l_n_units + 1) * 4), kRsrcFlags};
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t u0 = (uint32_t)(p * l_n_units + (blockIdx.x * RB + rb) * l_spr + w0);  // uniform
          dma_dword(cbuf_lds + (KC + rb * Q + p) * 256, (uint32_t)(lane * 4), odesc, u0 * 4u);
        }
    }
  }
  if constexpr (XDIR) {
    if (cnt > 0) {
      load_comp_hidden(w0);
      dma_x(w0);
    }
  } else {
    if (cnt > 0) {
      load_comp(w0, ring[0]);
      if constexpr (PRO2)
        load_x(w0, xr0);
      else
        load_x(w0, xr);
    }
    if (cnt > 1) {
      load_comp(w0 + 1, ring[1]);
      if constexpr (PRO2) load_x(w0 + 1, xr);
    }
  }
  // patch offsets of the whole range: lane i holds the offset of unit i of the range
  uint32_t offv[RB][Q];
  if constexpr (!OFF_DMA) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int rbg = blockIdx.x * RB + rb;
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        offv[rb][p] = 0u;
        if (rbg < l_nrb && pre_ok && cnt > 0) {
          const uint32_t *po = l_patch_off + ((int64_t)p * l_n_units + (int64_t)rbg * l_spr + w0);
          if (lane <= cnt) offv[rb][p] = po[lane];
        }
      }
    }
  }

  __builtin_amdgcn_s_setprio(0);

  // ---- XOR tables T_b[v] = XOR of the columns 8b..8b+7 of M selected by the bits of v, and alpha
  if constexpr (PRIV_LUT) {
    for (int b = 0; b < NIBT; ++b) build_xor_table(lane, L.Mcol_lo + 8 * b, L.Mcol_hi + 8 * b, lut + 512 * b);
  } else {
    build_shared_tables(L, wave, NW, lane, l_J, nib, lut, LUT_WORD);
  }
  for (int i = tid; i < Q * ROWS; i += NW * 64) {  // read only after the barrier that follows the loop
    const int p = i / ROWS, r = row0 + i % ROWS;
    alpha_s[i] = (r < l_m) ? -0.5f * l_alpha[(int64_t)p * l_m + r] : 0.f;
  }
  if constexpr (!PRIV_LUT) __syncthreads();

  if constexpr (OFF_DMA) {
    // the offsets were the first loads of the wave: everything younger (the NGRP loads of the first slice)
    // may still be in flight
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) offv[rb][p] = 0u;
    if (cnt > 0 && pre_ok) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NGRP) : "memory");
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t v = cbuf[(KC + rb * Q + p) * 64 + lane];
          if (blockIdx.x * RB + rb < l_nrb && lane <= cnt) offv[rb][p] = v;
        }
    }
  }
  // ---- patch entries of the range: lane j holds the j-th entry (relative to the range start).
  // A range with more than 63 units or more than 64 entries of one (row block, plane) reads its
  // lists from memory inside the loop instead.
  uint32_t offrel[RB][Q], entv[RB][Q];
  bool pfast = pre_ok;
  uint32_t most_entries = 0;  // longest list of the range
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const uint32_t base = __builtin_amdgcn_readlane(offv[rb][p], 0);
      const uint32_t total = __builtin_amdgcn_readlane(offv[rb][p], pre_ok ? cnt : 0) - base;
      offrel[rb][p] = offv[rb][p] - base;
      entv[rb][p] = 0u;
      if (total > 64u) pfast = false;
      most_entries = max(most_entries, total);
      if ((uint32_t)lane < min(total, 64u)) entv[rb][p] = (l_patch + base)[lane];
    }

  f32x16 acc[Q][RB][NCB];
#pragma unroll
  for (int p = 0; p < Q; ++p)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[p][rb][cb][i] = 0.f;

  static_assert(TERMS == 1 || (TERMS == 3 && XDIR && !NARROW), "split X runs on the direct path");
  f32x16 acc_low[TERMS > 1 ? Q : 1][TERMS > 1 ? RB : 1][TERMS > 1 ? NCB : 1];  // mid and lo
  if constexpr (TERMS > 1) {
#pragma unroll
    for (int p = 0; p < Q; ++p)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc_low[p][rb][cb][i] = 0.f;
  }

  // per-lane address of the transposing reads inside the wave's buffer (see lds_read_tr16)
  const int jj = (lane >> 2) & 3, c4 = lane & 3;
  const uint8_t *tr_ptr =
      xbuf + (32 * g + 8 * (jj >> 1) + 4 * (jj & 1)) * RSB + (16 * ((lane >> 4) & 1) + 4 * c4) * 2;
  // XDIR: byte offset of this lane's 8 bytes inside a slice buffer, per column block
  uint32_t tr_off[NCB];
  {
    const int pos_lane = jj | (g << 5);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int c = NARROW ? 0 : 4 * cb + 2 * ((lane >> 4) & 1) + (c4 >> 1);
      tr_off[cb] = (uint32_t)(pos_lane * RSB + ((c ^ swz_of_pos(pos_lane)) * 16) + 8 * (c4 & 1));
    }
  }
  uint32_t *const flip_area = reinterpret_cast<uint32_t *>(xbuf + (SCATTER ? XBUF0 : 0));
  const uint32_t *lut_g0 = lut + g;
  const uint32_t lane_id5 = (uint32_t)(rl * 2 + g);  // (row, half) as it appears in a patch entry

  // table look-ups of one slice: S[rb][p] = sign half-word of this lane (before patches)
  auto lookup = [&](const Comp &c, uint32_t(&S)[RB][Q], int s) {
    // word s of a row is word s % J of its slice: that word's tables
    const uint32_t *lut_g = lut_g0 + ((JT > 1) ? (s % l_J) * LUT_WORD : 0);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        uint32_t x;
        if (two_dw)
          x = __builtin_amdgcn_alignbit(c.e1[rb][p], c.e0[rb][p], e_shift);
        else
          x = c.e0[rb][p] >> e_shift;
        uint32_t v;
        if constexpr (NIBT == 1) {
          v = lut_g[2 * (x & 255)];
        } else if constexpr (NIBT == 2) {
          const uint32_t t0 = lut_g[2 * (x & 255)], t1 = lut_g[2 * (256 + ((x >> 8) & 255))];
          v = t0 ^ t1;
        } else if constexpr (NIBT == 3) {
          const uint32_t t0 = lut_g[2 * (x & 255)], t1 = lut_g[2 * (256 + ((x >> 8) & 255))];
          const uint32_t t2 = lut_g[2 * (512 + ((x >> 16) & 255))];
          v = t0 ^ t1 ^ t2;
        } else if constexpr (NIBT == 4) {
          const uint32_t t0 = lut_g[2 * (x & 255)], t1 = lut_g[2 * (256 + ((x >> 8) & 255))];
          const uint32_t t2 = lut_g[2 * (512 + ((x >> 16) & 255))], t3 = lut_g[2 * (768 + (x >> 24))];
          v = t0 ^ t1 ^ t2 ^ t3;
        } else {
          if (n_in < 32) x &= (1u << n_in) - 1u;
          v = lut_g[2 * (x & 255)];
          if (nib > 1) v ^= lut_g[2 * (256 + ((x >> 8) & 255))];  // uniform branches
          if (nib > 2) v ^= lut_g[2 * (512 + ((x >> 16) & 255))];
          if (nib > 3) v ^= lut_g[2 * (768 + (x >> 24))];
        }
        S[rb][p] = v;
      }
  };
  // B operands of MFMA step t of the slice currently in LDS
  auto read_bfrag = [&](int t, bf16x8(&bf)[NCB]) {
    const int par = t >> 1, e = t & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      s16x4 lo, hi;
      if constexpr (XDIR) {
        // X rows +par, +2e, +16 are row positions +4, +8, +16
        const uint8_t *src = xbuf + tr_off[cb] + (4 * par + 8 * e) * RSB;
        lo = lds_read_tr16(src);
        hi = lds_read_tr16(src + 16 * RSB);
      } else {
        const uint8_t *src = tr_ptr + (2 * e + par) * RSB + cb * 64;
        lo = lds_read_tr16(src);             // operand slots 0..3
        hi = lds_read_tr16(src + 16 * RSB);  // operand slots 4..7: sixteen X rows further
      }
      bf[cb] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // Software pipeline of one wave.  While slice s is multiplied, slice s+1 moves registers -> LDS ->
  // operand registers (each operand set is refilled as soon as its MFMAs have been issued), the
  // table look-ups of slice s+1 are started, and the global loads of slice s+2 are issued.
  auto main_loop = [&](auto pf_tag, auto dense_tag) {
    constexpr bool PF = decltype(pf_tag)::value, DENSE = decltype(dense_tag)::value;
    if (cnt <= 0) return;
    uint32_t pcur[RB][Q];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < Q; ++p) pcur[rb][p] = 0u;
    // Long lists (!PF): GS slices at a time, lane j holds entry j of the group's list, requested a group ahead (offsets
    // two groups ahead), finds its slice by counting list ends and flips its bit in the slice's flip words.  (One entry
    // after the other, read from memory: 4096 x 4096, two planes, S = 0.8, n_in = 13, B = 64: 30 us, now 14.)
    constexpr bool GROUPS = !PF && SCATTER;
    uint32_t goff[3][GROUPS ? RB : 1][GROUPS ? Q : 1], gent[2][GROUPS ? RB : 1][GROUPS ? Q : 1];
    uint32_t glist[GROUPS ? RB : 1][GROUPS ? Q : 1];  // entries of the group
    auto load_group_off = [&](int s, uint32_t(&o)[GROUPS ? RB : 1][GROUPS ? Q : 1]) {
#pragma unroll
      for (int rb = 0; rb < (GROUPS ? RB : 0); ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const int rbg = blockIdx.x * RB + rb;
          o[rb][p] = 0u;
          if (rbg < l_nrb && lane <= GS)  // (units behind the range: the end of the range's last list)
            o[rb][p] = l_patch_off[(int64_t)p * l_n_units + (int64_t)rbg * l_spr + min(s + lane, w1)];
        }
    };
    auto load_group_ent = [&](const uint32_t(&o)[GROUPS ? RB : 1][GROUPS ? Q : 1], uint32_t(&e)[GROUPS ? RB : 1][GROUPS ? Q : 1]) {
#pragma unroll
      for (int rb = 0; rb < (GROUPS ? RB : 0); ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t a = __builtin_amdgcn_readlane(o[rb][p], 0);
          e[rb][p] = 0u;
          if ((uint32_t)lane < __builtin_amdgcn_readlane(o[rb][p], GS) - a) e[rb][p] = (l_patch + a)[lane];
        }
    };
    auto group_patches = [&](int s) {
      if (s > w0) {
#pragma unroll
        for (int rb = 0; rb < (GROUPS ? RB : 0); ++rb)
#pragma unroll
          for (int p = 0; p < Q; ++p) {
            goff[0][rb][p] = goff[1][rb][p];
            goff[1][rb][p] = goff[2][rb][p];
            gent[0][rb][p] = gent[1][rb][p];
          }
      }
      load_group_ent(goff[1], gent[1]);
      load_group_off(s + 2 * GS, goff[2]);
#pragma unroll
      for (int rb = 0; rb < (GROUPS ? RB : 0); ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          const uint32_t a = __builtin_amdgcn_readlane(goff[0][rb][p], 0);
          const uint32_t total = __builtin_amdgcn_readlane(goff[0][rb][p], GS) - a;
          glist[rb][p] = total;
          for (uint32_t j0 = 0; j0 < total; j0 += 64u) {  // uniform
            const uint32_t j = j0 + (uint32_t)lane;
            if (j < total) {
              uint32_t v = gent[0][rb][p];
              if (j0) v = (l_patch + a)[j];
              uint32_t t = 0;
#pragma unroll
              for (int k = 1; k < GS; ++k) t += j >= __builtin_amdgcn_readlane(goff[0][rb][p], k) - a ? 1u : 0u;
              // entry = (row%32) << 6 | bit: the word half is bit 5
              atomicXor(flip_area + (t * RB * Q + rb * Q + p) * 64 + ((v >> 6) | (v & 32u)), 1u << (v & 31u));
            }
          }
        }
    };
    // Short lists (PF): the entries of a slice are read one after the other with v_readlane, about ten instructions each;
    // where a slice has more than a few on average (DENSE), all flip their bits in the slice's flip words at once.  The
    // choice is made for the whole range: made for every slice it cost ranges with few patches 2 to 4 %.  2048 x 2048, two
    // planes, S = 0.8, n_in = 13, B = 64 11.1 -> 8.9 us; one plane, B = 8 8.4 -> 7.4.
    if constexpr (DENSE) {
#pragma unroll
      for (int i = 0; i < RB * Q; ++i) flip_area[i * 64 + lane] = 0u;
    }
    if constexpr (GROUPS) {
      // (here and not for every launch: short lists never use the area, and its 16 KB of stores ahead of the loop cost
      // 4096 x 9216, two planes, B = 64 0.15 us of 13.0)
#pragma unroll
      for (int i = 0; i < GS * RB * Q; ++i) flip_area[i * 64 + lane] = 0u;
      load_group_off(w0, goff[0]);
      load_group_off(w0 + GS, goff[1]);
      load_group_ent(goff[0], gent[0]);
    }
    bf16x8 bfrag[4][NCB];
    uint32_t Snext[RB][Q];
    if constexpr (XDIR) {
      // the first slice has landed in LDS
      wait_loads();
      read_comp(ring[0]);
      // the compiler places its own wait for the patch words here, not at their first use in the loop
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int p = 0; p < Q; ++p) {
          asm volatile("" : "+v"(offrel[rb][p]));
          asm volatile("" : "+v"(entv[rb][p]));
        }
    } else if constexpr (PRO2) {
      store_x(xr0);
    } else {
      store_x(xr);
      if (cnt > 1) load_x(w0 + 1, xr);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) read_bfrag(t, bfrag[t]);
    lookup(ring[0], Snext, w0);
    if constexpr (XDIR) {
      if (cnt > 1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the buffers have been read out
        if constexpr (TERMS == 1) {
          dma_x(w0 + 1);
          load_comp_hidden(w0 + 1);
        }
      }
      if constexpr (TERMS > 1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        dma_x(w0, 1);
      }
    }

    for (int sb = w0; sb < w1; sb += 2) {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int s = sb + d;
        if (s >= w1) break;  // uniform
        const bool has_next = s + 1 < w1;
        // the two waves that share a SIMD take turns at the higher issue priority so that neither
        // falls behind (arbitration otherwise favours the older wave for the whole kernel)
        if (((wave >> 2) & 1) == d)
          __builtin_amdgcn_s_setprio(1);
        else
          __builtin_amdgcn_s_setprio(0);
        if constexpr (!PF && SCATTER) {
          if (((s - w0) & (GS - 1)) == 0) group_patches(s);
        }
        uint32_t mw[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) mw[rb] = ring[d].mw[rb];
        // patch flips, then interleave sign and mask bits
        uint32_t Iw[RB][Q][4];  // FP4 code words, one per MFMA step
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int p = 0; p < Q; ++p) {
            uint32_t S = Snext[rb][p];
            if constexpr (!PF && SCATTER) {
              if (glist[rb][p]) {  // uniform
                uint32_t *const f = flip_area + (((s - w0) & (GS - 1)) * RB * Q + rb * Q + p) * 64 + lane;
                S ^= *f;
                *f = 0u;
              }
            } else if constexpr (PF) {
              const uint32_t pe = __builtin_amdgcn_readlane(offrel[rb][p], s - w0 + 1);
              if constexpr (DENSE) {
                uint32_t *const f = flip_area + (rb * Q + p) * 64;
                const uint32_t v = entv[rb][p];
                if ((uint32_t)lane >= pcur[rb][p] && (uint32_t)lane < pe)
                  atomicXor(f + ((v >> 6) | (v & 32u)), 1u << (v & 31u));
                S ^= f[lane];
                f[lane] = 0u;
              } else {
                for (uint32_t j = pcur[rb][p]; j < pe; ++j) {
                  const uint32_t v = __builtin_amdgcn_readlane(entv[rb][p], j);
                  if ((v >> 5) == lane_id5) S ^= 1u << (v & 31);
                }
              }
              pcur[rb][p] = pe;
            } else {
              const int rbg = blockIdx.x * RB + rb;
              if (rbg < l_nrb) {
                const int64_t u = (int64_t)p * l_n_units + (int64_t)rbg * l_spr + s;
                const uint32_t pa = __builtin_amdgcn_readfirstlane(l_patch_off[u]);
                const uint32_t pe = __builtin_amdgcn_readfirstlane(l_patch_off[u + 1]);
                for (uint32_t j = pa; j < pe; ++j) {
                  const uint32_t v = l_patch[j];
                  if ((v >> 5) == lane_id5) S ^= 1u << (v & 31);
                }
              }
            }
            const uint32_t I0 = (mw[rb] & 0x55555555u) | ((S << 1) & 0xAAAAAAAAu);
            const uint32_t I1 = ((mw[rb] >> 1) & 0x55555555u) | (S & 0xAAAAAAAAu);
            // (mask, sign) pair k of I_par moves to the top two bits of code k/2 of word k%2
            Iw[rb][p][0] = (I0 << 2) & 0xCCCCCCCCu;
            Iw[rb][p][1] = I0 & 0xCCCCCCCCu;
            Iw[rb][p][2] = (I1 << 2) & 0xCCCCCCCCu;
            Iw[rb][p][3] = I1 & 0xCCCCCCCCu;
          }
        auto mfma_step = [&](int t) {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int p = 0; p < Q; ++p) {
              const bf16x8 afrag = __builtin_bit_cast(bf16x8, expand_fp4_codes(Iw[rb][p][t]));
#pragma unroll
              for (int cb = 0; cb < NCB; ++cb)
                acc[p][rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag[t][cb], acc[p][rb][cb], 0, 0, 0);
            }
        };
        if constexpr (TERMS > 1) {
          // the buffer holds one slice of one term: while it is multiplied, the next one lands
#pragma unroll
          for (int term = 0; term < TERMS; ++term) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int p = 0; p < Q; ++p) {
                  const bf16x8 afrag = __builtin_bit_cast(bf16x8, expand_fp4_codes(Iw[rb][p][t]));
#pragma unroll
                  for (int cb = 0; cb < NCB; ++cb) {
                    f32x16 &c = term == 0 ? acc[p][rb][cb] : acc_low[p][rb][cb];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag[t][cb], c, 0, 0, 0);
                  }
                }
            if (term < TERMS - 1 || has_next) {  // uniform
              __builtin_amdgcn_sched_barrier(0);
              wait_loads();
              __builtin_amdgcn_sched_barrier(0);
              if (term == TERMS - 1) {
                read_comp(ring[d ^ 1]);
                lookup(ring[d ^ 1], Snext, s + 1);
              }
#pragma unroll
              for (int t = 0; t < 4; ++t) read_bfrag(t, bfrag[t]);
              __builtin_amdgcn_sched_barrier(0);
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              if (term == 0) {
                dma_x(s, 2);
              } else if (term == 1) {
                if (has_next) {
                  dma_x(s + 1, 0);
                  load_comp_hidden(s + 1);
                }
              } else {
                dma_x(s + 1, 1);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
          continue;
        }
        mfma_step(0);
        if constexpr (XDIR) {
          // slice s is entirely in operand registers, slice s+1 is landing; it is read
          // out at the end of the iteration and the buffer handed to slice s+2
          mfma_step(1);
          mfma_step(2);
          mfma_step(3);
          if (has_next) {
            __builtin_amdgcn_sched_barrier(0);
            wait_loads();
            __builtin_amdgcn_sched_barrier(0);
            read_comp(ring[d ^ 1]);
            lookup(ring[d ^ 1], Snext, s + 1);
#pragma unroll
            for (int t = 0; t < 4; ++t) read_bfrag(t, bfrag[t]);
            if (s + 2 < w1) {
              __builtin_amdgcn_sched_barrier(0);
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              dma_x(s + 2);
              load_comp_hidden(s + 2);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        } else {
          mfma_step(1);
          // all operands of slice s are in registers: the LDS buffer takes slice s+1, whose operand
          // reads follow in program order (LDS ops of one wave execute in order)
          if (has_next) store_x(xr);
          if (s + 2 < w1) {
            load_comp(s + 2, ring[d]);
            load_x(s + 2, xr);
          }
          if (has_next) {
            read_bfrag(0, bfrag[0]);
            read_bfrag(1, bfrag[1]);
          }
          mfma_step(2);
          if (has_next) read_bfrag(2, bfrag[2]);
          mfma_step(3);
          if (has_next) {
            read_bfrag(3, bfrag[3]);
            lookup(ring[d ^ 1], Snext, s + 1);
          }
        }
      }
    }
  };
  constexpr uint32_t kFewEntries = 3;  // of a slice's list, on average
  if (!pfast)
    main_loop(BoolC<false>{}, BoolC<false>{});
  else if (SCATTER && most_entries > kFewEntries * (uint32_t)cnt)
    main_loop(BoolC<true>{}, BoolC<SCATTER>{});
  else
    main_loop(BoolC<true>{}, BoolC<false>{});

  // ---- epilogue: scale by alpha (fp32) and reduce the waves in a fixed order.  NREG tiles of
  // CW x TS floats (column-major) live in LDS over the (now idle) X buffers; wave w adds into tile w % NREG in round
  // w / NREG, then every thread sums the NREG tiles of its outputs pairwise.
  // acc element i of a lane is row 8*(i/4) + 4*g + i%4, column rl of its 32x32 block.
  // every wave has left its loop: the X buffers are idle and alpha_s (written by the first waves
  // without a barrier of its own) is complete
  __syncthreads();
  // One plane: its scales wait until the waves' sums have been added, 4 multiplications a thread there instead of 16 per 32 x 32
  // block in every wave here, where all of them issue at once, and one rounding a sum less: 2.6e-8 instead of 5.4e-8 from the
  // exact result.  (Time: 0 to 1 %, no more than two placements of the same buffers differ.)
  // A sum that leaves the range of fp32 (or is not a number) is taken again from scaled parts, which may stay inside it: by its
  // thread where every wave has a tile of its own, by the workgroup where two waves share one, behind a barrier that costs
  // what the multiplications did (16384 x 4096, B = 128 22.0 -> 22.4 us, B = 256 35.0 -> 35.7).
  constexpr bool SCALE_LAST = Q == 1 && !XF32 && TERMS == 1;
  constexpr bool REDO = SCALE_LAST && NREG < NW;
  bool out_of_range = false;
  for (bool scaled = !SCALE_LAST;; scaled = true) {
    if (scaled) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
          f32x4 a4[Q];
#pragma unroll
          for (int p = 0; p < Q; ++p)
            a4[p] = *reinterpret_cast<const f32x4 *>(alpha_s + p * ROWS + rb * 32 + 8 * j4 + 4 * g);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if constexpr (TERMS > 1) {
#pragma unroll
                for (int p = 0; p < Q; ++p) acc[p][rb][cb][4 * j4 + k] += acc_low[p][rb][cb][4 * j4 + k];
              }
              float v = a4[0][k] * acc[0][rb][cb][4 * j4 + k];
#pragma unroll
              for (int p = 1; p < Q; ++p) v += a4[p][k] * acc[p][rb][cb][4 * j4 + k];
              acc[0][rb][cb][4 * j4 + k] = v;  // plane 0's accumulator now holds the scaled sum
            }
        }
    }
    float *red = reinterpret_cast<float *>(xbuf_all);
    for (int round = 0; round < NW / NREG; ++round) {
      if (wave / NREG == round) {
        float *tile = red + (wave % NREG) * TILE;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
              // four consecutive rows of one column: one 16-byte LDS access; columns beyond B are never
              // stored, so their lanes stay out (with few columns most of the tile is such padding)
              if (XF32 || col0 + cb * 32 + rl < B) {
                f32x4 *dst = reinterpret_cast<f32x4 *>(tile + (cb * 32 + rl) * TS + rb * 32 + 8 * j4 + 4 * g);
                f32x4 v = {acc[0][rb][cb][4 * j4], acc[0][rb][cb][4 * j4 + 1], acc[0][rb][cb][4 * j4 + 2],
                           acc[0][rb][cb][4 * j4 + 3]};
                if (round != 0) v += *dst;
                *dst = v;
              }
            }
      }
      __syncthreads();
    }
    // final pass: a thread owns four consecutive rows of one column; lanes run over columns, so each
    // of its four stores is contiguous across the wave
    auto reduced4 = [&](int col, int rq) {
      // (added in pairs, pairs of pairs, ...: fewer roundings on the way of each part than one after the other)
      const float *src = red + col * TS + 4 * rq;
      f32x4 v[NREG];
#pragma unroll
      for (int r = 0; r < NREG; ++r) v[r] = *reinterpret_cast<const f32x4 *>(src + r * TILE);
#pragma unroll
      for (int s = 1; s < NREG; s *= 2)
#pragma unroll
        for (int r = 0; r + s < NREG; r += 2 * s) v[r] += v[r + s];
      if constexpr (SCALE_LAST) {
        if (scaled) return v[0];
        const f32x4 a = *reinterpret_cast<const f32x4 *>(alpha_s + 4 * rq);
        const bool in_range = fabsf(v[0][0]) + fabsf(v[0][1]) + fabsf(v[0][2]) + fabsf(v[0][3]) < __builtin_huge_valf();
        v[0] *= a;
        if (!in_range) {
          out_of_range = true;
          if constexpr (!REDO) {
#pragma unroll
            for (int r = 0; r < NREG; ++r) v[r] = *reinterpret_cast<const f32x4 *>(src + r * TILE) * a;
#pragma unroll
            for (int s = 1; s < NREG; s *= 2)
#pragma unroll
              for (int r = 0; r + s < NREG; r += 2 * s) v[r] += v[r + s];
          }
        }
      }
      return v[0];
    };
    // n_splits > 1: this workgroup holds one of n_splits partial sums of its tile.  It parks the tile in the
    // scratch area and takes a ticket; the workgroup that arrives last adds the parts in the order
    // of their slice ranges (so the result does not depend on who was last) and writes Y.  No zero-fill, no
    // atomics on Y, nobody waits for anybody.
    float *const my_part =
        n_splits > 1 ? L.split_part + ((int64_t)(blockIdx.y * gridDim.x + blockIdx.x) * n_splits + blockIdx.z) * kSplitTileFloats
                     : nullptr;
    for (int idx = tid; idx < (ROWS / 4) * NR; idx += NW * 64) {
      const int rq = idx / NR, nn = idx % NR;
      const int gc = col0 + nn;
      if (gc < B) {
        f32x4 v;
        if (XF32) {
          const int c = 96 * (nn >> 5) + (nn & 31);
          v = (reduced4(c, rq) + reduced4(c + 32, rq)) + reduced4(c + 64, rq);
        } else {
          v = reduced4(nn, rq);
        }
        if (n_splits > 1) {
          split_store4(split_rsrc(my_part), 16u * idx, __builtin_bit_cast(u32x4, v));
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int gr = row0 + 4 * rq + k;
            if (gr < l_m) Y[(int64_t)gr * ldy + gc] = v[k];
          }
        }
      }
    }
    if (!REDO || scaled || !__syncthreads_or(out_of_range)) break;  // uniform
  }
  if (n_splits > 1) {
    static_assert(ROWS * NR <= kSplitTileFloats || RB > 2, "a split launch's tile must fit its slot");
    __shared__ uint32_t last_arrival;
    const int tile_id = blockIdx.y * gridDim.x + blockIdx.x;
    // the parts were written with device-coherent stores; once they are acknowledged the ticket may be taken
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) last_arrival = __hip_atomic_fetch_add(L.split_ticket + tile_id, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(n_splits - 1) ? 1u : 0u;
    __syncthreads();
    if (last_arrival) {
      const __amdgpu_buffer_rsrc_t parts = split_rsrc(L.split_part + (int64_t)tile_id * n_splits * kSplitTileFloats);
      for (int idx = tid; idx < (ROWS / 4) * NR; idx += NW * 64) {
        const int rq = idx / NR, nn = idx % NR;
        const int gc = col0 + nn;
        if (gc < B) {
          // two to four parts, (0 + 1) + (2 + 3)
          auto part = [&](int z) {
            return __builtin_bit_cast(f32x4, split_load4(parts, (uint32_t)z * (kSplitTileFloats * 4u) + 16u * idx));
          };
          f32x4 v = part(0) + part(1);
          if (n_splits > 2) v += n_splits > 3 ? part(2) + part(3) : part(2);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int gr = row0 + 4 * rq + k;
            if (gr < l_m) Y[(int64_t)gr * ldy + gc] = v[k];
          }
        }
      }
      if (tid == 0) L.split_ticket[tile_id] = 0u;  // ready for the next launch
    }
  }
}

template <int NCB, int Q, int RB, bool XF32, int NW, bool XFAST, int NIBV, int JT, bool NARROW = false, int TERMS = 1>
inline void launch_variant(const DevLayer &D, const void *X, int64_t ldx, int B, float *Y, int64_t ldy, dim3 grid,
                           int sps, int n_splits, hipStream_t st) {
  hipLaunchKernelGGL((spmm_kernel<NCB, Q, RB, XF32, NW, XFAST, NIBV, JT, NARROW, TERMS>), grid, dim3(NW * 64), 0, st,
                     layer_argument<JT>(D), X,
                     ldx, B, Y, ldy, sps, n_splits);
}

// XMODE: 0 = the call site may see either layout, 1 = aligned X only, 2 = generic X only (keeps
// variants that are never launched from being compiled)
template <int NCB, int Q, int RB, bool XF32, int NW = 8, int XMODE = 0, int JMODE = 0, bool NARROW = false, int TERMS = 1>
int32_t launch_spmm(const DevLayer &D, const void *X, int64_t ldx, int B, float *Y, int64_t ldy, int x_fast,
                    hipStream_t st) {
  constexpr int NR = XF32 ? (32 * NCB) / 3 : 32 * NCB;
  const int row_groups = (D.nrb + RB - 1) / RB;
  const int col_groups = (B + NR - 1) / NR;
  const ReductionCut cut = cut_reduction(CutVariant{Q, NR / 32, RB, NW, D.J == 1, TERMS > 1, !x_fast || XF32}, D.spr, row_groups,
                                         col_groups, D.split_part && D.split_ticket);
  const int sps = cut.sps;
  const dim3 grid(row_groups, col_groups, cut.ks);
  const int atomic = cut.ks;  // number of splits: the kernel reduces them through the scratch area when > 1
  // JMODE: 1 = slices of one 64-bit word only, 4 = up to four words (more table space), 0 = both
  if (D.J > 1 && JMODE == 1) return XORENC_EUNSUPPORTED;
  const bool wide = (JMODE == 4) || (JMODE == 0 && D.J > 1);
  if (!x_fast) {
    if constexpr (XMODE != 1) {
      if constexpr (JMODE != 1)
        if (wide) launch_variant<NCB, Q, RB, XF32, NW, false, 0, 4>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st);
      if constexpr (JMODE != 4)
        if (!wide) launch_variant<NCB, Q, RB, XF32, NW, false, 0, 1>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st);
    } else {
      return XORENC_EUNSUPPORTED;
    }
  } else if constexpr (XMODE == 2) {
    return XORENC_EUNSUPPORTED;
  } else {
    if constexpr (JMODE != 1)
      if (wide) switch (D.nib_variant) {
          case 1: launch_variant<NCB, Q, RB, XF32, NW, true, 1, 4, false, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          case 2: launch_variant<NCB, Q, RB, XF32, NW, true, 2, 4, false, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          case 3: launch_variant<NCB, Q, RB, XF32, NW, true, 3, 4, false, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          case 4: launch_variant<NCB, Q, RB, XF32, NW, true, 4, 4, false, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          default: launch_variant<NCB, Q, RB, XF32, NW, true, kFourTablesTwoDwords, 4, false, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
        }
    if constexpr (JMODE != 4)
      if (!wide) switch (D.nib_variant) {
          case 1: launch_variant<NCB, Q, RB, XF32, NW, true, 1, 1, NARROW, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          case 2: launch_variant<NCB, Q, RB, XF32, NW, true, 2, 1, NARROW, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st); break;
          case 3:
            // (the four-wave workgroups that share a CU have LDS for one or two tables per wave only)
            if constexpr (NW == 4 && !XF32) return XORENC_EUNSUPPORTED;
            else launch_variant<NCB, Q, RB, XF32, NW, true, 3, 1, NARROW, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st);
            break;
          case 4:
            if constexpr (NW == 4 && !XF32) return XORENC_EUNSUPPORTED;
            else launch_variant<NCB, Q, RB, XF32, NW, true, 4, 1, NARROW, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st);
            break;
          default:
            if constexpr (NW == 4 && !XF32) return XORENC_EUNSUPPORTED;
            else launch_variant<NCB, Q, RB, XF32, NW, true, kFourTablesTwoDwords, 1, NARROW, TERMS>(D, X, ldx, B, Y, ldy, grid, sps, atomic, st);
            break;
        }
  }
  return xorenc_internal_check_launch();
}

// Tile shapes per (Q, column blocks): Q*RB*NCB accumulator sets of 16 registers must leave room
// for the X prefetch registers at two waves per SIMD.
template <int Q>
int32_t dispatch_spmm_q(const DevLayer &D, const void *X, int32_t x_dtype, int64_t ldx, int B, float *Y, int64_t ldy,
                        int x_fast, hipStream_t st) {
  if (x_dtype == kXSplit) {  // fp32 X as three bf16 matrices
    if constexpr (Q <= 2) {
      if (B > 32) {
        if constexpr (Q == 1) {
          // (64-row tiles once they give every CU one; X is re-read half as often)
          if ((int64_t)((D.nrb + 1) / 2) * ((B + 63) / 64) >= 200)
            return launch_spmm<2, Q, 2, false, 8, 1, 0, false, 3>(D, X, ldx, B, Y, ldy, x_fast, st);
        }
        return launch_spmm<2, Q, 1, false, 8, 1, 0, false, 3>(D, X, ldx, B, Y, ldy, x_fast, st);
      }
      return launch_spmm<1, Q, 1, false, 12, 1, 0, false, 3>(D, X, ldx, B, Y, ldy, x_fast, st);
    } else {
      // (four planes keep 8 to 10 registers in scratch memory, 5 without the loop for short lists of several entries: 4096 x
      // 4096, S = 0.91, n_in = 16, B = 64 24.3 us with and without that loop, 2048 x 2048, S = 0.8, n_in = 14, B = 32 12.5
      // against 13.7)
      return launch_spmm<1, Q, 1, false, 8, 1, 0, false, 3>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
  }
  if (x_dtype == XORENC_X_F32) {
    if constexpr (Q <= 2)
      return launch_spmm<3, Q, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    else
      return launch_spmm<3, Q, 1, true, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
  }
  const int blocks = (B + 31) / 32;
  // Small layers take 32-row tiles: twice the workgroups (still one round), half the accumulators and half the tile
  // exchange per wave.  It pays while a wave's share of the reduction stays short (measured: up to eight slices
  // per wave it wins, 2048 x 16384 at B = 64 14.4 against 16.8 us; at sixteen it loses, 8192 x 8192 19.7 against
  // 16.6 us): slices per wave with 32-row tiles, nw waves and the most workgroups per tile.
  auto rb1_slices_per_wave = [&](int nw, int col_groups) {
    const int64_t tiles = (int64_t)D.nrb * col_groups;
    if (tiles > kSplitMaxGroups) return 1 << 30;
    int ks = 1;
    if (tiles < kSplitMaxGroups) ks = max(1, min(min((D.spr + nw - 1) / nw, (int)(kSplitMaxGroups / tiles)), kSplitMaxParts));
    const int sps = (D.spr + ks - 1) / ks;
    return (sps + nw - 1) / nw;
  };
  const bool small_wide = rb1_slices_per_wave(8, (B + 63) / 64) <= 8;    // 33 and more columns, eight waves
  const bool small_block = rb1_slices_per_wave(12, blocks) <= 8;         // one column block, twelve waves
  const bool small_narrow = rb1_slices_per_wave(12, 1) <= 12;            // at most eight columns
  // Among 32-row tiles: eight or twelve waves, one or two blocks of columns, by the estimate of cut_reduction.  Twelve
  // waves have shorter shares and more partial tiles to add (2048 x 4096, B = 8 6.4 against 6.7 us; 1024 x 1024, three
  // planes 6.4 against 6.2); one block of columns spares the meeting of workgroups while its tiles fit one round
  // (2048 x 2048, B = 64 5.9 against 7.8 us; 2048 x 8192 10.6 against 10.0).
  auto estimate = [&](int ncb, int nw) {
    const int groups = (blocks + ncb - 1) / ncb;
    if ((int64_t)D.nrb * groups > kSplitMaxGroups) return 1e9;
    return cut_reduction(CutVariant{Q, ncb, 1, nw, D.J == 1, false, false}, D.spr, D.nrb, groups,
                         D.split_part && D.split_ticket).us;
  };
  const bool eight_waves = estimate(1, 8) <= estimate(1, 12);
  const bool one_block = estimate(1, 8) < estimate(2, 8);
  // Slices of several words: 32-row tiles, twelve waves, while they fit one round, also with one plane (us, 64-row tiles /
  // here: n_out = 192, n_in = 20, 2048 x 2048, B = 64 11.9 / 7.5, 1024 x 8192 16.8 / 10.7; three planes 16.4 / 12.1;
  // n_out = 128, n_in = 16, 2500 x 1500, three planes, B = 32 11.5 / 8.7; 6000 x 3000, two blocks of columns 13.1 / 10.9).
  if constexpr (Q <= 3) {
    if (x_fast && D.J > 1) {
      if constexpr (Q <= 2)
        if (blocks > 1 && estimate(2, 8) < estimate(1, 12)) return launch_spmm<2, Q, 1, false, 8, 1, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
      if ((int64_t)D.nrb * blocks <= kSplitMaxGroups) return launch_spmm<1, Q, 1, false, 12, 1, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
  }
  if constexpr (Q == 1) {
    if (!x_fast) {
      if (blocks == 1) return launch_spmm<1, Q, 2, false, 16, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<2, Q, 2, false, 8, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    if (B <= 8 && D.J == 1 && small_narrow) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // more than one round of 64-row tiles: four-wave workgroups, several per CU, so that one's prologue and epilogue
    // overlap another's loop (65536 x 4096 at B = 8: 28.9 against 30.4 us)
    if (B <= 8 && D.J == 1 && D.nib_variant <= 2 && (D.nrb + 1) / 2 > kSplitMaxGroups)
      return launch_spmm<1, Q, 2, false, 4, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (B <= 8 && D.J == 1) return launch_spmm<1, Q, 2, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    // (small layers: 32-row tiles while they fit one round, see above)
    if (blocks == 1 && D.J == 1 && small_block) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // (several rounds: four-wave workgroups as above; 65536 x 4096 at B = 32: 32.5 against 34.8 us)
    if (blocks == 1 && D.J == 1 && D.nib_variant <= 2 && (D.nrb + 1) / 2 > kSplitMaxGroups)
      return launch_spmm<1, Q, 2, false, 4, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (blocks == 1) return launch_spmm<1, Q, 2, false, 12, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    // 128-row tiles halve the number of times X is re-read; used once they still fill most of the chip.
    // Up to 256 of them run as eight-wave workgroups, one per CU, in a single round; more run as
    // four-wave workgroups, two per CU, which share the CU's LDS so that one's prologue and epilogue do
    // not wait for the other's to finish.
    const int64_t tiles128 = (int64_t)((D.nrb + 3) / 4) * ((B + 63) / 64);
    if (D.J == 1 && D.nib_variant <= 2 && tiles128 > 256)
      return launch_spmm<2, Q, 4, false, 4, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (D.J == 1 && tiles128 >= 200) return launch_spmm<2, Q, 4, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (D.J == 1 && small_wide) {
      if (one_block) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<2, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    return launch_spmm<2, Q, 2, false, 8, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
  } else if constexpr (Q == 2) {
    if (B <= 8 && x_fast && D.J == 1 && small_narrow) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    if (B <= 8 && x_fast && D.J == 1 && D.nib_variant <= 2 && (D.nrb + 1) / 2 > kSplitMaxGroups)
      return launch_spmm<1, Q, 2, false, 4, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (B <= 8 && x_fast && D.J == 1) return launch_spmm<1, Q, 2, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (blocks == 1 && x_fast && D.J == 1 && small_block) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    if (blocks == 1 && x_fast) return launch_spmm<1, Q, 2, false, 12, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (blocks == 1) return launch_spmm<1, Q, 2, false, 8, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (!x_fast) return launch_spmm<2, Q, 1, false, 8, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (D.J > 1) return launch_spmm<2, Q, 1, false, 8, 1, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
    // 64-row tiles once they fill most of the chip: X is re-read half as often; more than 256 of them run as
    // four-wave workgroups, two per CU
    const int64_t tiles64 = (int64_t)((D.nrb + 1) / 2) * ((B + 63) / 64);
    if (D.nib_variant <= 2 && tiles64 > 256) return launch_spmm<2, Q, 2, false, 4, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (tiles64 >= 200) return launch_spmm<2, Q, 2, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (one_block) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    return launch_spmm<2, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
  } else if constexpr (Q == 3) {
    if (B <= 8 && x_fast && D.J == 1 && small_narrow) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // (64-row tiles: eight waves, which have registers for lists of many patches (16384 x 1024, S = 0.8, n_in = 16, B = 32
    // 14.8 -> 9.9 us, n_out = 192, n_in = 30 82.9 -> 16.2); twelve on longer rows of one-word slices with few patches,
    // 16384 x 4096, S = 0.95, n_in = 8, B = 8 16.3 against 17.3, 16384 x 3000, S = 0.91, n_in = 16 12.6 against 12.7, 4096 x
    // 9216, B = 64 19.0 against 18.8.  Twelve take lists of more than 64 entries one after the other from memory: S = 0.8,
    // n_in = 13, 8200 x 2600, B = 8 66 against 20, 4096 x 9216, B = 64 109 against 31.  The host does not know the lists.)
    const bool twelve = D.J == 1 && D.spr > 40;
    if (B <= 8 && x_fast && D.J == 1) {
      if (twelve) return launch_spmm<1, Q, 2, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 2, false, 8, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // (32-row tiles on small layers: 6000 x 3000 at B = 32 9.8 against 12.3 us)
    if (x_fast && D.J == 1 && small_block) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // (more than one round of them: two blocks of columns, 6000 x 3000 at B = 64 12.6 against 14.8 us, 8192 x 1024 at
    // B = 128 13.7 against 16.5)
    if (x_fast && D.J == 1 && blocks > 1 && (int64_t)D.nrb * blocks > kSplitMaxGroups)
      return launch_spmm<2, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (x_fast && twelve) return launch_spmm<1, Q, 2, false, 12, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (x_fast) return launch_spmm<1, Q, 2, false, 8, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    return launch_spmm<1, Q, 2, false, 8, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
  } else {
    if (!x_fast) return launch_spmm<1, Q, 1, false, 8, 2>(D, X, ldx, B, Y, ldy, x_fast, st);
    if (D.J > 1) {
      if ((int64_t)D.nrb * blocks <= kSplitMaxGroups) return launch_spmm<1, Q, 1, false, 12, 1, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 8, 1, 4>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    // (one slice buffer per wave instead of two: 1024 x 8192, B = 64 11.4 against 12.1 us)
    if (B <= 8) {
      if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
      return launch_spmm<1, Q, 1, false, 12, 1, 1, true>(D, X, ldx, B, Y, ldy, x_fast, st);
    }
    if (eight_waves) return launch_spmm<1, Q, 1, false, 8, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
    return launch_spmm<1, Q, 1, false, 12, 1, 1>(D, X, ldx, B, Y, ldy, x_fast, st);
  }
}

}  // namespace xorenc_spmm_detail

// one translation unit per Q instantiates these
int32_t xorenc_spmm_dispatch_q1(const DevLayer &, const void *, int32_t, int64_t, int, float *, int64_t, int, hipStream_t);
int32_t xorenc_spmm_dispatch_q2(const DevLayer &, const void *, int32_t, int64_t, int, float *, int64_t, int, hipStream_t);
int32_t xorenc_spmm_dispatch_q3(const DevLayer &, const void *, int32_t, int64_t, int, float *, int64_t, int, hipStream_t);
int32_t xorenc_spmm_dispatch_q4(const DevLayer &, const void *, int32_t, int64_t, int, float *, int64_t, int, hipStream_t);

#endif

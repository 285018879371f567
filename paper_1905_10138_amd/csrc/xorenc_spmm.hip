// xorenc_spmm entry point: argument validation and dispatch to the per-Q kernel instantiations.
#include <mutex>

#include "xorenc_scratch.h"
#include "xorenc_spmm_f4.h"

// Memory that products need beside their arguments, on every GPU from the time the library is loaded: sets of tickets and
// slots (xorenc_scratch.h says whose they are).  A slot holds the partial tiles of one launch that splits the reduction
// dimension over several workgroups per output tile (small layers that would otherwise leave most of the chip idle), and
// a staging area for X.  Tickets are zero between launches: the array starts zeroed and the last workgroup of a tile
// resets its counter.  In host code an array's name is only a handle for hipGetSymbolAddress; kernels get the
// looked-up address.
//
// Staging: the fast kernels fetch X in 16-byte pieces and need rows that start on 16-byte boundaries.  When the caller's
// X does not (a leading dimension that is not a multiple of eight bf16 or four fp32 values, or an odd base address) and
// it fits, a small kernel copies it into the staging area with padded rows first (one more launch, about 2 us) and the
// product runs on the copy (B = 33: 16 against 43 us, B = 65: 25 against 170 us on a 16384 x 4096 layer); larger X are
// copied and multiplied in parts (4096 x 9216, two planes, B = 1023: 2700 us on the element-wise kernels, 278 us).
namespace {
constexpr int64_t kXSplitMinWeights = 6000000;   // fp32 X: weights (of all planes), or weights times columns, from which
constexpr int64_t kXSplitMinWork = 600000000;    // it is split by a kernel of its own
constexpr int kStageMinB = 5;                    // (fewer columns are faster on the kernels that read X element by element)
constexpr int kSplitMinWords = 5;  // no kernel splits the reduction of rows with fewer words (the narrowest has four waves)
static_assert(kTicketBytes % 256 == 0 && kPartBytes % 256 == 0 && kSlotBytes % 256 == 0, "all keep the arrays' alignment");
static_assert(kSlotBytes == XORENC_SPMM_WORKSPACE_BYTES, "a workspace holds what a slot holds");

// dst[k][0 .. cpr*16) = row k of X (B elements of esz bytes, leading dimension ldx), zero-filled to whole 16-byte
// pieces; one thread per piece
__global__ __launch_bounds__(256) void stage_x_kernel(const unsigned char *__restrict__ X, int64_t ldx, int n, int B,
                                                      int esz, int cpr, unsigned char *__restrict__ dst) {
  const int64_t piece = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (piece >= (int64_t)n * cpr) return;
  const int k = (int)(piece / cpr), c = (int)(piece - (int64_t)k * cpr);
  const int per = 16 / esz;
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  const unsigned char *row = X + (int64_t)k * ldx * esz;
  if (esz == 2) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int col = c * per + e;
      if (col < B) w[e >> 1] |= (uint32_t) * reinterpret_cast<const uint16_t *>(row + 2 * col) << (16 * (e & 1));
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int col = c * per + e;
      if (col < B) w[e] = *reinterpret_cast<const uint32_t *>(row + 4 * col);
    }
  }
  *reinterpret_cast<uint4 *>(dst + piece * 16) = make_uint4(w[0], w[1], w[2], w[3]);
}

// fp32 X -> three bf16 matrices hi, mid, lo of `rows` x 8 cpr values whose sum is X exactly; one thread per 8 columns
// of a row, rows from n on and columns from B on are zero
__global__ __launch_bounds__(256) void split_x_kernel(const float *__restrict__ X, int64_t ldx, int n, int rows, int B,
                                                      int cpr, unsigned char *__restrict__ dst) {
  const int64_t piece = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (piece >= (int64_t)rows * cpr) return;
  const int k = (int)(piece / cpr), c = 8 * (int)(piece - (int64_t)k * cpr);
  const float *row = X + (int64_t)k * ldx + c;
  const bool wide = (reinterpret_cast<uintptr_t>(row) & 15) == 0 && c + 8 <= B;
  float v[8];
  if (k >= n) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.f;
  } else if (wide) {
    const float4 a = *reinterpret_cast<const float4 *>(row), b = *reinterpret_cast<const float4 *>(row + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = c + e < B ? row[e] : 0.f;
  }
  uint32_t w[3][4];
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) w[t][e] = 0u;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t h0 = f32_to_bf16_rne(v[e]);
    const float r1 = v[e] - __uint_as_float(h0 << 16);
    const uint32_t h1 = f32_to_bf16_rne(r1);
    const uint32_t h2 = f32_to_bf16_rne(r1 - __uint_as_float(h1 << 16));
    w[0][e >> 1] |= h0 << (16 * (e & 1));
    w[1][e >> 1] |= h1 << (16 * (e & 1));
    w[2][e >> 1] |= h2 << (16 * (e & 1));
  }
  const int64_t term = (int64_t)rows * cpr;
#pragma unroll
  for (int t = 0; t < 3; ++t)
    *reinterpret_cast<uint4 *>(dst + (t * term + piece) * 16) = make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]);
}
}  // namespace
static __device__ __align__(256) unsigned char scratch_area[kScratchOwners * kTicketBytes + kScratchSlots * kSlotBytes];

namespace {
constexpr int kMaxDevices = 64;

// Tickets and, unless the caller brings memory, a slot for a call on `st` of the current device; null where none are left.
struct Scratch {
  uint32_t *tickets;
  unsigned char *slot;
  uint32_t ring;
};

int32_t take_scratch(hipStream_t st, bool captured, uint64_t capture, bool want_slot, int copies, size_t copy_bytes, Scratch *out) {
  static std::mutex lock;
  static unsigned char *address[kMaxDevices] = {};
  static ScratchOwners owners[kMaxDevices];
  static thread_local char this_thread;
  int dev = -1;
  const hipError_t ed = hipGetDevice(&dev);
  if (ed != hipSuccess) return xorenc_internal_hip_status((int32_t)ed);
  if (dev < 0 || dev >= kMaxDevices) return XORENC_EUNSUPPORTED;
  std::lock_guard<std::mutex> guard(lock);
  if (!address[dev]) {
    void *p = nullptr;
    const hipError_t es = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch_area));
    if (es != hipSuccess) return xorenc_internal_hip_status((int32_t)es);
    if (!p) return XORENC_EHIP;
    address[dev] = static_cast<unsigned char *>(p);
  }
  const ScratchOwner owner{st, st == hipStreamPerThread ? &this_thread : nullptr, captured ? capture : 0};
  const ScratchShare share = owners[dev].share(owner, want_slot, copies, copy_bytes);
  out->tickets = share.tickets < 0 ? nullptr : reinterpret_cast<uint32_t *>(address[dev] + share.tickets * kTicketBytes);
  out->slot = share.slot < 0 ? nullptr : address[dev] + kScratchOwners * kTicketBytes + share.slot * kSlotBytes;
  out->ring = share.ring;
  return XORENC_OK;
}

// Without a workspace and a slot the call runs on the kernels that need neither, or is refused (limit_is_error).
int32_t spmm_common(const xorenc_layer *layer, const void *X, int32_t x_dtype, int64_t ldx, int32_t B, float *Y, int64_t ldy,
                    unsigned char *workspace, bool limit_is_error, void *hip_stream) {
  DevLayer D;
  const int32_t rc = xorenc_fill_dev_layer(layer, &D);
  if (rc != XORENC_OK) return rc;
  if (!X || !Y || B <= 0 || ldx < B || ldy < B) return XORENC_EINVAL;
  if (x_dtype != XORENC_X_F32 && x_dtype != XORENC_X_BF16) return XORENC_EUNSUPPORTED;
  const int esz = x_dtype == XORENC_X_F32 ? 4 : 2;
  // X, the mask and the encrypted stream are addressed through buffer descriptors with 32-bit offsets
  if ((int64_t)layer->n * ldx * esz >= ((int64_t)1 << 32) || D.n_slots * 8 >= ((int64_t)1 << 32) ||
      D.n_eslots * D.q * D.n_in / 8 >= ((int64_t)1 << 32))
    return XORENC_EUNSUPPORTED;
  if (((uintptr_t)Y & 3) || ((uintptr_t)X & (esz - 1))) return XORENC_EALIGN;
  // 16-byte loads of X need whole chunks (8 bf16 / 4 fp32 columns) and 16-byte aligned rows
  const int per = 16 / esz;
  // (a last piece with fewer columns is fetched whole: what lies behind column B inside the row's pitch only
  // reaches output columns that are never stored)
  const bool aligned = (ldx % per == 0) && (((uintptr_t)X & 15) == 0);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // fp32 X: split into three bf16 matrices in the staging area, as many columns at a time as fit (in whole 64s where
  // there are more).  The product then runs on the direct-to-LDS kernels, which convert nothing; the launch and the pass
  // over X cost 2 to 3 us, so small layers keep the kernels that split X on its way into LDS (us, B = 1 / 8 / 64 / 200:
  // 1024 x 1024 9.8 8.3 8.5 12.6, here 9.4 9.3 9.8 12.2; 2048 x 2048 11.2 9.9 10.9 29.2, here 9.9 9.9 12.0 20.4;
  // 4096 x 4096 17.6 15.2 22.6 83.7, here 12.1 12.1 16.9 47.6; 4096 x 9216 with two planes 34.6 29.3 51.5 465, here
  // 18.8 18.8 32.0 120).
  int split_parts = 0, split_cols = 0;
  size_t copy_bytes = 0;  // of the largest part
  const int64_t weights = (int64_t)layer->m * layer->n * layer->q;
  // Slices of several words: smaller layers, and few columns of bf16 (below), gain from a split or a copy too, because the
  // kernels behind it have 32-row tiles and scatter long patch lists.  In a graph nearly always (1.7x in the mean of 141
  // random layers, few patches 1.0 to 1.7, long lists up to 8).  But a second launch costs a program that calls directly 3 us
  // of host time: 11 us a call become 14 where the kernels are shorter than that.  So it is made where the kernels that do
  // without take longest: many tables to build, or many words of all planes per row to walk through, or large layers.  Over
  // the 141 layers direct calls are 1.29 times as fast so, 1.27 with two launches at any size; 34 of the 49 that lost more
  // than 5 % no longer do (us, direct calls, one launch / two: n_out = 128, 1024 x 1024, n_in = 8, B = 1 11.1 / 14.0; fp32,
  // 2223 x 1002, two planes, n_in = 24, B = 8 11.6 / 14.0), the others have tables for 12 and more (n_out = 192, n_in = 32,
  // S = 0.9, 1000 x 1000, B = 2 13.3 / 15.0, in a graph 14.3 / 8.8; S = 0.8, 768 x 2400, B = 1 29.8 / 14.9).
  // Rows of fewer than kSplitMinWords words, for which no call needed memory before, stay as they were: accepted without any.
  const bool two_launches = D.J > 1 && D.spr >= kSplitMinWords &&
                            (D.J * tables_of_variant(D.nib_variant) >= 12 || D.q * D.spr >= 40 || weights >= 20000000);
  // (us, split on the way / before: n_out = 192, n_in = 24, three planes, 1024 x 1024, B = 33 18.6 / 13.7; n_out = 256,
  // 768 x 2400, B = 33 23.3 / 14.5; S = 0.8, n_in = 30, 2048 x 2048, B = 64 40.7 / 14.1.  One plane with few tables and two
  // blocks of columns stays with the sizes above: n_out = 128, n_in = 16, 1024 x 1024, B = 64 10.2 / 11.5.)
  const bool wide_split = two_launches && (D.q > 1 || B <= 32 || D.nib_variant > 2);
  if (x_dtype == XORENC_X_F32 && (weights >= kXSplitMinWeights || weights * B >= kXSplitMinWork || wide_split)) {
    const int64_t fit = (int64_t)(kStageBytes / ((size_t)D.spr * 64 * 48)) * 8;  // columns that fit
    if (fit >= min(B, 64)) {
      split_cols = fit >= B ? B : (int)(fit / 64 * 64);
      split_parts = (B + split_cols - 1) / split_cols;
      copy_bytes = (size_t)D.spr * 64 * ((split_cols + 7) / 8) * 48;
    }
    // Parts of few tiles leave most of the chip idle, one after the other, and each builds the tables anew, where the
    // kernels that split X on its way run all columns at once: parts only from 64 tiles each (32 where X would have to be
    // copied in parts instead, 24 with four tables for each of four words per slice, which the others take longest to
    // build), and on small layers not at all (us, in parts / otherwise: 264 x 4157,
    // B = 911 114 / 41; 595 x 6443, two planes, B = 376 98 / 39; 438 x 2378, two planes, B = 508 39 / 23; 236 x 2033, four
    // planes, B = 370 41 / 28; 913 x 2042, n_in = 32, n_out = 256, B = 734 68 / 168; 2186 x 3700, unaligned, B = 570 101 / 116).  Over
    // 242 calls in parts, 200 x 1500 to 14000 x 9216: 2 % from the better choice in the mean, 19 % without the rule.
    if (split_parts > 1) {
      const int64_t tiles = (int64_t)D.nrb * ((split_cols + (D.q <= 2 ? 63 : 31)) / (D.q <= 2 ? 64 : 32));
      const bool copied = !aligned && (int64_t)layer->n * ((B + per - 1) / per) * 16 > (int64_t)kStageBytes;
      const bool most_tables = D.J * tables_of_variant(D.nib_variant) >= 16;
      if (tiles < (most_tables ? 24 : copied ? 32 : 64) || (weights < 3000000 && !copied && !most_tables)) split_parts = 0;
    }
  }
  // rows of X that do not start on 16-byte boundaries: a padded copy, unless the few-column kernel (which reads X
  // element by element anyway) takes the call.  A copy that does not fit the staging area is made and multiplied a part
  // of the columns at a time: at least 64 columns have to fit (n <= 32768 bf16, 16384 fp32), and the parts differ by one
  // piece at most, so that none is so narrow (25 columns at least) that it would run, and round, as a call with few
  // columns does.
  int copy_parts = 0;
  const int pieces_per_row = (int)(((int64_t)B + per - 1) / per);  // 16-byte pieces
  // Widths whose fields straddle dwords, 17 to 24 bits aside, and one block of columns: the copy and the three or four
  // tables per word of the kernels for aligned X cost small calls more than reading X element by element does (us, copied /
  // not: 212 x 1558, two planes, n_out = 192, n_in = 5, B = 7 15.4 / 11.9; 2698 x 460, fp32, n_in = 5, B = 9 9.5 / 8.2;
  // 2918 x 1006, four planes, n_out = 128, n_in = 13, B = 11 11.5 / 9.6; with one word per slice bf16 gains all the same,
  // 752 x 2716, three planes, B = 18 10.7 / 15.9, and fp32 from seventeen columns on, 6217 x 842, B = 27 10.9 / 14.1).
  const bool odd_width = (D.n_in & (D.n_in - 1)) != 0 && (D.n_in < 17 || D.n_in > 24);
  const bool copy_pays = !odd_width || B > 32 ||
                         (D.J == 1 ? x_dtype == XORENC_X_BF16 || B > 16 : weights >= (D.n_in > 24 ? 2000000 : 20000000));
  // Few columns of bf16 and slices of several words, as above (us, element by element / copied: n_out = 192, n_in = 24, two
  // planes, 4096 x 4096, B = 1 19.5 / 12.6; three planes, n_out = 256, 1024 x 1024, B = 2 19.2 / 10.8; S = 0.85, n_in = 30,
  // 9968 x 6732, two planes 240 / 33; four planes 1024 x 1024 11.2 / 11.7, 768 x 7424 18.4 / 15.8).
  const bool few_wide = two_launches && x_dtype == XORENC_X_BF16 && (layer->q < 4 || weights >= 20000000);
  if (!split_parts && !aligned && (B >= kStageMinB || few_wide) && copy_pays) {
    const int64_t fit = (int64_t)(kStageBytes / ((size_t)layer->n * 16)) * per / 64 * 64;  // columns, in whole 64s
    const bool whole = (int64_t)layer->n * pieces_per_row * 16 <= (int64_t)kStageBytes;
    F4Plan unused;
    if ((whole || fit > 0) && !xorenc_spmm_detail::f4_applies(D, x_dtype, B, 0, &unused))
      copy_parts = whole ? 1 : (int)((B + fit - 1) / fit);
    // (fp32 parts of few tiles of 32 columns: as above, 225 x 6154, three planes, B = 171 46 / 40 us without the copies,
    // 624 x 5320, B = 199 37 / 74)
    if (copy_parts > 1 && x_dtype == XORENC_X_F32) {
      const int cols = (pieces_per_row + copy_parts - 1) / copy_parts * per;
      if ((int64_t)D.nrb * ((cols + 31) / 32) < 48) copy_parts = 0;
    }
    if (copy_parts) copy_bytes = (size_t)layer->n * ((pieces_per_row + copy_parts - 1) / copy_parts) * 16;
  }
  Scratch scratch{};
  // A copy and the product that reads it are enqueued together: another thread's call on the same stream must not get its
  // copy, which may go to the same place, in between.
  static std::mutex enqueue[64];
  std::unique_lock<std::mutex> together;
  if (split_parts || copy_parts)
    together = std::unique_lock<std::mutex>(enqueue[(reinterpret_cast<uintptr_t>(st) >> 4) % 64]);
  if (split_parts || copy_parts || D.spr >= kSplitMinWords) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    unsigned long long capture = 0;
    // (an error here, such as a capture elsewhere that bars the default stream, comes back from the launch)
    if (hipStreamGetCaptureInfo(st, &capturing, &capture) != hipSuccess) capturing = hipStreamCaptureStatusNone;
    const bool captured = capturing != hipStreamCaptureStatusNone;
    if (captured && !workspace && limit_is_error) return XORENC_ELIMIT;
    const int32_t rs = take_scratch(st, captured, capture, !workspace, split_parts + copy_parts, copy_bytes, &scratch);
    if (rs != XORENC_OK) return rs;
    if (workspace) scratch.slot = workspace;
    if (!scratch.slot && limit_is_error) return XORENC_ELIMIT;
  }
  xorenc_internal_begin_call();
  D.split_part = scratch.tickets ? reinterpret_cast<float *>(scratch.slot) : nullptr;
  D.split_ticket = scratch.tickets;
  auto next_copy = [&] { return scratch.slot + kPartBytes + ring_place(scratch.ring, copy_bytes); };
  auto product = [&](const void *Xp, int64_t ld, int32_t cols, float *Yp, int fast, int32_t x_dtype) -> int32_t {
    switch (layer->q) {
      case 1: return xorenc_spmm_dispatch_q1(D, Xp, x_dtype, ld, cols, Yp, ldy, fast, st);
      case 2: return xorenc_spmm_dispatch_q2(D, Xp, x_dtype, ld, cols, Yp, ldy, fast, st);
      case 3: return xorenc_spmm_dispatch_q3(D, Xp, x_dtype, ld, cols, Yp, ldy, fast, st);
      default: return xorenc_spmm_dispatch_q4(D, Xp, x_dtype, ld, cols, Yp, ldy, fast, st);
    }
  };
  if (scratch.slot) {
    for (int i = 0, c0 = 0; i < split_parts; ++i, c0 += split_cols) {
      unsigned char *const copy = next_copy();
      const int rows = D.spr * 64, cols = min(split_cols, B - c0), cpr = (cols + 7) / 8;
      const int64_t pieces = (int64_t)rows * cpr;
      hipLaunchKernelGGL(split_x_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st,
                         static_cast<const float *>(X) + c0, ldx, (int)layer->n, rows, cols, cpr, copy);
      const int32_t rp = product(copy, (int64_t)cpr * 8, cols, Y + c0, 1, xorenc_spmm_detail::kXSplit);
      if (rp != XORENC_OK) return rp;
    }
    for (int i = 0, c0 = 0; i < copy_parts; ++i) {
      unsigned char *const copy = next_copy();
      const int cpr = pieces_per_row / copy_parts + (i < pieces_per_row % copy_parts ? 1 : 0);
      const int cols = min(cpr * per, B - c0);
      const int64_t pieces = (int64_t)layer->n * cpr;
      hipLaunchKernelGGL(stage_x_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st,
                         static_cast<const unsigned char *>(X) + (int64_t)c0 * esz, ldx, (int)layer->n, cols, esz, cpr,
                         copy);
      const int32_t rp = product(copy, (int64_t)cpr * per, cols, Y + c0, 1, x_dtype);
      if (rp != XORENC_OK) return rp;
      c0 += cols;
    }
    if (split_parts || copy_parts) return XORENC_OK;
  }
  return product(X, ldx, B, Y, aligned ? 1 : 0, x_dtype);
}
}  // namespace

extern "C" int32_t xorenc_spmm(const xorenc_layer *layer, const void *X, int32_t x_dtype, int64_t ldx, int32_t B,
                               float *Y, int64_t ldy, void *hip_stream) {
  return spmm_common(layer, X, x_dtype, ldx, B, Y, ldy, nullptr, false, hip_stream);
}

extern "C" int32_t xorenc_spmm_ws(const xorenc_layer *layer, const void *X, int32_t x_dtype, int64_t ldx, int32_t B,
                                  float *Y, int64_t ldy, void *workspace, int64_t workspace_bytes, void *hip_stream) {
  if (workspace && workspace_bytes < (int64_t)XORENC_SPMM_WORKSPACE_BYTES) return XORENC_EINVAL;
  if ((uintptr_t)workspace & 15) return XORENC_EALIGN;
  return spmm_common(layer, X, x_dtype, ldx, B, Y, ldy, static_cast<unsigned char *>(workspace), true, hip_stream);
}

// Kernels and C ABI of libnvfp4_46.so (gfx950).  See include/nvfp4_46.h for the
// contract of every entry point.
//
// Data movement
//   rowwise   A row-major tensor whose rows are multiples of 16 is one flat
//             stream of 16-element blocks, and so are its outputs: block k reads
//             32 bytes at 32k, writes 8 code bytes at 8k and 1 scale byte at k.
//             One lane owns one block (two 128-bit loads, all 16 values in
//             registers, no cross-lane traffic); a wave's 64 lanes cover 2 KiB of
//             contiguous input, 512 B of codes and 64 B of scales.
//   columnwise / both
//             A workgroup stages a 64x128 tile of x in LDS (coalesced 128-bit
//             loads), every lane then reads two adjacent columns x 16 rows from
//             LDS, and the results go back through LDS so that each column's 32
//             code bytes leave as one contiguous run.  When both orientations
//             are wanted the rowwise half is produced from the registers of the
//             staging loads, so x is read from HBM once.
#include <hip/hip_runtime.h>

#include <atomic>

#include "block.hpp"
#include "launch.hpp"
#include "layer.hpp"
#include "nvfp4_46.h"
#include "nvfp4_46_fused.h"
#include "small_tensors.hpp"
#include "tensor.hpp"
#include "tile_shapes.hpp"

// The quantizing kernels exist once per (input type, rounding mode, selection rule, ...):
// several hundred instantiations.  To compile them side by side this file can be built in
// parts: NVFP4_46_PART = 1..6 holds the kernels of one (input type, rounding mode) pair and
// nothing else, NVFP4_46_PART = 0 holds everything else (the entry points included) and
// refers to the six groups as explicit instantiations defined elsewhere.  Without the
// macro the file is one self-contained translation unit.
#ifndef NVFP4_46_PART
#define NVFP4_46_PART (-1)
#endif
#define NVFP4_46_MAIN (NVFP4_46_PART <= 0)

namespace nvfp4_46 {

constexpr int kThreads = 256;
enum : int { kOutCodes = 0, kOutFake = 1, kOutAmax = 2, kOutScaleAndCodes = 3 };

// Launch shapes (workgroups per compute unit; every kernel strides over its input).  Each
// value is the fastest of a timed sweep on 8192 x 8192 tensors.
constexpr int kAmaxUnroll = 8;          // independent 128-bit loads per lane in k_amax_plain
constexpr int kAmaxWgPerCu = 1;         // k_amax_plain: few, long-lived workgroups, each ends
                                        // with a serialising access to the one result word
constexpr int kFlatLongWgPerCu = 6;     // k_flat with outputs: long-lived workgroups (5 ... 8
                                        // timed; 8 leaves no slot for the short ones)
constexpr int kFlatShortRoundsPerCu = 16;  // ... and rounds left to one-round workgroups
constexpr int kFlatAmaxWgPerCu = 2;     // k_flat as the amax pass of the Hadamard transform
constexpr int kAmaxRhtColWgPerCu = 8;   // k_amax_rht_col

// The pass for the tensor scale reads x just before the quantizing pass, both usually first to
// last.  A tensor larger than what the 256 MB memory-side cache holds of it has then always just
// lost the part that is read next; read last to first, the quantizing pass finds most of a
// cacheful.  Scale + quantize, us, forwards / backwards, (a) on seven tensors in turn, (b) on one that a
// kernel has just written, (c) on the same one again (the next scale pass then finds its head):
//                                                       (a)        (b)          (c)
//   fp32 8192 x 8192, both packings of 16x16 tiles   137 / 116   143 / 130   121 / 116
//                     rowwise                        103 / 98    115 / 113    92 / 92
//                     both orientations              128 / 120   138 / 134   118 / 115
//   BF16 16384 x 8192, columnwise                    127 / 119   136 / 131   113 / 113
//                      rowwise                       118 / 114   126 / 126   103 / 104
// (d) On a tensor whose last write the host has waited for the orders differ little (tiles 124 / 124,
// BF16 columnwise 138 / 136, fp32 rowwise 99 / 100).  Below the line everything is found either way (BF16
// 8192 x 8192: 16x16 tiles 70 / 71, both orientations 81 / 82), so small tensors keep their order.
constexpr int64_t kLastLevelBytes = (int64_t)192 << 20;
constexpr uint32_t runs_backwards(int64_t elements, bool xf32) {
  return elements * (xf32 ? 4 : 2) > kLastLevelBytes;
}

// Streaming accesses.  Dequantized BF16 tensors are write-once streams and leave with
// nontemporal stores (dequantize 45 -> 28 us per 8192 x 8192, and their write-back no
// longer competes with the next kernel).  Codes, scales and choice bytes use ordinary
// stores so that the consumer finds them in L2 / the memory-side cache (nontemporal
// stores gain 1.5 us here and cost the following dequantize 4-5 us).  Loads are ordinary
// (nontemporal loads are slower when x is cache-resident and neutral otherwise).
constexpr bool kNtCodes = false;   // codes / scales / choice bytes
constexpr bool kNtBf16 = true;     // dequantized BF16 tensors
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <bool NT>
NV_DEV void store_as(uint4 *p, const uint4 &v) {
  if (NT) {
    u32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4 *>(p));
  } else {
    *p = v;
  }
}
template <bool NT>
NV_DEV void store_as(uint2 *p, const uint2 &v) {
  if (NT) {
    u32x2 t = {v.x, v.y};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x2 *>(p));
  } else {
    *p = v;
  }
}
template <bool NT>
NV_DEV void store_as(uint8_t *p, uint8_t v) {
  if (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// Where a reduction kernel leaves its result.  Plain form (scratch == nullptr): `amax_bits` is
// the caller's alpha word, zeroed by a launch before and turned into alpha by a launch after.
// One-launch form: `scratch` is zeroed scratch memory (layout below); the workgroup that
// finishes last applies Eq. (1), writes alpha, and the scratch is all zero again.
//
// Device-scope atomics on one address are carried out one after the other at the memory side
// (about 15-35 ns each here: 256 workgroups that all finish together queued up for 9 of the
// 27 us of a pass over 8192 x 8192).  So the workgroups report in a two-level tree: sixteen
// groups, each with its own maximum and ticket words on cache lines of their own; the last workgroup of a
// group draws a top ticket, and who draws the last of those collects the sixteen maxima at once.  Two
// chains of at most ~grid/16 + 16 atomics replace one of 2 x grid.  What a pass over a small tensor then waits
// for is the last workgroup's dependent trips to the memory side, about a quarter of a microsecond each: its
// maximum, two tickets, the collection (us in a replayed graph, x in the memory-side cache, against eight
// trips where each maximum was looked at first, fetched from its group and raised at the top: 256 KiB 4.65 ->
// 3.9, 1 MiB 4.9 -> 4.1, 16 MiB 5.4 -> 4.7, 2 MiB with the columnwise transform 6.5 -> 5.7).
struct AmaxFinish {
  uint32_t *scratch;   // kScratchWords words, or nullptr
  float *alpha;
  float fp8_max;
};
constexpr uint32_t kAmaxGroups = 16;
constexpr uint32_t kScratchStride = 32;   // words between two slots: one 128-byte line each
// slot g: maximum of group g; slot 16 + g: its ticket; slot 33: top ticket.  Two tensors in one launch: the second has
// the upper eight groups and slot 32 for its top ticket.
constexpr uint32_t kScratchWords = (2 * kAmaxGroups + 2) * kScratchStride;
constexpr uint32_t kGroupMayQueue = 32;   // members from which on a group's maximum is looked at before it is raised
NV_DEV uint32_t *scratch_slot(uint32_t *scratch, uint32_t i) { return scratch + i * kScratchStride; }

// max into *word; the returning form, waited for, so that the maximum is in before anything the
// caller does next.  `look`: skipped when a read already shows a value at least as large (the value only
// ever grows), for words that many workgroups queue for.
NV_DEV void atomic_max_now(uint32_t *word, uint32_t bits, bool look) {
  if (look && bits <= __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  uint32_t old = __hip_atomic_fetch_max(word, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(old) : : "memory");
}

// Fold a workgroup's maximum magnitude into the global one.  Bit patterns of non-negative
// floats order like the values, so an integer atomic max is exact and order-free.
// Device-scope atomics are carried out at the one place all compute dies share, so "carried
// out before" needs no cache maintenance, only program order: a workgroup's maximum is in
// before its ticket is drawn, a group's last ticket before the top one, and whoever draws the grid's last
// ticket collects the maxima after that.
// `share`: which of a launch's workgroups belong to the tensor, and which half of the words, if not all.
struct AmaxShare {
  uint32_t block, blocks, half, halves;
};
NV_DEV AmaxShare whole_launch() { return AmaxShare{blockIdx.x, gridDim.x, 0u, 1u}; }
NV_DEV void publish_amax(float m, uint32_t *amax_bits, const AmaxFinish &fin, const AmaxShare share) {
  __shared__ float wave_part[kThreads / 64];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x >= 64) return;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) m = fmaxf(m, wave_part[w]);
  const uint32_t bits = f2u(m);
  if (!fin.scratch) {
    if (threadIdx.x == 0) atomic_max_now(amax_bits, bits, true);
    return;
  }
  const uint32_t most = kAmaxGroups / share.halves, first = most * share.half;
  const uint32_t groups = share.blocks < most ? share.blocks : most;
  const uint32_t g = share.block % groups;
  const uint32_t members = (share.blocks - g + groups - 1) / groups;  // workgroups b with b % groups == g
  uint32_t *gticket = scratch_slot(fin.scratch, kAmaxGroups + first + g);
  uint32_t *top_ticket = scratch_slot(fin.scratch, 2 * kAmaxGroups + 1 - share.half);
  uint32_t last = 0;
  if (threadIdx.x == 0) {
    atomic_max_now(scratch_slot(fin.scratch, first + g), bits, members >= kGroupMayQueue);
    if (__hip_atomic_fetch_add(gticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1) {
      __hip_atomic_store(gticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = __hip_atomic_fetch_add(top_ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == groups - 1;
    }
  }
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  // last of all: the groups' maxima, one per lane, and all words zero again
  uint32_t all = 0;
  if (threadIdx.x < groups)
    all = __hip_atomic_exchange(scratch_slot(fin.scratch, first + threadIdx.x), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (uint32_t off = kAmaxGroups / 2; off > 0; off >>= 1) {
    const uint32_t other = (uint32_t)__shfl_xor((int)all, (int)off, 64);
    all = other > all ? other : all;
  }
  if (threadIdx.x != 0) return;
  __hip_atomic_store(top_ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *fin.alpha = alpha_of(u2f(all), fin.fp8_max);
}

// ------------------------------------------------------------ tensor scale

#if NVFP4_46_MAIN
__global__ void k_store_u32(uint32_t *p, uint32_t v) { *p = v; }

__global__ void k_finish_alpha(float *alpha, float fp8_max) { *alpha = alpha_of(*alpha, fp8_max); }
#endif

// max|x| without the transform.  Several independent 128-bit loads per lane are in flight at a time.
template <bool XF32>
__global__ __launch_bounds__(kThreads) void k_amax_plain(const uint4 *__restrict__ x, int64_t n16,
                                                         uint32_t *amax_bits, AmaxFinish fin) {
  PlainAmax<XF32> m;
  constexpr int U = kAmaxUnroll;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (; i + (U - 1) * stride < n16; i += U * stride) {
    uint4 w[U];
#pragma unroll
    for (int j = 0; j < U; ++j) w[j] = load_stream(x + i + j * stride);
#pragma unroll
    for (int j = 0; j < U; ++j) m.fold(w[j]);
  }
  for (; i < n16; i += stride) m.fold(load_stream(x + i));
  publish_amax(m.value(), amax_bits, fin, whole_launch());
}

// A small tensor, one workgroup for all of it: nothing has to be agreed on between workgroups, so
// no scratch words, no atomics and no launches before and after.  Sixteen waves with eight
// loads each in flight take what one compute unit can (256 KiB in 3.3 us); small_tensors.hpp says
// where that ends.
constexpr int kSmallThreads = 1024;
constexpr int kSmallBlocks = 256;             // blocks per workgroup of k_scale_quantize_small
template <bool XF32>
NV_DEV float small_tensor_alpha(const uint4 *__restrict__ x, uint32_t n16, float fp8_max) {
  __shared__ float wave_part[kSmallThreads / 64];
  PlainAmax<XF32> acc;
  constexpr int U = 8;
  uint32_t i = threadIdx.x;
  for (; i + (U - 1) * kSmallThreads < n16; i += U * kSmallThreads) {
    uint4 w[U];
#pragma unroll
    for (int j = 0; j < U; ++j) w[j] = load_stream(x + i + j * kSmallThreads);
#pragma unroll
    for (int j = 0; j < U; ++j) acc.fold(w[j]);
  }
  if (i < n16) {
    // the rest, still with all its loads in flight; past the end the lane's first piece again
    uint4 w[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t k = i + j * kSmallThreads;
      w[j] = load_stream(x + (k < n16 ? k : i));
    }
#pragma unroll
    for (int j = 0; j < U; ++j) acc.fold(w[j]);
  }
  float m = wave_max(acc.value());
  if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSmallThreads / 64; ++w) m = fmaxf(m, wave_part[w]);
  return alpha_of(m, fp8_max);
}

#if NVFP4_46_MAIN
template <bool XF32>
__global__ __launch_bounds__(kSmallThreads) void k_scale_small(const uint4 *__restrict__ x, uint32_t n16,
                                                               float *alpha, float fp8_max) {
  const float a = small_tensor_alpha<XF32>(x, n16, fp8_max);
  if (threadIdx.x == 0) *alpha = a;
}
#endif

// max|y| over the Hadamard-transformed column blocks (16 consecutive rows of one column),
// without LDS: a lane loads WORDS words (one, or four: 8 BF16 or 4 fp32 columns, a wave's loads cover 1 KiB of each
// row) from each of the 16 rows of a row block and transforms every column in registers.  The signs depend on the row only, so they are flipped in the packed
// words; the factor 1/4 of the transform is applied once to the maximum (scaling by a power
// of two is monotonic, so the maximum of the scaled values is the scaled maximum).
template <bool XF32, int WORDS>
NV_DEV float amax_rht_col(const uint32_t *__restrict__ x, int64_t row_blocks, int64_t pieces_per_row, uint64_t rht_seed,
                          uint32_t block, uint32_t blocks) {
  const int64_t items = row_blocks * pieces_per_row;
  const int64_t stride = (int64_t)blocks * kThreads;
  float m = 0.0f;
  for (int64_t item = (int64_t)block * kThreads + threadIdx.x; item < items; item += stride) {
    const int64_t rb = item / pieces_per_row, piece = item - rb * pieces_per_row;
    const uint32_t *src = x + (rb * 16 * pieces_per_row + piece) * WORDS;
    struct alignas(4 * WORDS) Piece {
      uint32_t w[WORDS];
    } p[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) p[j] = *reinterpret_cast<const Piece *>(src + j * pieces_per_row * WORDS);
    const uint32_t sw = rht_sign_word(rht_seed, (uint64_t)rb);
    constexpr uint32_t kSignBits = XF32 ? 0x80000000u : 0x80008000u;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint32_t flip = (0u - ((sw >> j) & 1u)) & kSignBits;    // row j of the block
#pragma unroll
      for (int q = 0; q < WORDS; ++q) p[j].w[q] ^= flip;
    }
#pragma unroll
    for (int c = 0; c < (XF32 ? WORDS : 2 * WORDS); ++c) {
      float v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const uint32_t word = p[j].w[XF32 ? c : c >> 1];
        v[j] = u2f(XF32 || (c & 1) ? (XF32 ? word : word & 0xffff0000u) : word << 16);
      }
      // the butterflies of rht16() (strides 1, 2, 4, 8), signs already applied, no scaling
#pragma unroll
      for (int h = 1; h < 16; h <<= 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if ((i & h) == 0) {
            const float a = v[i], b = v[i + h];
            v[i] = a + b;
            v[i + h] = a - b;
          }
        }
      }
#pragma unroll
      for (int j = 0; j < 16; j += 2) m = fmaxf(m, fmaxf(fabsf(v[j]), fabsf(v[j + 1])));
    }
  }
  return m * 0.25f;
}
template <bool XF32, int WORDS>
__global__ __launch_bounds__(kThreads) void k_amax_rht_col(const uint32_t *__restrict__ x,
                                                           int64_t row_blocks, int64_t pieces_per_row,
                                                           uint64_t rht_seed, uint32_t *amax_bits,
                                                           AmaxFinish fin) {
  const float m = amax_rht_col<XF32, WORDS>(x, row_blocks, pieces_per_row, rht_seed, blockIdx.x, gridDim.x);
  publish_amax(m, amax_bits, fin, whole_launch());
}

// The maxima of two BF16 tensors after the columnwise transform, in one launch: the operands of a weight gradient, whose
// blocks share their rows and signs.  The first `blocks_a` workgroups take a, the others b.
struct AmaxPair {
  const uint32_t *x[2];
  int64_t pieces_per_row[2];
  float *alpha[2];
};
template <int WORDS>
__global__ __launch_bounds__(kThreads) void k_amax_rht_col_pair(AmaxPair p, int64_t row_blocks, uint64_t rht_seed,
                                                                uint32_t blocks_a, uint32_t *scratch, float fp8_max) {
  const uint32_t i = blockIdx.x >= blocks_a;
  const uint32_t block = blockIdx.x - (i ? blocks_a : 0u), blocks = i ? gridDim.x - blocks_a : blocks_a;
  const float m = amax_rht_col<false, WORDS>(p.x[i], row_blocks, p.pieces_per_row[i], rht_seed, block, blocks);
  publish_amax(m, nullptr, AmaxFinish{scratch, p.alpha[i], fp8_max}, AmaxShare{block, blocks, i, 2u});
}

// -------------------------------------------------------- rowwise (flat)

template <bool XF32, int ROUNDING, int SELECT, bool RHT, int OUT>
__global__ __launch_bounds__(kThreads) void k_flat(
    const uint4 *__restrict__ x, const float *__restrict__ alpha_p, uint2 *__restrict__ codes,
    uint8_t *__restrict__ scales, uint8_t *__restrict__ choice, uint4 *__restrict__ out_bf16,
    uint32_t *amax_bits, int64_t nblocks, uint32_t nb_per_row, uint64_t sr_seed,
    uint64_t rht_seed, uint32_t n_long, uint32_t rounds_long, uint32_t backwards, AmaxFinish fin) {
  __shared__ ScaleTable tab;
  // fake-quant only: a wave's 2 KiB of output is turned round in LDS so that each of its
  // two store instructions writes 1 KiB of whole cache lines (streaming stores of half
  // lines are slow), instead of every lane writing its own 32 bytes
  __shared__ uint4 xpose[OUT == kOutFake ? 2 * kThreads : 1];
  // The tensor is cut into rounds of 256 consecutive blocks, dealt to two classes of
  // workgroups: the first n_long workgroups take rounds_long rounds each (w, w + n_long, ...,
  // all below n_long * rounds_long), the others share the remaining rounds (one each, when
  // the launcher sizes the grid for it; in general w', w' + n_short, ...).  A workgroup pays
  // a full memory latency before its first round, with its wave slots idle: the long ones,
  // few enough to be resident all at once, pay it once for most of the tensor, and the short
  // ones, launched as slots fall free, even out the end.  Everything that depends on the
  // round only (base pointers, the number of live lanes) is wave-uniform and stays on the
  // scalar unit; a lane adds its own constant offset.
  const uint32_t tid = threadIdx.x;
  const uint32_t rounds = (uint32_t)((nblocks + kThreads - 1) / kThreads);
  const uint32_t tail = (uint32_t)(nblocks - (int64_t)(rounds - 1) * kThreads);  // 1..256
  // The sign flips of the transform as XOR masks of a lane, in LDS (piece q of lane t at [q][t]: a wave's 128-bit
  // reads are conflict-free): one per value, or, kPacked, one per word of two BF16 values, which are then flipped before
  // they are unpacked.  The second is eight instructions and two LDS reads a block instead of sixteen and four,
  // but they stand before everything else.  It pays under the squared-error rule, by registers (Hadamard + SR 98 -> 89, five
  // waves per SIMD), and costs the others (BF16, us, per value / packed: 8192 x 8192 to nearest by mean absolute error
  // 4.2 %, with SR 5.1 %, always 6 with SR 1.2 %; 20000 x 8192 5.5, 4.8 and 3.1 %).  A lane writes and reads only its own
  // slots, and the LDS operations of one wave execute in order, so no barrier is involved.
  constexpr bool kPacked = !XF32 && SELECT == kSel46;
  using Raw = RawBlock<XF32>;
  constexpr int kMaskPieces = kPacked ? Raw::kPieces : 4;
  __shared__ uint4 sign_masks[RHT ? kMaskPieces : 1][RHT ? kThreads : 1];
  uint32_t B_lane = 0, sign_B = 0xffffffffu;
  if (RHT) B_lane = tid % nb_per_row;
  // the values of a block as it arrived
  auto values = [&](const Raw &raw, float (&w)[16]) {
    if constexpr (!RHT) {
      unpack16(raw, w);
    } else if constexpr (kPacked) {
      Raw flipped;
#pragma unroll
      for (int q = 0; q < Raw::kPieces; ++q) {
        const uint4 m = sign_masks[q][tid];
        flipped.w[q] = make_uint4(raw.w[q].x ^ m.x, raw.w[q].y ^ m.y, raw.w[q].z ^ m.z, raw.w[q].w ^ m.w);
      }
      unpack16(flipped, w);
      hadamard16_quarter(w);
    } else {
      unpack16(raw, w);
      uint32_t mask[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 m = sign_masks[q][tid];
        mask[4 * q] = m.x;
        mask[4 * q + 1] = m.y;
        mask[4 * q + 2] = m.z;
        mask[4 * q + 3] = m.w;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) w[i] = u2f(f2u(w[i]) ^ mask[i]);
      hadamard16_quarter(w);
    }
  };
  float amax = 0.0f;
  ScaleConsts sc{};

  auto lanes_in_round = [&](uint32_t r) { return (r == rounds - 1) ? tail : (uint32_t)kThreads; };

  // one block, already loaded; `live` = lanes of this round that hold a block (fewer than
  // 256 only in the last round of a ragged tensor)
  auto work = [&](uint32_t r, uint32_t live, const Raw &raw) {
    const int64_t base = (int64_t)r * kThreads;
    if (RHT) {
      // the sign word depends on the block's position in its row only; with the usual
      // shapes a lane meets the same position in every round and keeps its masks
      uint32_t B = (uint32_t)(base % nb_per_row) + B_lane;
      if (B >= nb_per_row) B -= nb_per_row;
      if (B != sign_B) {
        sign_B = B;
        uint32_t mask[4 * kMaskPieces];
        rht_sign_masks(rht_sign_word(rht_seed, B), mask);
#pragma unroll
        for (int q = 0; q < kMaskPieces; ++q)
          sign_masks[q][tid] = make_uint4(mask[4 * q], mask[4 * q + 1], mask[4 * q + 2], mask[4 * q + 3]);
      }
    }
    float v[16];
    values(raw, v);
    if (OUT == kOutAmax) {
#pragma unroll
      for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(v[i]));
      return;
    }
    // base is a multiple of 256 blocks, 1024 groups of four words, so a lane's own part of the counter
    // never carries out of the lower word.  Eight words at a time: 8192 x 8192 with the transform
    // takes 80.3 / 80.4 / 82.5 us with four / eight / sixteen, 1008 x 4096 without 7.5 / 7.5 / 7.9.
    const uint64_t q0 = (uint64_t)base * 4u;
    constexpr int kStep = 8;
    auto words = words_on_demand<kStep>([&](int q, uint32_t (&w)[kStep]) {
      sr_words_in_wave<kStep / 4>(sr_seed, (uint32_t)q0 + (4u * tid + kStep / 4 * q), (uint32_t)(q0 >> 32), w);
    });
    // words that are needed for one candidate alone, at the very end: drawn ahead, beside the candidates
    constexpr bool kAhead = ROUNDING != kRTN && !kTogether<ROUNDING, SELECT>;
    uint32_t u[kAhead ? 16 : 1];
    if constexpr (kAhead) sr_words_in_wave<4>(sr_seed, (uint32_t)q0 + 4u * tid, (uint32_t)(q0 >> 32), u);
    // the block once more, from memory (a lane without a block of its own holds a copy of
    // the round's last block, as fetch() gave it)
    auto again = [&](float (&w)[16], uint32_t (&uu)[16]) {
      Raw r2;
      load_block<XF32>(x + Raw::kPieces * (base + (tid < live ? tid : live - 1)), r2);
      values(r2, w);
      if constexpr (kAhead && !RHT) {
        // (there is room to keep them: 111 registers instead of 84, and the one wave in some hundreds that comes here
        // ends sooner, 1008 x 4096 7.7 -> 6.9 us; with the transform 123 instead of 98 cost 4 % of any size)
#pragma unroll
        for (int i = 0; i < 16; ++i) uu[i] = u[i];
      } else if constexpr (ROUNDING != kRTN) {
#pragma unroll
        for (int j = 0; j < 4; ++j) sr_words4(sr_seed, q0 + 4u * tid + j, &uu[4 * j]);
      }
    };
    BlockResult res;
    if constexpr (kAhead) res = quantize_block<ROUNDING, SELECT>(v, u, sc, tab, again);
    else res = quantize_block<ROUNDING, SELECT, (SELECT == kSel46 ? kNothing : kPairs)>(v, words, sc, tab, again);
    if (OUT == kOutCodes) {
      store_as<kNtCodes>(codes + base + tid, make_uint2(res.lo, res.hi));
      store_as<kNtCodes>(scales + base + tid, (uint8_t)res.scale);
      if (choice) store_as<kNtCodes>(choice + base + tid, (uint8_t)res.four);
    } else {
      float D0[8], D1[8];
      dequant8(res.lo, res.dec, D0);
      dequant8(res.hi, res.dec, D1);
      // lane l of a wave holds 16-byte pieces 2l and 2l+1 of the wave's output and
      // stores pieces l and 64+l; LDS operations of one wave execute in order, so the
      // reads below see the writes above without a barrier
      const uint32_t wave0 = tid & ~63u, lane = tid & 63u;
      uint4 *slot = xpose + 2 * wave0;
      slot[2 * lane] = make_uint4(pack_bf16x2(D0[0], D0[1]), pack_bf16x2(D0[2], D0[3]),
                                  pack_bf16x2(D0[4], D0[5]), pack_bf16x2(D0[6], D0[7]));
      slot[2 * lane + 1] = make_uint4(pack_bf16x2(D1[0], D1[1]), pack_bf16x2(D1[2], D1[3]),
                                      pack_bf16x2(D1[4], D1[5]), pack_bf16x2(D1[6], D1[7]));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      uint4 *ob = out_bf16 + 2 * (base + wave0);
      if (wave0 + (lane >> 1) < live) store_as<kNtBf16>(ob + lane, slot[lane]);
      if (wave0 + 32 + (lane >> 1) < live) store_as<kNtBf16>(ob + 64 + lane, slot[64 + lane]);
    }
  };

  // Loads run one round ahead of the arithmetic: while a wave works on one block the
  // 128-bit loads of its next block are already in flight (two register sets, used
  // alternately), so a round costs max(memory latency, arithmetic) instead of their sum.
  // The first round's loads also go out before the scale table is built.
  // In the fake-quant kernel lanes without a block still run (their results are not
  // stored), because they store pieces of their neighbours' blocks; elsewhere they skip
  // the round.
  // The loads are unconditional (a conditional load would have to be waited for right
  // where the two control paths join): a round past the workgroup's share re-reads round 0
  // (every workgroup ends with that, so the L2 serves it) and a lane past the end of a ragged
  // last round re-reads that round's last block; what they fetch is never used.
  uint32_t r, step, end;
  if (blockIdx.x < n_long) {
    r = blockIdx.x;
    step = n_long;
    end = n_long * rounds_long;
  } else {
    r = n_long * rounds_long + (blockIdx.x - n_long);
    step = gridDim.x - n_long;
    end = rounds;
  }
  // turn t of the deal above works on round t, or on the t-th from the end (kLastLevelBytes)
  auto place = [&](uint32_t t) { return OUT != kOutAmax && backwards ? rounds - 1u - t : t; };
  auto fetch = [&](uint32_t next, Raw &raw) {
    const uint32_t rr = place(next < end ? next : 0u);
    const uint32_t last = lanes_in_round(rr) - 1;
    const uint32_t lane = tid < last ? tid : last;
    const uint4 *xb = x + Raw::kPieces * ((int64_t)rr * kThreads);
    load_block<XF32>(xb + Raw::kPieces * lane, raw);
  };
  auto run = [&](uint32_t turn, const Raw &raw) {
    const uint32_t r = place(turn);
    const uint32_t live = lanes_in_round(r);
    if (OUT == kOutFake || tid < live) work(r, live, raw);
  };
  Raw a, b;
  fetch(r, a);
  if (OUT != kOutAmax) sc = build_scale_table(tab, *alpha_p);
  while (r < end) {
    fetch(r + step, b);
    run(r, a);
    r += step;
    if (r >= end) break;
    fetch(r + step, a);
    run(r, b);
    r += step;
  }
  if (OUT == kOutAmax) publish_amax(amax, amax_bits, fin, whole_launch());
}

// Tensor scale and rowwise codes of a small tensor in one launch: every workgroup reads the whole
// tensor for its maximum (it comes out of the L2 after the first), then its first four waves, one per SIMD,
// quantize its own 256 blocks, one per lane (with a block for each of the 1024 lanes four waves of a SIMD queue
// for its vector unit: us in a replayed graph, x in the memory-side cache, BF16 / fp32, 1024 and 256 blocks:
// 128 KiB 4.8 / 5.0 and 4.1 / 3.8, 256 KiB 5.6 / 6.0 and 5.0 / 4.7, 384 KiB 6.9 / 7.1 and 6.2 / 5.7; two kernels
// and the gap between them 7 to 8).  small_tensors.hpp says where that ends.
template <bool XF32, int SELECT>
__global__ __launch_bounds__(kSmallThreads) void k_scale_quantize_small(
    const uint4 *__restrict__ x, float *__restrict__ alpha_out, uint2 *__restrict__ codes,
    uint8_t *__restrict__ scales, uint8_t *__restrict__ choice, uint32_t nblocks, float fp8_max) {
  __shared__ ScaleTable tab;
  using Raw = RawBlock<XF32>;
  const bool mine = threadIdx.x < kSmallBlocks;
  const uint32_t k = blockIdx.x * kSmallBlocks + threadIdx.x;
  Raw raw;
  if (mine) load_block<XF32>(x + Raw::kPieces * (k < nblocks ? k : nblocks - 1), raw);
  const float alpha = small_tensor_alpha<XF32>(x, nblocks * Raw::kPieces, fp8_max);
  if (mine && k == 0) *alpha_out = alpha;
  const ScaleConsts sc = build_scale_table(tab, alpha);
  if (!mine || k >= nblocks) return;
  float v[16];
  const uint32_t u[16] = {};
  unpack16(raw, v);
  auto again = [&](float (&w)[16], uint32_t (&)[16]) { unpack16(raw, w); };
  const BlockResult res = quantize_block<kRTN, SELECT>(v, u, sc, tab, again);
  store_as<kNtCodes>(codes + k, make_uint2(res.lo, res.hi));
  store_as<kNtCodes>(scales + k, (uint8_t)res.scale);
  if (choice) store_as<kNtCodes>(choice + k, (uint8_t)res.four);
}

#if NVFP4_46_MAIN
// One lane per 8 elements: 4 code bytes + the block's scale -> 8 BF16.
__global__ __launch_bounds__(kThreads) void k_dequant_flat(const uint32_t *__restrict__ codes,
                                                           const uint8_t *__restrict__ scales,
                                                           const float *__restrict__ alpha_p,
                                                           uint4 *__restrict__ out, int64_t n8) {
  const float alpha = *alpha_p;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < n8; t += stride) {
    float dec = e4m3_decode(scales[t >> 1]) * alpha;
    float D[8];
    dequant8(codes[t], dec, D);
    store_as<kNtBf16>(out + t, make_uint4(pack_bf16x2(D[0], D[1]), pack_bf16x2(D[2], D[3]),
                                          pack_bf16x2(D[4], D[5]), pack_bf16x2(D[6], D[7])));
  }
}
#endif

// ------------------------------------------------ columnwise / both (tiled)

constexpr int kRowBlocksPerTileRow = TC / 16;          // 16-element row blocks across a tile row
constexpr int kRowBlocksPerTile = TR * TC / 16;
constexpr int kRowBlocksPerLane = kRowBlocksPerTile / kThreads;
constexpr int kColPairs = TC / 2;                      // pairs of adjacent columns
constexpr int kColBlockRows = TR / 16;                 // 16-row blocks down a tile column
constexpr int kPairUnits = kColPairs * kColBlockRows;  // (column pair, row block) units
constexpr int kPairUnitsPerLane = kPairUnits / kThreads;
constexpr int kColItems = TC * kColBlockRows;          // (column, row block) results per tile
constexpr int kColItemsPerLane = kColItems / kThreads;
constexpr int kPieces = TR * TC / 8;                   // 128-bit pieces of a BF16 tile
constexpr int kPiecesPerLane = kPieces / kThreads;
static_assert(TR % 16 == 0 && TC % 16 == 0, "tiles are made of whole blocks both ways");
static_assert(kRowBlocksPerTile % kThreads == 0 && kPairUnits % kThreads == 0 &&
              kColItems % kThreads == 0, "tile work must divide evenly over the workgroup");

struct TileCoord {
  int64_t r0, c0;
  bool valid;
};

NV_DEV TileCoord tile_of_workgroup(int64_t rows, int64_t cols, TileMap m, uint32_t block) {
  const uint32_t nt_r = (uint32_t)((rows + TR - 1) / TR), nt_c = (uint32_t)((cols + TC - 1) / TC);
  const uint32_t per = m.sx * m.sy, nsx = (nt_c + m.sx - 1) / m.sx;
  const uint32_t id = m.last ? m.last - block : block;
  const uint32_t xcd = id & 7u, slot = id >> 3;
  const uint32_t round = slot / per, within = slot - round * per;
  const uint32_t S = round * 8u + xcd;                      // super-tile, row-major
  const uint32_t sy = S / nsx, sx = S - sy * nsx;
  const uint32_t wy = within / m.sx, wx = within - wy * m.sx;
  const uint32_t tr = sy * m.sy + wy, tc = sx * m.sx + wx;
  return TileCoord{(int64_t)tr * TR, (int64_t)tc * TC, tc < nt_c && tr < nt_r};
}

// What a workgroup of k_tile keeps in LDS.
template <bool XF32, int ROUNDING, int SELECT, bool RHT, bool WANT_ROW, int OUT>
struct TileLds {
  // Only columnwise codes wanted: nothing needs the tile in LDS -- a lane reads its two columns
  // straight from memory, a row at a time (a wave's load covers 256 contiguous bytes of a row).
  static constexpr bool kDirect = !WANT_ROW && OUT == kOutCodes;
  // The random words of the tile, one Philox call per four neighbouring elements of a row, as the
  // generator hands them out.  A lane of phase 2 owns two of the four columns, so without this
  // place every call was made twice and its other half dropped, and the words of both columns sat in
  // registers (224 of them, two waves per SIMD).  Columnwise Hadamard + SR on 8192 x 8192:
  // 138 -> 110 us with its tensor scale, both orientations with SR 200 -> 166.
  // Fake-quant of fp32 keeps its tile in LDS as well, 32 KiB that with 32 KiB of words leave two
  // workgroups per compute unit.  That pays where registers allow no third one anyway: the squared-error
  // rule, and with the transform the other two that compare errors (columnwise, 8192 x 8192, words from
  // LDS / drawn by their lane: 4/6 115 / 120 us, with the transform 123 / 131; by absolute error with the
  // transform 121 / 134, without 113 / 101; always 6 96 / 86, with the transform 102 / 90; absolute error on
  // nearest-rounded candidates with the transform 113 / 104).  Elsewhere the lane draws the words of
  // its two columns itself, half of every call for nothing.
  static constexpr bool kTwoWavesAnyway =
      SELECT == kSel46 || (RHT && ROUNDING == kSR && (SELECT == kSel46Mae || SELECT == kSel46AbsMax));
  static constexpr bool kWords = ROUNDING != kRTN && (!XF32 || OUT != kOutFake || kTwoWavesAnyway);
  static constexpr bool kDrawn = ROUNDING != kRTN && !kWords;
  // the tile, row-major: one 32-bit word (two BF16) or two (two fp32) per pair of columns
  static constexpr int kXW = XF32 ? 2 : 1;

  typedef uint32_t Tile[kDirect ? 4 : TR * TC / 2 * kXW];
  typedef uint4 Words[kWords ? TR * TC / 4 : 1];                 // [TR][TC / 4]
  // columnwise results wait here until a whole column segment can leave at once: [TC][TR/16]
  typedef uint2 Codes[OUT == kOutCodes ? kColItems : 1];
  typedef uint8_t Bytes[OUT == kOutCodes ? kColItems : 1];
  // (references to arrays of their own: the compiler then knows that they do not overlap)
  ScaleTable &tab;
  Tile &tile;
  Words &words;
  Codes &stage_codes;
  Bytes &stage_scale, &stage_choice;
};

template <bool XF32, int ROUNDING, int SELECT, bool RHT, bool WANT_ROW, int OUT>
NV_DEV void quantize_tile(
    TileLds<XF32, ROUNDING, SELECT, RHT, WANT_ROW, OUT> lds, const void *__restrict__ x_any,
    float alpha, uint8_t *__restrict__ codes_row, uint8_t *__restrict__ scales_row,
    uint8_t *__restrict__ choice_row, uint8_t *__restrict__ codes_col,
    uint8_t *__restrict__ scales_col, uint8_t *__restrict__ choice_col,
    uint16_t *__restrict__ out_bf16, int64_t rows, int64_t cols,
    uint64_t sr_seed, uint64_t rht_seed, TileMap map, uint32_t block) {
  typedef TileLds<XF32, ROUNDING, SELECT, RHT, WANT_ROW, OUT> Lds;
  constexpr bool kDirect = Lds::kDirect, kWords = Lds::kWords, kDrawn = Lds::kDrawn;
  constexpr int kXW = Lds::kXW;
  using Raw = RawBlock<XF32>;
  ScaleTable &tab = lds.tab;
  auto &tile = lds.tile;
  auto &words = lds.words;
  auto &stage_codes = lds.stage_codes;
  auto &stage_scale = lds.stage_scale;
  auto &stage_choice = lds.stage_choice;

  const TileCoord tcd = tile_of_workgroup(rows, cols, map, block);
  if (!tcd.valid) return;  // uniform over the workgroup
  const int64_t r0 = tcd.r0, c0 = tcd.c0;
  const int t = threadIdx.x;

  if (kWords) {
    // (cols is a multiple of 8, so four columns are in or out together and share a call)
    auto draw_all = [&](auto &&draw4) {
#pragma unroll 2
      for (int j = 0; j < TR * TC / 4 / kThreads; ++j) {
        const int idx = t + j * kThreads;
        const int64_t gr = r0 + idx / (TC / 4), gc = c0 + idx % (TC / 4) * 4;
        if (gr < rows && gc < cols) {
          uint32_t w[4];
          draw4(((uint64_t)gr * (uint64_t)cols + (uint64_t)gc) >> 2, w);
          words[idx] = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    };
    if (((uint64_t)rows * (uint64_t)cols >> 34) == 0)       // the upper counter word is 0 throughout
      draw_all([&](uint64_t q, uint32_t (&w)[4]) { sr_words_in_wave<1>(sr_seed, (uint32_t)q, 0u, w); });
    else
      draw_all([&](uint64_t q, uint32_t (&w)[4]) { sr_words4(sr_seed, q, w); });
  }   // (the barrier at the end of the scale table comes before the first use)

  // ---- phase 1: global -> LDS (and the rowwise outputs on the way); the loads go out
  // before the scale table is built
  if (!kDirect) {
    constexpr int kElemsPerPiece = XF32 ? 4 : 8, kPiecesPerEight = 8 / kElemsPerPiece;
    Raw w[kRowBlocksPerLane];
#pragma unroll
    for (int j = 0; j < kRowBlocksPerLane; ++j) {
      const int unit = t + j * kThreads;
      const int row = unit / kRowBlocksPerTileRow, rbk = unit % kRowBlocksPerTileRow;
      const int64_t gr = r0 + row, gc = c0 + rbk * 16;
      // (gr * cols + gc) elements into x, counted in 128-bit pieces
      const uint4 *src = static_cast<const uint4 *>(x_any) + (gr * cols + gc) / kElemsPerPiece;
      // (cols is a multiple of 8: the pieces of eight columns are in the tensor together, or outside, and then zeros)
#pragma unroll
      for (int q = 0; q < Raw::kPieces; q += kPiecesPerEight) {
#pragma unroll
        for (int i = q; i < q + kPiecesPerEight; ++i) w[j].w[i] = make_uint4(0, 0, 0, 0);
        if (gr < rows && gc + q * kElemsPerPiece < cols) {
#pragma unroll
          for (int i = q; i < q + kPiecesPerEight; ++i) w[j].w[i] = src[i];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kRowBlocksPerLane; ++j) {
      const int unit = t + j * kThreads;
      uint4 *dst = reinterpret_cast<uint4 *>(tile) + unit * Raw::kPieces;
#pragma unroll
      for (int q = 0; q < Raw::kPieces; ++q) dst[q] = w[j].w[q];
    }
  }
  const ScaleConsts sc = build_scale_table(tab, alpha);     // ends with a barrier

  if (WANT_ROW) {
    // the lane's own row blocks, taken back from LDS one at a time (keeps the register
    // footprint of the quantizer to a single block)
    const int64_t nb_per_row = cols / 16;
    const int blocks = cols - c0 < TC ? (int)(cols - c0) / 16 : kRowBlocksPerTileRow;
#pragma unroll 1
    for (int j = 0; j < kRowBlocksPerLane; ++j) {
      const int unit = t + j * kThreads;
      const int row = unit / kRowBlocksPerTileRow, own = unit % kRowBlocksPerTileRow;
      const int rbk = own < blocks ? own : blocks - 1;      // outside the tensor: the last block again, as in phase 2
      const int64_t gr = r0 + row, gc = c0 + rbk * 16;
      if (gr < rows) {
        float v[16];
        const int64_t k = gr * nb_per_row + (gc >> 4);
        // the lane's block out of the tile, and its random words (WANT_ROW is for codes: words are in LDS)
        auto block = [&](float (&w)[16]) {
          const uint4 *at = reinterpret_cast<const uint4 *>(tile) + (row * kRowBlocksPerTileRow + rbk) * Raw::kPieces;
          Raw mine;
#pragma unroll
          for (int q = 0; q < Raw::kPieces; ++q) mine.w[q] = at[q];
          unpack16(mine, w);
        };
        constexpr int kStep = 16;
        auto some = [&](int s, uint32_t (&w)[kStep]) {
#pragma unroll
          for (int q = 0; q < kStep / 4; ++q) {
            const uint4 w4 = words[kWords ? row * (TC / 4) + rbk * 4 + kStep / 4 * s + q : 0];
            w[4 * q] = w4.x;
            w[4 * q + 1] = w4.y;
            w[4 * q + 2] = w4.z;
            w[4 * q + 3] = w4.w;
          }
        };
        auto take = [&](float (&w)[16], uint32_t (&uu)[16]) {
          block(w);
          if (kWords) {
#pragma unroll
            for (int s = 0; s < 16 / kStep; ++s) {
              uint32_t got[kStep];
              some(s, got);
#pragma unroll
              for (int i = 0; i < kStep; ++i) uu[kStep * s + i] = got[i];
            }
          }
        };
        block(v);
        BlockResult r = quantize_block<ROUNDING, SELECT>(v, words_on_demand<kStep>(some), sc, tab, take);
        if (own == rbk) {
          reinterpret_cast<uint2 *>(codes_row)[k] = make_uint2(r.lo, r.hi);
          scales_row[k] = (uint8_t)r.scale;
          if (choice_row) choice_row[k] = (uint8_t)r.four;
        }
      }
    }
  }

  // ---- phase 2: every lane takes two adjacent columns x 16 rows.  A (column pair, row
  // block) unit is read and, for the fake-quant output, rewritten in place by its owner
  // lane only, so no barrier is needed inside this phase.
  static_assert(kColPairs == 64, "a wave's lanes are the column pairs of one row block");
  const int pairs = cols - c0 < TC ? (int)(cols - c0) / 2 : kColPairs;
#pragma unroll 1
  for (int j = 0; j < kPairUnitsPerLane; ++j) {
    // (the row block is the wave's: what follows from it stays on the scalar unit)
    const int own = t % kColPairs, rb = __builtin_amdgcn_readfirstlane(t / kColPairs) + j * (kThreads / kColPairs);
    const int64_t gr = r0 + rb * 16;              // first row of the block
    if (gr >= rows) continue;
    // A lane whose pair is outside the tensor (cols is even, so it is in or out together) does the last one inside over again
    // and leaves it in its own place, which nobody reads: a wave of 8 lanes, a tile's last 16 columns, takes nearly twice
    // as long as one of 12 or of 64 (BF16, codes with the transform and SR, us: 64 x 16 9.2, 64 x 24 6.1; the lanes all
    // at work 64 x 16 6.1).
    const int cp = own < pairs ? own : pairs - 1;
    const int64_t gc = c0 + 2 * cp;               // even column of the pair
    float va[16], vb[16];
    // the lane's two column blocks (transformed) out of the tile or memory
    auto take = [&](float (&wa)[16], float (&wb)[16]) {
      const uint32_t sw = RHT ? rht_sign_word_of_wave(rht_seed, (uint32_t)(gr >> 4), (uint32_t)(gr >> 36)) : 0u;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int64_t row = ((gr + i) * cols + c0) >> 1;   // pairs before the tile's first in row i of the block
        const uint32_t flip = 0u - ((sw >> i) & 1u);       // the transform's sign: one per row
        if constexpr (XF32) {
          uint2 pair = kDirect ? (static_cast<const uint2 *>(x_any) + row)[cp]
                               : reinterpret_cast<const uint2 *>(tile)[(rb * 16 + i) * kColPairs + cp];
          if (RHT) {
            pair.x ^= flip & 0x80000000u;
            pair.y ^= flip & 0x80000000u;
          }
          wa[i] = u2f(pair.x);
          wb[i] = u2f(pair.y);
        } else {
          uint32_t pair = kDirect ? (static_cast<const uint32_t *>(x_any) + row)[cp]
                                  : tile[(rb * 16 + i) * kColPairs + cp];
          if (RHT) pair ^= flip & 0x80008000u;
          wa[i] = bf16_lo(pair);
          wb[i] = bf16_hi(pair);
        }
      }
      if (RHT) {
        hadamard16_quarter(wa);
        hadamard16_quarter(wb);
      }
    };
    auto word_at = [&](int i, int column) {                             // row i, column 0 or 1 of the pair
      return reinterpret_cast<const uint32_t *>(words)[kWords ? (rb * 16 + i) * TC + 2 * cp + column : 0];
    };
    auto random_words = [&](int column, uint32_t (&uu)[16]) {
      if (kWords) {
#pragma unroll
        for (int i = 0; i < 16; ++i) uu[i] = word_at(i, column);
      }
    };
    auto draw = [&](uint32_t (&uua)[16], uint32_t (&uub)[16]) {         // both columns of the pair
      // element (row, col) has flat index g = row*cols + col; gc is even and cols a multiple of 4,
      // so the pair's words come from one call
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint64_t g = (uint64_t)(gr + i) * (uint64_t)cols + (uint64_t)gc;
        uint32_t w[4];
        sr_words4(sr_seed, g >> 2, w);
        uua[i] = (g & 2u) ? w[2] : w[0];
        uub[i] = (g & 2u) ? w[3] : w[1];
      }
    };
    take(va, vb);
    auto first = [&](float (&w)[16], uint32_t (&uu)[16]) {
      float other[16];
      uint32_t other_u[16];
      take(w, other);
      if (kDrawn) draw(uu, other_u);
      random_words(0, uu);
    };
    auto second = [&](float (&w)[16], uint32_t (&uu)[16]) {
      float other[16];
      uint32_t other_u[16];
      take(other, w);
      if (kDrawn) draw(other_u, uu);
      random_words(1, uu);
    };
    BlockResult ra, rbk;
    if constexpr (kDrawn) {
      uint32_t ua[16], ub[16];
      draw(ua, ub);
      ra = quantize_block<ROUNDING, SELECT, kSingles | kPairs>(va, ua, sc, tab, first);
      rbk = quantize_block<ROUNDING, SELECT, kSingles | kPairs>(vb, ub, sc, tab, second);
    } else {
      constexpr int kStep = 16;
      auto words_of = [&](int column) {
        return words_on_demand<kStep>([&, column](int q, uint32_t (&w)[kStep]) {
#pragma unroll
          for (int i = 0; i < kStep; ++i) w[i] = word_at(kStep * q + i, column);
        });
      };
      ra = quantize_block<ROUNDING, SELECT>(va, words_of(0), sc, tab, first);
      rbk = quantize_block<ROUNDING, SELECT>(vb, words_of(1), sc, tab, second);
    }
    if (OUT == kOutCodes) {
      const int ia = (2 * own) * kColBlockRows + rb, ib = ia + kColBlockRows;
      stage_codes[ia] = make_uint2(ra.lo, ra.hi);
      stage_codes[ib] = make_uint2(rbk.lo, rbk.hi);
      stage_scale[ia] = (uint8_t)ra.scale;
      stage_scale[ib] = (uint8_t)rbk.scale;
      stage_choice[ia] = (uint8_t)ra.four;
      stage_choice[ib] = (uint8_t)rbk.four;
    } else {
      float Da[16], Db[16];
      {
        float h[8];
        dequant8(ra.lo, ra.dec, h);
#pragma unroll
        for (int i = 0; i < 8; ++i) Da[i] = h[i];
        dequant8(ra.hi, ra.dec, h);
#pragma unroll
        for (int i = 0; i < 8; ++i) Da[8 + i] = h[i];
        dequant8(rbk.lo, rbk.dec, h);
#pragma unroll
        for (int i = 0; i < 8; ++i) Db[i] = h[i];
        dequant8(rbk.hi, rbk.dec, h);
#pragma unroll
        for (int i = 0; i < 8; ++i) Db[8 + i] = h[i];
      }
      // the BF16 pair takes the first word of the pair's slot
#pragma unroll
      for (int i = 0; i < 16; ++i)
        tile[((rb * 16 + i) * kColPairs + own) * kXW] = pack_bf16x2(Da[i], Db[i]);
    }
  }
  __syncthreads();

  // ---- phase 3: LDS -> global, contiguous runs
  if (OUT == kOutCodes) {
    const int64_t col_codes = rows / 2, col_scales = rows / 16;
#pragma unroll
    for (int j = 0; j < kColItemsPerLane; ++j) {
      const int it = t + j * kThreads;
      const int cl = it / kColBlockRows, rb = it % kColBlockRows;
      const int64_t gc = c0 + cl, gr = r0 + rb * 16;
      if (gc < cols && gr < rows) {
        *reinterpret_cast<uint2 *>(codes_col + gc * col_codes + (gr >> 1)) = stage_codes[it];
        scales_col[gc * col_scales + (gr >> 4)] = stage_scale[it];
        if (choice_col) choice_col[gc * col_scales + (gr >> 4)] = stage_choice[it];
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < kPiecesPerLane; ++j) {
      const int idx = t + j * kThreads;
      const int row = idx / (TC / 8), seg = idx % (TC / 8);
      const int64_t gr = r0 + row, gc = c0 + seg * 8;
      if (gr < rows && gc < cols) {
        // piece idx = the four column pairs 4*idx .. 4*idx+3 of the tile
        const uint4 piece = XF32 ? make_uint4(tile[8 * idx], tile[8 * idx + 2], tile[8 * idx + 4],
                                              tile[8 * idx + 6])
                                 : reinterpret_cast<const uint4 *>(tile)[idx];
        store_as<kNtBf16>(reinterpret_cast<uint4 *>(out_bf16 + gr * cols + gc), piece);
      }
    }
  }
}

template <bool XF32, int ROUNDING, int SELECT, bool RHT, bool WANT_ROW, int OUT>
__global__ __launch_bounds__(kThreads) void k_tile(
    const void *__restrict__ x, const float *__restrict__ alpha, uint8_t *__restrict__ codes_row,
    uint8_t *__restrict__ scales_row, uint8_t *__restrict__ choice_row, uint8_t *__restrict__ codes_col,
    uint8_t *__restrict__ scales_col, uint8_t *__restrict__ choice_col, uint16_t *__restrict__ out_bf16, int64_t rows,
    int64_t cols, uint64_t sr_seed, uint64_t rht_seed, TileMap map) {
  typedef TileLds<XF32, ROUNDING, SELECT, RHT, WANT_ROW, OUT> Lds;
  __shared__ ScaleTable tab;
  __shared__ __align__(16) typename Lds::Tile tile;
  __shared__ typename Lds::Words words;
  __shared__ typename Lds::Codes stage_codes;
  __shared__ typename Lds::Bytes stage_scale, stage_choice;
  quantize_tile(Lds{tab, tile, words, stage_codes, stage_scale, stage_choice}, x, *alpha, codes_row, scales_row, choice_row, codes_col, scales_col, choice_col, out_bf16, rows, cols,
                sr_seed, rht_seed, map, blockIdx.x);
}

// Both operands of a weight gradient in one launch: BF16 tensors of the same rows, columnwise with the transform, the
// first (the gradient, its tiles the first `blocks_a` workgroups) rounded stochastically, the other to nearest.
struct TilePair {
  const void *x[2];
  const float *alpha[2];
  uint8_t *codes[2], *scales[2];
  int64_t cols[2];
  TileMap map[2];
};
template <int SELECT>
__global__ __launch_bounds__(kThreads) void k_tile_pair(TilePair p, int64_t rows, uint64_t sr_seed, uint64_t rht_seed,
                                                        uint32_t blocks_a) {
  typedef TileLds<false, kSR, SELECT, true, false, kOutCodes> LdsA;
  typedef TileLds<false, kRTN, SELECT, true, false, kOutCodes> LdsB;
  // (the second kind has no words)
  __shared__ ScaleTable tab;
  __shared__ typename LdsA::Tile tile;
  __shared__ typename LdsA::Words words;
  __shared__ typename LdsA::Codes stage_codes;
  __shared__ typename LdsA::Bytes stage_scale, stage_choice;
  if (blockIdx.x < blocks_a)
    quantize_tile(LdsA{tab, tile, words, stage_codes, stage_scale, stage_choice}, p.x[0], *p.alpha[0], nullptr, nullptr, nullptr, p.codes[0], p.scales[0],
                  nullptr, nullptr, rows, p.cols[0], sr_seed, rht_seed, p.map[0], blockIdx.x);
  else
    quantize_tile(LdsB{tab, tile, reinterpret_cast<typename LdsB::Words &>(words), stage_codes, stage_scale, stage_choice}, p.x[1], *p.alpha[1], nullptr, nullptr, nullptr, p.codes[1], p.scales[1],
                  nullptr, nullptr, rows, p.cols[1], sr_seed, rht_seed, p.map[1], blockIdx.x - blocks_a);
}

// Columnwise codes/scales -> row-major BF16, through an LDS tile.  TILE2D: the scales are
// per 16x16 tile of the matrix, stored [cols/16][rows/16].
template <bool TILE2D>
__global__ __launch_bounds__(kThreads) void k_dequant_col(const uint8_t *__restrict__ codes,
                                                          const uint8_t *__restrict__ scales,
                                                          const float *__restrict__ alpha_p,
                                                          uint16_t *__restrict__ out, int64_t rows,
                                                          int64_t cols, TileMap map) {
  __shared__ __align__(16) uint16_t tile16[TR * TC];
  const TileCoord tcd = tile_of_workgroup(rows, cols, map, blockIdx.x);
  if (!tcd.valid) return;
  const int64_t r0 = tcd.r0, c0 = tcd.c0;
  const int t = threadIdx.x;
  const float alpha = *alpha_p;
  const int64_t col_codes = rows / 2, col_scales = rows / 16;
#pragma unroll 1
  for (int j = 0; j < kColItemsPerLane; ++j) {
    const int it = t + j * kThreads;
    const int cl = it / kColBlockRows, rb = it % kColBlockRows;
    const int64_t gc = c0 + cl, gr = r0 + rb * 16;
    if (gc < cols && gr < rows) {
      const uint2 c = *reinterpret_cast<const uint2 *>(codes + gc * col_codes + (gr >> 1));
      const float dec =
          e4m3_decode(scales[(TILE2D ? (gc >> 4) : gc) * col_scales + (gr >> 4)]) * alpha;
      float D[8];
      dequant8(c.x, dec, D);
#pragma unroll
      for (int i = 0; i < 8; ++i) tile16[(rb * 16 + i) * TC + cl] = (uint16_t)pack_bf16x2(D[i], 0.0f);
      dequant8(c.y, dec, D);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        tile16[(rb * 16 + 8 + i) * TC + cl] = (uint16_t)pack_bf16x2(D[i], 0.0f);
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPiecesPerLane; ++j) {
    const int idx = t + j * kThreads;
    const int row = idx / (TC / 8), seg = idx % (TC / 8);
    const int64_t gr = r0 + row, gc = c0 + seg * 8;
    if (gr < rows && gc < cols)
      store_as<kNtBf16>(reinterpret_cast<uint4 *>(out + gr * cols + gc),
                        reinterpret_cast<const uint4 *>(tile16)[idx]);
  }
}

// ------------------------------------------------------- 2D (16x16) blocks

// One scale per 16x16 tile (the weight-matrix variant named in Section 4.1).  Sixteen
// adjacent lanes own the sixteen rows of a tile (one row block each); the tile's
// maximum, and the two candidates' errors, are combined across those lanes with XOR
// shuffles.  A tile's error is defined as a row's sixteen terms in the usual fixed order,
// then the sixteen row sums in the same order (strides 4, 2, 1 within each half, then the
// two halves), which is the order of the shuffles 4, 2, 1, 8; for the squared-error rule the
// decision is first tried on cheap row estimates summed the same way and falls back to the
// defined errors when the two sums are too close to call.
// Lane -> (tile, row): lanes 0-15 are the rows of one tile, the next sixteen lanes the
// tile to its right, so four lanes 16 apart read 128 contiguous bytes of one row.

// Sixteen adjacent lanes each hold one row of a 16x16 matrix of 4-bit codes (lo = columns
// 0-7, hi = columns 8-15, column j in bits 4j..4j+3); on return lane j of the sixteen holds
// column j packed the same way (row i in bits 4i..4i+3).  The usual recursive transpose:
// swap the off-diagonal 8x8 blocks between lanes 8 apart, then 4x4 blocks between lanes 4
// apart inside every 8x8 block, and so on down to single codes.
// 8-byte pieces per row of the LDS staging of transposed codes in k_block2d: 16 + 2, so that
// sixteen lanes writing one piece each to sixteen rows fall in different banks
constexpr uint32_t kColStagePitch = 18;

NV_DEV void transpose_codes16(uint32_t &lo, uint32_t &hi) {
  const uint32_t lane = threadIdx.x;
  {
    const bool upper = lane & 8u;
    const uint32_t got = __shfl_xor(upper ? lo : hi, 8, 64);
    if (upper) lo = got; else hi = got;
  }
  auto stage = [&](uint32_t &w, uint32_t bit, uint32_t keep_low, int shift) {
    // keep_low masks the groups a lane with (lane & bit) == 0 keeps in place
    const bool upper = lane & bit;
    const uint32_t give = upper ? (w & keep_low) : ((w >> shift) & keep_low);
    const uint32_t got = __shfl_xor(give, (int)bit, 64);
    w = upper ? ((w & ~keep_low) | got) : ((w & keep_low) | (got << shift));
  };
  stage(lo, 4u, 0x0000ffffu, 16);
  stage(hi, 4u, 0x0000ffffu, 16);
  stage(lo, 2u, 0x00ff00ffu, 8);
  stage(hi, 2u, 0x00ff00ffu, 8);
  stage(lo, 1u, 0x0f0f0f0fu, 4);
  stage(hi, 1u, 0x0f0f0f0fu, 4);
}

// UNIT_ROWS: tile rows of a unit (4, 8 or 16; as a number of the launch they cost 1 to 2 %), or 0 for one packing.
template <bool XF32, int ROUNDING, int SELECT, int OUT, int UNIT_ROWS>
__global__ __launch_bounds__(kThreads) void k_block2d(
    const void *__restrict__ x_any, const float *__restrict__ alpha_p, uint8_t *__restrict__ codes,
    uint8_t *__restrict__ scales, uint8_t *__restrict__ choice, uint8_t *__restrict__ codes_col,
    uint8_t *__restrict__ scales_col, uint8_t *__restrict__ choice_col,
    uint16_t *__restrict__ out_bf16, int64_t rows, int64_t cols, uint64_t sr_seed, uint32_t backwards) {
  __shared__ ScaleTable tab;
  const ScaleConsts sc = build_scale_table(tab, *alpha_p);
  const uint32_t tid = threadIdx.x, r_in_tile = tid & 15u, grp = tid >> 4;
  // rows, cols <= 2^31 and rows * cols <= 2^40 (checked by the entry point): tile coordinates
  // and tile numbers fit 32 bits
  const uint32_t ncb = (uint32_t)(cols / 16), nrb = (uint32_t)(rows / 16);
  const uint64_t n_tiles = (uint64_t)nrb * ncb;
  constexpr int kCandRounding = ROUNDING == kSRAfterRtnSelect ? kRTN : ROUNDING;
  constexpr int kErr = SELECT == kSel46     ? kErrMseEstimate
                       : SELECT == kSel46Mae ? kErrMae
                       : SELECT == kSel46AbsMax ? kErrAbsMax : kErrNone;
  // Two ways to hand tiles to workgroups (the launcher's grid matches):
  //  * one packing: workgroup id -> sixteen consecutive tiles along a row of tiles, one per group
  //    of sixteen lanes; a row of x is read, and its codes written, 128 contiguous bytes at a
  //    time by the workgroup;
  //  * with the packing for the transposed matrix as well, whose codes are 8 bytes per lane 4 KiB
  //    and more apart (stored like that they cost 1.9x their bytes in HBM writes and 35 us on
  //    8192 x 8192): workgroup id -> a unit of 4, 8 or 16 tile rows (tile_unit_rows()) x 4 tile columns, taken in
  //    steps of 4 x 4 tiles (wave w: tile row 4 * step + w; its four groups: the tile columns).
  //    The unit's transposed codes (64 rows of the transposed matrix x 4 to 16 pieces of 8 bytes) are
  //    gathered in LDS and leave as runs of 32 to 128 bytes; row codes leave as 32 contiguous bytes
  //    per store instruction, and id -> unit keeps the four units that share the 128-byte
  //    lines of row codes on one die's L2 (ids 8 apart).
  constexpr bool by_units = UNIT_ROWS > 0;
  static_assert(!by_units || OUT == kOutCodes, "units are for the transposed packing");
  __shared__ uint2 col_stage[by_units ? 64 * kColStagePitch : 1];
  const uint32_t wave = tid >> 6, g4 = grp & 3u;
  const uint32_t ncq = (ncb + 3u) / 4u;
  constexpr uint32_t unit_rows = by_units ? UNIT_ROWS : 4;
  const uint32_t n_units = ((nrb + unit_rows - 1u) / unit_rows) * ncq;
  const uint32_t n_ids = by_units ? ((n_units + 31u) / 32u) * 32u : (uint32_t)((n_tiles + 15u) / 16u);
  constexpr uint32_t n_steps = unit_rows / 4u;
  auto tile_body = [&](uint32_t tr, uint32_t tc, uint32_t trl) {
    const uint64_t row = (uint64_t)tr * 16 + r_in_tile;
    const uint64_t first = row * (uint64_t)cols + tc * 16u;  // flat index of the lane's first element
    const uint64_t T = (uint64_t)tr * ncb + tc;
    RawBlock<XF32> raw;
    load_block<XF32>(static_cast<const uint4 *>(x_any) + first / (XF32 ? 4 : 8), raw);
    float v[16];
    uint32_t u[16];
    unpack16(raw, v);
    if (ROUNDING != kRTN) {
#pragma unroll
      for (int j = 0; j < 4; ++j) sr_words4(sr_seed, (uint64_t)(first >> 2) + j, &u[4 * j]);
    }
    float b = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) b = fmaxf(fmaxf(b, fabsf(v[i])), fabsf(v[i + 1]));
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) b = fmaxf(b, __shfl_xor(b, m, 64));

    // Eq. (2) for the tile, as for 1x16 blocks (the same for all sixteen lanes of the tile)
    uint32_t S6, S4;
    block_scales(b, sc, S6, S4);
    BlockResult r6{}, r4{};
    float E6 = 0.0f, E4 = 0.0f, enc6 = 0.0f, enc4 = 0.0f;
    if (SELECT != kSelForce4) {
      r6.scale = S6;
      const float4 t = tab.e[r6.scale];
      r6.dec = t.x;
      enc6 = t.y;
      if (!(ROUNDING == kSRAfterRtnSelect && SELECT == kSelForce6))
        E6 = candidate<kCandRounding, kErr>(v, u, t.x, t.y, r6.lo, r6.hi);
    }
    if (SELECT != kSelForce6) {
      r4.scale = S4;
      r4.four = 1u;
      const float4 t = tab.e[r4.scale];
      r4.dec = t.x;
      enc4 = t.y;
      if (!(ROUNDING == kSRAfterRtnSelect && SELECT == kSelForce4))
        E4 = candidate<kCandRounding, kErr>(v, u, t.x, t.y, r4.lo, r4.hi);
    }
    // the sixteen row values -> the tile's, in the fixed order; every lane ends with the same sum
    auto over_tile = [&](float &e6, float &e4) {
      constexpr int order[4] = {4, 2, 1, 8};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float o6 = __shfl_xor(e6, order[s], 64), o4 = __shfl_xor(e4, order[s], 64);
        e6 = SELECT == kSel46AbsMax ? fmaxf(e6, o6) : e6 + o6;
        e4 = SELECT == kSel46AbsMax ? fmaxf(e4, o4) : e4 + o4;
      }
    };
    bool four = SELECT == kSelForce4;
    if (SELECT == kSel46Mae || SELECT == kSel46AbsMax) {
      over_tile(E6, E4);      // evaluated as defined
      four = E4 < E6;
    } else if (SELECT == kSel46) {
      // E6, E4 are row estimates (see decide_from_estimates).  Outside the margin of
      // tile_decision_tolerance() the summed estimates order the defined errors; inside it
      // the defined errors are evaluated.  All sixteen lanes hold the same sums and take the
      // same path.
      over_tile(E6, E4);
      const float tol = tile_decision_tolerance(r6.dec, E6, r4.dec, E4);
      const float diff = E4 - E6;
      four = diff < 0.0f;
      if (!(fabsf(diff) > tol)) {
        float e6 = exact_error(v, r6.lo, r6.hi, r6.dec), e4 = exact_error(v, r4.lo, r4.hi, r4.dec);
        over_tile(e6, e4);
        four = e4 < e6;
      }
    }
    BlockResult res = four ? r4 : r6;
    if (ROUNDING == kSRAfterRtnSelect)
      (void)candidate<kSR, kErrNone>(v, u, res.dec, four ? enc4 : enc6, res.lo, res.hi);
    if (OUT == kOutCodes) {
      if (codes) {
        *reinterpret_cast<uint2 *>(codes + first / 2) = make_uint2(res.lo, res.hi);
        if (r_in_tile == 0) {
          scales[T] = (uint8_t)res.scale;
          if (choice) choice[T] = (uint8_t)res.four;
        }
      }
      if (by_units) {
        // the same tile for the transposed matrix: column (tc*16 + lane) of x is its row
        uint32_t lo = res.lo, hi = res.hi;
        transpose_codes16(lo, hi);
        col_stage[(g4 * 16u + r_in_tile) * kColStagePitch + trl] = make_uint2(lo, hi);
        if (r_in_tile == 0) {
          const uint64_t Tt = (uint64_t)tc * nrb + tr;
          scales_col[Tt] = (uint8_t)res.scale;
          if (choice_col) choice_col[Tt] = (uint8_t)res.four;
        }
      }
    } else {
      float D0[8], D1[8];
      dequant8(res.lo, res.dec, D0);
      dequant8(res.hi, res.dec, D1);
      uint4 *dst = reinterpret_cast<uint4 *>(out_bf16 + first);
      dst[0] = make_uint4(pack_bf16x2(D0[0], D0[1]), pack_bf16x2(D0[2], D0[3]),
                          pack_bf16x2(D0[4], D0[5]), pack_bf16x2(D0[6], D0[7]));
      dst[1] = make_uint4(pack_bf16x2(D1[0], D1[1]), pack_bf16x2(D1[2], D1[3]),
                          pack_bf16x2(D1[4], D1[5]), pack_bf16x2(D1[6], D1[7]));
    }
  };
  for (uint32_t turn = blockIdx.x; turn < n_ids; turn += gridDim.x) {
    const uint32_t id = backwards ? n_ids - 1u - turn : turn;
    // by units: the same for the whole workgroup
    const uint32_t slot = id >> 3, unit = (((slot >> 2) << 3) + (id & 7u)) * 4u + (slot & 3u);
    const uint32_t mr = unit / ncq, cq = unit - mr * ncq;
#pragma unroll 1
    for (uint32_t step = 0; step < n_steps; ++step) {
      uint32_t tr, tc, trl = step * 4u + wave;
      bool live;
      if (by_units) {
        tr = mr * unit_rows + trl;
        tc = cq * 4u + g4;
        live = unit < n_units && tr < nrb && tc < ncb;
      } else {
        const uint32_t t = id * 16u + grp;
        tr = t / ncb;
        tc = t - tr * ncb;
        live = (uint64_t)id * 16u + grp < n_tiles;
      }
      if (live) tile_body(tr, tc, trl);
      if (by_units && step == n_steps - 1u) {
        // the unit's 64 rows of the transposed matrix, 4 to 16 pieces of 8 bytes each, which as many
        // consecutive lanes store
        __syncthreads();
        if (unit < n_units) {
#pragma unroll 1
          for (uint32_t j = 0; j < n_steps; ++j) {
            const uint32_t piece = tid + j * kThreads, line = piece / unit_rows, k = piece % unit_rows;
            const uint64_t col = ((uint64_t)cq * 4 + (line >> 4)) * 16 + (line & 15u);
            const uint32_t tr_k = mr * unit_rows + k;
            if (col < (uint64_t)cols && tr_k < nrb)
              *reinterpret_cast<uint2 *>(codes_col + col * (uint64_t)(rows / 2) + tr_k * 8u) =
                  col_stage[line * kColStagePitch + k];
          }
        }
        __syncthreads();
      }
    }
  }
}

#if NVFP4_46_MAIN
// 2D-block data -> BF16: one lane per 8 codes; the scale is the tile's.
__global__ __launch_bounds__(kThreads) void k_dequant_2d(const uint32_t *__restrict__ codes,
                                                         const uint8_t *__restrict__ scales,
                                                         const float *__restrict__ alpha_p,
                                                         uint4 *__restrict__ out, int64_t n8,
                                                         int64_t cols) {
  const float alpha = *alpha_p;
  const int64_t per_row = cols / 8, ncb = cols / 16;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < n8; t += stride) {
    const int64_t row = t / per_row, c8 = t - row * per_row;
    const float dec = e4m3_decode(scales[(row >> 4) * ncb + (c8 >> 1)]) * alpha;
    float D[8];
    dequant8(codes[t], dec, D);
    store_as<kNtBf16>(out + t, make_uint4(pack_bf16x2(D[0], D[1]), pack_bf16x2(D[2], D[3]),
                                          pack_bf16x2(D[4], D[5]), pack_bf16x2(D[6], D[7])));
  }
}

// ------------------------------------------------------------ debug kernels

__global__ void k_dbg_e2m1_rtn(uint32_t first, int64_t n, uint8_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    float y = u2f(first + (uint32_t)i);
    out[i] = (uint8_t)(hw_pk_fp4<0>(0u, y, 0.0f) & 15u);
  }
}

__global__ void k_dbg_e4m3(uint32_t first, int64_t n, uint8_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    out[i] = (uint8_t)e4m3_encode(u2f(first + (uint32_t)i));
}

__global__ void k_dbg_tables(float *out) {
  const int t = threadIdx.x;
  if (t < 16) {
    float D[8];
    dequant8((uint32_t)t, 1.0f, D);     // code t in nibble 0
    out[t] = D[0];
  }
  if (t < 256) out[16 + t] = e4m3_decode((uint32_t)t & 0x7fu);
}

__global__ void k_dbg_bf16(uint32_t first, uint32_t stride_bits, int64_t n, uint16_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    out[i] = (uint16_t)pack_bf16x2(u2f(first + (uint32_t)i * stride_bits), 0.0f);
}

__global__ void k_dbg_e2m1_sr(const float *y, const uint32_t *w, int64_t n, uint8_t *out,
                              uint8_t *out_fast) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    out[i] = (uint8_t)e2m1_code_of_grid_value(e2m1_sr_value(y[i], sr_uniform_of_word(w[i])));
    float margin = __builtin_inff();
    const uint32_t code = e2m1_sr_code_fast<0>(0u, y[i], ~w[i], (float)w[i], margin) & 0x0fu;
    out_fast[i] = (uint8_t)(code | (margin > kSrMarginAtRisk ? 0u : 0x80u));
  }
}

__global__ void k_dbg_philox(const uint32_t *ctr, uint32_t k0, uint32_t k1, int64_t n,
                             uint32_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    Philox4 p = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1);
#pragma unroll
    for (int j = 0; j < 4; ++j) out[4 * i + j] = p.w[j];
  }
}

#endif

// ---------------------------------------------------------------- launchers

constexpr int kMaxDevices = 64;
// Compute units of the device that is current for the calling thread (two devices of one process may differ), which does not
// change: asked for in a device's first calls (once for each part that the library is built of) and kept; threads that ask at the
// same time are told the same.
static int compute_units() {
  static std::atomic<int> known[kMaxDevices];
  int dev = -1, cus = 0;
  const bool counted = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices;
  if (counted && (cus = known[dev].load(std::memory_order_relaxed)) > 0) return cus;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  if (counted) known[dev].store(cus, std::memory_order_relaxed);
  return cus;
}

static int grid_for(int64_t work_items, int per_cu, int cus) {
  int64_t need = (work_items + kThreads - 1) / kThreads;
  int64_t cap = (int64_t)cus * per_cu;
  if (need < 1) need = 1;
  return (int)(need < cap ? need : cap);
}
static int grid_for(int64_t work_items, int per_cu) { return grid_for(work_items, per_cu, compute_units()); }

// every kernel of this file uses static LDS only
template <typename Kernel, typename... Args>
static int launch(Kernel kernel, dim3 grid, dim3 block, hipStream_t stream, Args... args) {
  return launch(kernel, grid, block, (size_t)0, stream, args...);
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct FlatArgs {
  bool xf32;        // x holds fp32 values instead of BF16
  const uint4 *x;
  const float *alpha;
  uint2 *codes;
  uint8_t *scales, *choice;
  uint4 *out;
  uint32_t *amax;
  int64_t nblocks;
  uint32_t nb_per_row;
  uint64_t sr_seed, rht_seed;
  hipStream_t stream;
  AmaxFinish fin{nullptr, nullptr, 0.0f};   // the amax pass, and (its alpha) kOutScaleAndCodes
};

template <bool XF32, int ROUNDING, int SELECT, bool RHT, int OUT>
static int launch_flat(const FlatArgs &a) {
  const int64_t rounds = (a.nblocks + kThreads - 1) / kThreads;
  const int cus = compute_units();
  int64_t n_long = 0, rounds_long = 0, grid;
  // With the transform a workgroup first draws its lanes' sign words, so a tensor of fewer rounds leaves fewer of them to
  // one-round workgroups, an eighth (us with sixteen rounds per compute unit / an eighth: Hadamard + SR
  // 4096 x 4096 24.8 / 23.5, 16384 x 2048 46.9 / 43.3, 8192 x 8192 70.3 / 68.3; to nearest 1 to 15 % in BF16 and under the rules
  // that compare in fp32; from 16384 x 8192 on the same).  Not the codes of one fp32 candidate rounded to nearest, which wait
  // for memory: 5248 x 6192 23.2 / 23.8, 6144 x 6144 3.7 %, 8192 x 4096 2.5 %.
  int64_t short_rounds = (int64_t)cus * kFlatShortRoundsPerCu;
  constexpr bool kMemoryBound =
      XF32 && ROUNDING == kRTN && OUT == kOutCodes && (SELECT == kSelForce6 || SELECT == kSelForce4);
  if (RHT && !kMemoryBound && short_rounds > rounds / 8) short_rounds = rounds / 8;
  if (OUT == kOutAmax) {
    // the amax pass ends with one access per workgroup to the one result word: few,
    // long-lived workgroups that stride over the whole tensor
    grid = (int64_t)cus * kFlatAmaxWgPerCu;
    if (grid > rounds) grid = rounds;
  } else {
    n_long = (int64_t)cus * kFlatLongWgPerCu;
    rounds_long = (rounds - short_rounds) / n_long;
    if (rounds_long < 2) n_long = rounds_long = 0;   // a small tensor: one round per workgroup
    grid = n_long + (rounds - n_long * rounds_long);
  }
  if (RHT) {
    // round r starts at block 256*r; if 256 * (a workgroup's stride) is a multiple of the
    // blocks per row, every lane sees one position along the row in all its rounds
    uint32_t g = a.nb_per_row, t = kThreads;
    while (t) { const uint32_t q = g % t; g = t; t = q; }      // gcd(nb_per_row, 256)
    const int64_t period = a.nb_per_row / g;
    if (OUT == kOutAmax) {
      if (period <= grid / 2) grid -= grid % period;
    } else if (n_long && period <= n_long / 2) {
      n_long -= n_long % period;
      rounds_long = (rounds - short_rounds) / n_long;
      grid = n_long + (rounds - n_long * rounds_long);
    }
  }
  auto go = [&](auto kernel) {
    return launch(kernel, dim3((uint32_t)grid), dim3(kThreads),
                  a.stream, a.x, a.alpha, a.codes, a.scales, a.choice, a.out, a.amax, a.nblocks,
                  a.nb_per_row, a.sr_seed, a.rht_seed, (uint32_t)n_long, (uint32_t)rounds_long,
                  runs_backwards(a.nblocks * 16, XF32), a.fin);
  };
  // The transform's maximum of BF16 is taken with packed flips (the kernel's kPacked, which for a maximum is all that SELECT
  // says) where a workgroup has at most two rounds: less to set up; else per value (us, per value / packed: 256 x 1024
  // 4.7 / 4.6, 2048 x 2048 6.4 / 6.0; 2560 x 2048 6.1 / 6.5, 5248 x 6192 17.2 / 17.8, 32768 x 8192 94 / 97).
  if constexpr (OUT == kOutAmax && !XF32)
    if (rounds > (int64_t)2 * cus * kFlatAmaxWgPerCu) return go(k_flat<XF32, ROUNDING, kSelForce6, RHT, OUT>);
  return go(k_flat<XF32, ROUNDING, SELECT, RHT, OUT>);
}

template <bool XF32, int ROUNDING, int SELECT>
static int launch_flat_variant(const FlatArgs &a, bool rht, int out) {
  if constexpr (ROUNDING == kRTN) {
    if (out == kOutScaleAndCodes)
      return launch(k_scale_quantize_small<XF32, SELECT>,
                    dim3((uint32_t)((a.nblocks + kSmallBlocks - 1) / kSmallBlocks)), dim3(kSmallThreads),
                    a.stream, a.x, a.fin.alpha, a.codes, a.scales, a.choice, (uint32_t)a.nblocks,
                    a.fin.fp8_max);
  }
  if (out == kOutCodes) {
    if (rht) return launch_flat<XF32, ROUNDING, SELECT, true, kOutCodes>(a);
    return launch_flat<XF32, ROUNDING, SELECT, false, kOutCodes>(a);
  }
  if (rht) return launch_flat<XF32, ROUNDING, SELECT, true, kOutFake>(a);
  return launch_flat<XF32, ROUNDING, SELECT, false, kOutFake>(a);
}

// All rowwise kernels of one (input type, rounding mode) pair.
template <bool XF32, int ROUNDING>
int run_flat(const FlatArgs &a, uint32_t select, bool rht, int out) {
  if (select == NVFP4_SEL_46_MSE) return launch_flat_variant<XF32, ROUNDING, kSel46>(a, rht, out);
  if (select == NVFP4_SEL_FORCE6) return launch_flat_variant<XF32, ROUNDING, kSelForce6>(a, rht, out);
  if (select == NVFP4_SEL_FORCE4) return launch_flat_variant<XF32, ROUNDING, kSelForce4>(a, rht, out);
  if (select == NVFP4_SEL_46_MAE) return launch_flat_variant<XF32, ROUNDING, kSel46Mae>(a, rht, out);
  return launch_flat_variant<XF32, ROUNDING, kSel46AbsMax>(a, rht, out);
}

struct TileArgs {
  bool xf32;
  const void *x;
  const float *alpha;
  uint8_t *codes_row, *scales_row, *choice_row, *codes_col, *scales_col, *choice_col;
  uint16_t *out;
  int64_t rows, cols;
  uint64_t sr_seed, rht_seed;
  hipStream_t stream;
};

template <bool XF32, int ROUNDING, int SELECT, bool RHT, bool WANT_ROW, int OUT>
static int launch_tile(const TileArgs &a) {
  TileMap map = tile_map(a.rows, a.cols);
  const int grid = tile_grid(a.rows, a.cols, map);
  if (runs_backwards(a.rows * a.cols, XF32)) map.last = (uint32_t)grid - 1u;
  return launch(k_tile<XF32, ROUNDING, SELECT, RHT, WANT_ROW, OUT>, dim3(grid), dim3(kThreads), a.stream,
                a.x, a.alpha, a.codes_row, a.scales_row, a.choice_row, a.codes_col, a.scales_col,
                a.choice_col, a.out, a.rows, a.cols, a.sr_seed, a.rht_seed, map);
}

// variant: 0 = columnwise codes, 1 = columnwise codes + rht, 2 = both orientations,
//          3 = columnwise fake-quant, 4 = columnwise fake-quant + rht
template <bool XF32, int ROUNDING, int SELECT>
static int launch_tile_variant(const TileArgs &a, int variant) {
  switch (variant) {
    case 0: return launch_tile<XF32, ROUNDING, SELECT, false, false, kOutCodes>(a);
    case 1: return launch_tile<XF32, ROUNDING, SELECT, true, false, kOutCodes>(a);
    case 2: return launch_tile<XF32, ROUNDING, SELECT, false, true, kOutCodes>(a);
    case 3: return launch_tile<XF32, ROUNDING, SELECT, false, false, kOutFake>(a);
    default: return launch_tile<XF32, ROUNDING, SELECT, true, false, kOutFake>(a);
  }
}

// All tiled (columnwise / both) kernels of one (input type, rounding mode) pair.
template <bool XF32, int ROUNDING>
int run_tile(const TileArgs &a, uint32_t select, int variant) {
  if (select == NVFP4_SEL_46_MSE) return launch_tile_variant<XF32, ROUNDING, kSel46>(a, variant);
  if (select == NVFP4_SEL_FORCE6) return launch_tile_variant<XF32, ROUNDING, kSelForce6>(a, variant);
  if (select == NVFP4_SEL_FORCE4) return launch_tile_variant<XF32, ROUNDING, kSelForce4>(a, variant);
  if (select == NVFP4_SEL_46_MAE) return launch_tile_variant<XF32, ROUNDING, kSel46Mae>(a, variant);
  return launch_tile_variant<XF32, ROUNDING, kSel46AbsMax>(a, variant);
}

struct TilePairArgs {
  TilePair p;
  int64_t rows;
  uint64_t sr_seed, rht_seed;
  uint32_t blocks_a, blocks;
  hipStream_t stream;
};
int run_tile_pair(const TilePairArgs &a, uint32_t select);
#if NVFP4_46_PART == 2 || NVFP4_46_PART < 0
int run_tile_pair(const TilePairArgs &a, uint32_t select) {
  auto go = [&](auto kernel) {
    return launch(kernel, dim3(a.blocks), dim3(kThreads), a.stream, a.p, a.rows, a.sr_seed, a.rht_seed, a.blocks_a);
  };
  if (select == NVFP4_SEL_46_MSE) return go(k_tile_pair<kSel46>);
  if (select == NVFP4_SEL_FORCE6) return go(k_tile_pair<kSelForce6>);
  if (select == NVFP4_SEL_FORCE4) return go(k_tile_pair<kSelForce4>);
  if (select == NVFP4_SEL_46_MAE) return go(k_tile_pair<kSel46Mae>);
  return go(k_tile_pair<kSel46AbsMax>);
}
#endif

struct Block2dArgs {
  bool xf32;
  const void *x;
  const float *alpha;
  uint8_t *codes, *scales, *choice, *codes_col, *scales_col, *choice_col;
  uint16_t *out;
  int64_t rows, cols;
  uint64_t sr_seed;
  hipStream_t stream;
};

template <bool XF32, int ROUNDING, int SELECT>
static int launch_block2d(const Block2dArgs &a, int out) {
  // ids as the kernel counts them: sixteen tiles each, or - with the transposed packing - units
  // of 4, 8 or 16 x 4 tiles in whole groups of 32
  const int64_t tiles = (a.rows / 16) * (a.cols / 16);
  const int cus = compute_units();
  const int64_t unit_rows = tile_unit_rows(a.rows, a.cols, XF32, cus);
  const int64_t units = ((a.rows / 16 + unit_rows - 1) / unit_rows) * ((a.cols / 16 + 3) / 4);
  const int64_t ids = out == kOutCodes && a.codes_col ? ((units + 31) / 32) * 32 : (tiles + 15) / 16;
  const int grid = grid_for(ids * kThreads, 16, cus);
  auto go = [&](auto kernel) {
    return launch(kernel, dim3(grid), dim3(kThreads), a.stream, a.x, a.alpha, a.codes, a.scales,
                  a.choice, a.codes_col, a.scales_col, a.choice_col, a.out, a.rows, a.cols,
                  a.sr_seed, runs_backwards(a.rows * a.cols, XF32));
  };
  if (out == kOutCodes && a.codes_col)
    return unit_rows == 4   ? go(k_block2d<XF32, ROUNDING, SELECT, kOutCodes, 4>)
           : unit_rows == 8 ? go(k_block2d<XF32, ROUNDING, SELECT, kOutCodes, 8>)
                            : go(k_block2d<XF32, ROUNDING, SELECT, kOutCodes, 16>);
  if (out == kOutCodes) return go(k_block2d<XF32, ROUNDING, SELECT, kOutCodes, 0>);
  return go(k_block2d<XF32, ROUNDING, SELECT, kOutFake, 0>);
}

// All 16x16-tile kernels of one (input type, rounding mode) pair.
template <bool XF32, int ROUNDING>
int run_block2d(const Block2dArgs &a, uint32_t select, int out) {
  if (select == NVFP4_SEL_46_MSE) return launch_block2d<XF32, ROUNDING, kSel46>(a, out);
  if (select == NVFP4_SEL_FORCE6) return launch_block2d<XF32, ROUNDING, kSelForce6>(a, out);
  if (select == NVFP4_SEL_FORCE4) return launch_block2d<XF32, ROUNDING, kSelForce4>(a, out);
  if (select == NVFP4_SEL_46_MAE) return launch_block2d<XF32, ROUNDING, kSel46Mae>(a, out);
  return launch_block2d<XF32, ROUNDING, kSel46AbsMax>(a, out);
}

// One group of kernels = the three run_* templates for one (XF32, ROUNDING) pair.  A part
// that holds a group defines it; the main part, when built apart, only declares them.
#define NVFP4_46_GROUP(KEYWORD, XF32, ROUNDING)                                                 \
  KEYWORD template int run_flat<XF32, ROUNDING>(const FlatArgs &, uint32_t, bool, int);         \
  KEYWORD template int run_tile<XF32, ROUNDING>(const TileArgs &, uint32_t, int);               \
  KEYWORD template int run_block2d<XF32, ROUNDING>(const Block2dArgs &, uint32_t, int);
#if NVFP4_46_PART == 0
NVFP4_46_GROUP(extern, false, kRTN)
NVFP4_46_GROUP(extern, false, kSR)
NVFP4_46_GROUP(extern, false, kSRAfterRtnSelect)
NVFP4_46_GROUP(extern, true, kRTN)
NVFP4_46_GROUP(extern, true, kSR)
NVFP4_46_GROUP(extern, true, kSRAfterRtnSelect)
#elif NVFP4_46_PART >= 1 && NVFP4_46_PART <= 6
static_assert(kRTN == 0 && kSR == 1 && kSRAfterRtnSelect == 2, "parts are numbered by these");
NVFP4_46_GROUP(, ((NVFP4_46_PART - 1) / 3 != 0), ((NVFP4_46_PART - 1) % 3))
#endif

#if NVFP4_46_MAIN
static int rounding_index(uint32_t rounding) {
  return rounding == NVFP4_SR ? kSR : rounding == NVFP4_SR_AFTER_RTN_SELECT ? kSRAfterRtnSelect : kRTN;
}

static int dispatch_flat(const FlatArgs &a, uint32_t rounding, uint32_t select, bool rht, int out) {
  typedef int (*Fn)(const FlatArgs &, uint32_t, bool, int);
  static const Fn table[2][3] = {
      {run_flat<false, kRTN>, run_flat<false, kSR>, run_flat<false, kSRAfterRtnSelect>},
      {run_flat<true, kRTN>, run_flat<true, kSR>, run_flat<true, kSRAfterRtnSelect>}};
  return table[a.xf32][rounding_index(rounding)](a, select, rht, out);
}

static int dispatch_tile(const TileArgs &a, uint32_t rounding, uint32_t select, int variant) {
  typedef int (*Fn)(const TileArgs &, uint32_t, int);
  static const Fn table[2][3] = {
      {run_tile<false, kRTN>, run_tile<false, kSR>, run_tile<false, kSRAfterRtnSelect>},
      {run_tile<true, kRTN>, run_tile<true, kSR>, run_tile<true, kSRAfterRtnSelect>}};
  return table[a.xf32][rounding_index(rounding)](a, select, variant);
}

static int dispatch_block2d(const Block2dArgs &a, uint32_t rounding, uint32_t select, int out) {
  typedef int (*Fn)(const Block2dArgs &, uint32_t, int);
  static const Fn table[2][3] = {
      {run_block2d<false, kRTN>, run_block2d<false, kSR>, run_block2d<false, kSRAfterRtnSelect>},
      {run_block2d<true, kRTN>, run_block2d<true, kSR>, run_block2d<true, kSRAfterRtnSelect>}};
  return table[a.xf32][rounding_index(rounding)](a, select, out);
}

// Checks shared by the entry points that take the parameter block.
static int check_params(const void *x, const nvfp4_46_params *p, bool one_layout_only) {
  if (!x || !p) return NVFP4_ERR_NULL;
  if (p->rows <= 0 || p->cols <= 0) return NVFP4_ERR_SHAPE;
  if (p->layout < 1u || p->layout > 3u) return NVFP4_ERR_PARAM;
  if (one_layout_only && p->layout == 3u) return NVFP4_ERR_PARAM;
  if (p->rounding > NVFP4_SR_AFTER_RTN_SELECT || p->select > NVFP4_SEL_46_ABSMAX || p->rht > 1u ||
      p->block2d > 1u || p->x_dtype > NVFP4_X_F32)
    return NVFP4_ERR_PARAM;
  if (!(p->fp8_max > 0.0f) || !(p->fp8_max <= 448.0f)) return NVFP4_ERR_PARAM;
  if ((p->layout & NVFP4_ROWWISE) && (p->cols % 16) != 0) return NVFP4_ERR_SHAPE;
  if ((p->layout & NVFP4_COLWISE) && ((p->rows % 16) != 0 || (p->cols % 8) != 0))
    return NVFP4_ERR_SHAPE;
  if (p->rows > (int64_t)1 << 31 || p->cols > (int64_t)1 << 31 ||
      p->rows * p->cols > (int64_t)1 << 40)
    return NVFP4_ERR_SHAPE;
  if (!aligned16(x)) return NVFP4_ERR_ALIGN;
  if (p->rht && p->layout == 3u) return NVFP4_ERR_UNSUPPORTED;
  if (p->block2d) {
    if ((p->rows % 16) != 0 || (p->cols % 16) != 0) return NVFP4_ERR_SHAPE;
    if (p->rht) return NVFP4_ERR_UNSUPPORTED;
  }
  return NVFP4_OK;
}

static int check_outputs(const nvfp4_46_params *p, const void *codes_row, const void *scales_row,
                         const void *codes_col, const void *scales_col, const void *choice_row,
                         const void *choice_col) {
  const bool want_row = p->layout & NVFP4_ROWWISE, want_col = p->layout & NVFP4_COLWISE;
  if (want_row && (!codes_row || !scales_row)) return NVFP4_ERR_NULL;
  if (want_col && (!codes_col || !scales_col)) return NVFP4_ERR_NULL;
  if (!want_row && (codes_row || scales_row || choice_row)) return NVFP4_ERR_PARAM;
  if (!want_col && (codes_col || scales_col || choice_col)) return NVFP4_ERR_PARAM;
  if (!aligned16(codes_row) || !aligned16(scales_row) || !aligned16(codes_col) ||
      !aligned16(scales_col) || !aligned16(choice_row) || !aligned16(choice_col))
    return NVFP4_ERR_ALIGN;
  return NVFP4_OK;
}

static int check_workspace(const void *workspace, size_t bytes) {
  if (bytes < NVFP4_46_TENSOR_SCALE_WS_BYTES) return NVFP4_ERR_PARAM;
  return aligned16(workspace) ? NVFP4_OK : NVFP4_ERR_ALIGN;
}

// Two sets of scratch words, the maximum and ticket words of the one-launch reduction (see AmaxFinish), 4352
// bytes each; every GPU the library runs on holds its own copy until the process ends.  The first belongs to
// nvfp4_46_tensor_scale_static, the second to calls on the default stream that bring no workspace.
// In host code the array's name only stands for the symbol: the device address is looked up once per device
// and that pointer is what kernels get (threads that look it up at the same time find the same).
static __device__ __align__(256) uint32_t scratch[2 * kScratchWords];
static_assert(kScratchWords * sizeof(uint32_t) == NVFP4_46_TENSOR_SCALE_WS_BYTES, "header and kernels agree on the scratch size");
static std::atomic<uint32_t *> g_scratch_ptr[kMaxDevices];   // per device; nullptr until that device's first call

static uint32_t *scratch_of_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  uint32_t *words = g_scratch_ptr[dev].load(std::memory_order_relaxed);
  if (!words) {
    void *sym = nullptr;
    if (hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)) != hipSuccess || !sym) return nullptr;
    words = static_cast<uint32_t *>(sym);
    g_scratch_ptr[dev].store(words, std::memory_order_relaxed);
  }
  return words;
}

// Scratch words for a call that brings none.  Work on a device's default stream (handle 0, one for all threads) runs in
// the order of its calls and is never captured into a graph, so one set serves all of it; any other
// stream gets nullptr, the form of three launches (us per call from Python among others, three / one: BF16 1 MiB
// 10.0 / 4.8, 8 MiB 9.6 / 4.8, 32 MiB 10.8 / 5.3, 128 MiB 23.6 / 22.0, with the columnwise transform 9.9 / 5.9,
// 9.8 / 6.0, 12.1 / 7.3 and 26.9 / 23.6).
static uint32_t *lent_words(hipStream_t stream) {
  if (stream) return nullptr;
  uint32_t *const words = scratch_of_device();
  return words ? words + kScratchWords : nullptr;
}

// Eq. (1) for all entry points.  scratch == nullptr: the reduction runs on the caller's
// alpha word between a zeroing launch and a finishing launch.  Otherwise scratch points at
// kScratchWords zeroed words and one launch does it all (see AmaxFinish).  `workspace`: the caller's words, or
// nullptr for such as can be lent.
static int tensor_scale(const void *x, const nvfp4_46_params *p, float *alpha, uint32_t *workspace,
                        hipStream_t s) {
  if (!alpha) return NVFP4_ERR_NULL;
  int rc = check_params(x, p, false);
  if (rc != NVFP4_OK) return rc;
  const int64_t n = p->rows * p->cols;
  const bool xf32 = p->x_dtype == NVFP4_X_F32;
  const uint4 *x4 = static_cast<const uint4 *>(x);
  const int64_t bytes = n * (xf32 ? 4 : 2);
  const ScratchWords words = workspace ? ScratchWords::kWorkspace : s ? ScratchWords::kNone : ScratchWords::kLent;
  if (!p->rht && scale_in_one_workgroup(bytes, words)) {
    const uint32_t n16 = (uint32_t)(bytes / 16);       // n is a multiple of 8 by the shape checks
    return xf32 ? launch(k_scale_small<true>, dim3(1), dim3(kSmallThreads), s, x4, n16, alpha, p->fp8_max)
                : launch(k_scale_small<false>, dim3(1), dim3(kSmallThreads), s, x4, n16, alpha, p->fp8_max);
  }
  uint32_t *const scratch = workspace ? workspace : lent_words(s);
  uint32_t *amax = reinterpret_cast<uint32_t *>(alpha);      // the plain form's running maximum
  const AmaxFinish fin{scratch, alpha, p->fp8_max};
  if (!scratch) {
    rc = launch(k_store_u32, dim3(1), dim3(1), s, amax, 0u);
    if (rc != NVFP4_OK) return rc;
  }
  if (!p->rht) {
    // 128-bit pieces (n is a multiple of 8 by the shape checks)
    const int64_t n16 = xf32 ? n / 4 : n / 8;
    const dim3 grid(grid_for(n16, kAmaxWgPerCu));
    rc = xf32 ? launch(k_amax_plain<true>, grid, dim3(kThreads), s, x4, n16, amax, fin)
              : launch(k_amax_plain<false>, grid, dim3(kThreads), s, x4, n16, amax, fin);
  } else if (p->layout == NVFP4_ROWWISE) {
    FlatArgs a{xf32, x4, nullptr, nullptr, nullptr, nullptr, nullptr, amax,
               n / 16, (uint32_t)(p->cols / 16), 0, p->rht_seed, s, fin};
    rc = xf32 ? launch_flat<true, kRTN, kSel46, true, kOutAmax>(a)
              : launch_flat<false, kRTN, kSel46, true, kOutAmax>(a);
  } else {
    // columnwise blocks (rows % 16 == 0, cols % 8 == 0): 16 or 4 bytes of a row per lane
    const int64_t row_blocks = p->rows / 16, words = p->cols / (xf32 ? 1 : 2);
    auto go = [&](auto kernel, int64_t pieces) {
      return launch(kernel, dim3(grid_for(row_blocks * pieces, kAmaxRhtColWgPerCu)), dim3(kThreads), s,
                    static_cast<const uint32_t *>(x), row_blocks, pieces, p->rht_seed, amax, fin);
    };
    if (scale_by_words(row_blocks * words, xf32))
      rc = xf32 ? go(k_amax_rht_col<true, 1>, words) : go(k_amax_rht_col<false, 1>, words);
    else
      rc = xf32 ? go(k_amax_rht_col<true, 4>, words / 4) : go(k_amax_rht_col<false, 4>, words / 4);
  }
  if (rc != NVFP4_OK || scratch) return rc;
  return launch(k_finish_alpha, dim3(1), dim3(1), s, alpha, p->fp8_max);
}

#endif  // NVFP4_46_MAIN

}  // namespace nvfp4_46

#if NVFP4_46_MAIN

using namespace nvfp4_46;

extern "C" {

int nvfp4_46_tensor_scale(const void *x, const nvfp4_46_params *p, float *alpha, void *stream) {
  return tensor_scale(x, p, alpha, nullptr, static_cast<hipStream_t>(stream));
}

int nvfp4_46_tensor_scale_ws(const void *x, const nvfp4_46_params *p, float *alpha,
                             void *workspace, size_t workspace_bytes, void *stream) {
  if (!workspace) return NVFP4_ERR_NULL;
  const int rc = check_workspace(workspace, workspace_bytes);
  if (rc != NVFP4_OK) return rc;
  return tensor_scale(x, p, alpha, static_cast<uint32_t *>(workspace), static_cast<hipStream_t>(stream));
}

int nvfp4_46_tensor_scale_static(const void *x, const nvfp4_46_params *p, float *alpha, void *stream) {
  uint32_t *const words = scratch_of_device();
  if (!words) return NVFP4_ERR_HIP;
  return tensor_scale(x, p, alpha, words, static_cast<hipStream_t>(stream));
}

int nvfp4_46_quantize(const void *x, const nvfp4_46_params *p, const float *alpha,
                      void *codes_row, void *scales_row, void *codes_col, void *scales_col,
                      void *choice_row, void *choice_col, void *stream) {
  if (!alpha) return NVFP4_ERR_NULL;
  int rc = check_params(x, p, false);
  if (rc != NVFP4_OK) return rc;
  const bool xf32 = p->x_dtype == NVFP4_X_F32;
  const bool want_row = p->layout & NVFP4_ROWWISE, want_col = p->layout & NVFP4_COLWISE;
  rc = check_outputs(p, codes_row, scales_row, codes_col, scales_col, choice_row, choice_col);
  if (rc != NVFP4_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->block2d) {
    Block2dArgs a{xf32, x, alpha, static_cast<uint8_t *>(codes_row),
                  static_cast<uint8_t *>(scales_row), static_cast<uint8_t *>(choice_row),
                  static_cast<uint8_t *>(codes_col), static_cast<uint8_t *>(scales_col),
                  static_cast<uint8_t *>(choice_col), nullptr, p->rows, p->cols, p->sr_seed, s};
    return dispatch_block2d(a, p->rounding, p->select, kOutCodes);
  }
  if (!want_col) {
    FlatArgs a{xf32, static_cast<const uint4 *>(x), alpha, static_cast<uint2 *>(codes_row),
               static_cast<uint8_t *>(scales_row), static_cast<uint8_t *>(choice_row), nullptr,
               nullptr, p->rows * p->cols / 16, (uint32_t)(p->cols / 16), p->sr_seed, p->rht_seed, s};
    return dispatch_flat(a, p->rounding, p->select, p->rht != 0, kOutCodes);
  }
  TileArgs a{xf32, x, alpha, static_cast<uint8_t *>(codes_row),
             static_cast<uint8_t *>(scales_row), static_cast<uint8_t *>(choice_row),
             static_cast<uint8_t *>(codes_col), static_cast<uint8_t *>(scales_col),
             static_cast<uint8_t *>(choice_col), nullptr, p->rows, p->cols, p->sr_seed,
             p->rht_seed, s};
  return dispatch_tile(a, p->rounding, p->select, want_row ? 2 : (p->rht ? 1 : 0));
}

int nvfp4_46_scale_quantize(const void *x, const nvfp4_46_params *p, float *alpha,
                            void *workspace, size_t workspace_bytes, void *codes_row,
                            void *scales_row, void *codes_col, void *scales_col,
                            void *choice_row, void *choice_col, void *stream) {
  // in the order of the two calls
  int rc = workspace ? check_workspace(workspace, workspace_bytes) : NVFP4_OK;
  if (rc == NVFP4_OK && !alpha) rc = NVFP4_ERR_NULL;
  if (rc == NVFP4_OK) rc = check_params(x, p, false);
  if (rc == NVFP4_OK)
    rc = check_outputs(p, codes_row, scales_row, codes_col, scales_col, choice_row, choice_col);
  if (rc != NVFP4_OK) return rc;
  const bool xf32 = p->x_dtype == NVFP4_X_F32;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->layout == NVFP4_ROWWISE && p->rounding == NVFP4_RTN && !p->rht && !p->block2d &&
      scale_and_codes_in_one_launch(p->rows * p->cols * (xf32 ? 4 : 2), workspace != nullptr)) {
    FlatArgs a{xf32, static_cast<const uint4 *>(x), nullptr, static_cast<uint2 *>(codes_row),
               static_cast<uint8_t *>(scales_row), static_cast<uint8_t *>(choice_row), nullptr,
               nullptr, p->rows * p->cols / 16, (uint32_t)(p->cols / 16), 0, 0, s,
               AmaxFinish{nullptr, alpha, p->fp8_max}};
    return dispatch_flat(a, p->rounding, p->select, false, kOutScaleAndCodes);
  }
  rc = tensor_scale(x, p, alpha, static_cast<uint32_t *>(workspace), s);
  if (rc != NVFP4_OK) return rc;
  return nvfp4_46_quantize(x, p, alpha, codes_row, scales_row, codes_col, scales_col, choice_row,
                           choice_col, stream);
}

// (see layer.hpp)
int nvfp4_46_wgrad_operands(const void *dy, const void *x, int64_t rows, int64_t n, int64_t k, uint32_t select,
                            uint64_t sr_seed, uint64_t rht_seed, float *alpha_dy, void *codes_dy, void *scales_dy,
                            float *alpha_x, void *codes_x, void *scales_x, void *workspace, size_t workspace_bytes,
                            void *stream) {
  const nvfp4_46_params pd{rows, n, NVFP4_COLWISE, NVFP4_SR, select, 1u, sr_seed, rht_seed, 256.0f, 0u, NVFP4_X_BF16};
  const nvfp4_46_params px{rows, k, NVFP4_COLWISE, NVFP4_RTN, select, 1u, 0u, rht_seed, 256.0f, 0u, NVFP4_X_BF16};
  int rc = workspace ? check_workspace(workspace, workspace_bytes) : NVFP4_OK;
  if (rc == NVFP4_OK && (!alpha_dy || !alpha_x)) rc = NVFP4_ERR_NULL;
  if (rc == NVFP4_OK) rc = check_params(dy, &pd, false);
  if (rc == NVFP4_OK) rc = check_params(x, &px, false);
  if (rc == NVFP4_OK) rc = check_outputs(&pd, nullptr, nullptr, codes_dy, scales_dy, nullptr, nullptr);
  if (rc == NVFP4_OK) rc = check_outputs(&px, nullptr, nullptr, codes_x, scales_x, nullptr, nullptr);
  if (rc != NVFP4_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const bool in_cache = rows * (n + k) * 2 <= kLastLevelBytes;
  uint32_t *const words = !in_cache ? nullptr : workspace ? static_cast<uint32_t *>(workspace) : lent_words(s);
  // (us in a replayed graph with the product, four launches / two: 64 tokens, 256 x 256 25.5 / 15.4, 736 tokens, 1024 x 1024
  // 35.8 / 20.1, 2048 tokens, 2048 x 2048 59 / 43, 4096 x 4096 103 / 94, 8192 tokens 307 / 297; what no longer fits the
  // memory-side cache goes one after the other, the second pass over a tensor last to first)
  if (!words) {
    rc = nvfp4_46_scale_quantize(dy, &pd, alpha_dy, workspace, workspace_bytes, nullptr, nullptr, codes_dy, scales_dy,
                                 nullptr, nullptr, stream);
    if (rc != NVFP4_OK) return rc;
    return nvfp4_46_scale_quantize(x, &px, alpha_x, workspace, workspace_bytes, nullptr, nullptr, codes_x, scales_x,
                                   nullptr, nullptr, stream);
  }
  const TileMap map[2] = {tile_map(rows, n), tile_map(rows, k)};
  const uint32_t tiles[2] = {(uint32_t)tile_grid(rows, n, map[0]), (uint32_t)tile_grid(rows, k, map[1])};
  const int64_t row_blocks = rows / 16;
  const bool narrow = scale_by_words(row_blocks * (n + k) / 2, false);     // of both together
  const int64_t per_piece = narrow ? 2 : 8;
  const AmaxPair both{{static_cast<const uint32_t *>(dy), static_cast<const uint32_t *>(x)},
                      {n / per_piece, k / per_piece},
                      {alpha_dy, alpha_x}};
  const int cus = compute_units();
  const uint32_t blocks_a = (uint32_t)grid_for(row_blocks * both.pieces_per_row[0], kAmaxRhtColWgPerCu / 2, cus);
  const uint32_t blocks_b = (uint32_t)grid_for(row_blocks * both.pieces_per_row[1], kAmaxRhtColWgPerCu / 2, cus);
  auto maxima = [&](auto kernel) {
    return launch(kernel, dim3(blocks_a + blocks_b), dim3(kThreads), s, both, row_blocks, rht_seed, blocks_a, words, 256.0f);
  };
  rc = narrow ? maxima(k_amax_rht_col_pair<1>) : maxima(k_amax_rht_col_pair<4>);
  if (rc != NVFP4_OK) return rc;
  const TilePair p{{dy, x},
                   {alpha_dy, alpha_x},
                   {static_cast<uint8_t *>(codes_dy), static_cast<uint8_t *>(codes_x)},
                   {static_cast<uint8_t *>(scales_dy), static_cast<uint8_t *>(scales_x)},
                   {n, k},
                   {map[0], map[1]}};
  return run_tile_pair(TilePairArgs{p, rows, sr_seed, rht_seed, tiles[0], tiles[0] + tiles[1], s}, select);
}

int nvfp4_46_dequantize(const void *codes, const void *scales, const float *alpha, int64_t rows,
                        int64_t cols, uint32_t layout, void *out_bf16, void *stream) {
  if (!codes || !scales || !alpha || !out_bf16) return NVFP4_ERR_NULL;
  if (rows <= 0 || cols <= 0) return NVFP4_ERR_SHAPE;
  if (layout != NVFP4_ROWWISE && layout != NVFP4_COLWISE && layout != NVFP4_BLOCK2D &&
      layout != (NVFP4_BLOCK2D | NVFP4_COLWISE))
    return NVFP4_ERR_PARAM;
  if ((layout & NVFP4_BLOCK2D) && ((rows % 16) != 0 || (cols % 16) != 0)) return NVFP4_ERR_SHAPE;
  if (layout == NVFP4_ROWWISE && (cols % 16) != 0) return NVFP4_ERR_SHAPE;
  if (layout == NVFP4_COLWISE && ((rows % 16) != 0 || (cols % 8) != 0)) return NVFP4_ERR_SHAPE;
  if (rows > (int64_t)1 << 31 || cols > (int64_t)1 << 31 || rows * cols > (int64_t)1 << 40)
    return NVFP4_ERR_SHAPE;
  if (!aligned16(codes) || !aligned16(scales) || !aligned16(out_bf16)) return NVFP4_ERR_ALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint8_t *c8 = static_cast<const uint8_t *>(codes), *s8 = static_cast<const uint8_t *>(scales);
  const int64_t n8 = rows * cols / 8;
  if (layout == NVFP4_BLOCK2D)
    return launch(k_dequant_2d, dim3(grid_for(n8, 16)), dim3(kThreads), s,
                  static_cast<const uint32_t *>(codes), s8, alpha, static_cast<uint4 *>(out_bf16),
                  n8, cols);
  if (layout == NVFP4_ROWWISE)
    return launch(k_dequant_flat, dim3(grid_for(n8, 16)), dim3(kThreads), s,
                  static_cast<const uint32_t *>(codes), s8, alpha, static_cast<uint4 *>(out_bf16),
                  n8);
  const TileMap map = tile_map(rows, cols);
  const dim3 grid(tile_grid(rows, cols, map));
  if (layout == NVFP4_COLWISE)
    return launch(k_dequant_col<false>, grid, dim3(kThreads), s, c8, s8, alpha, static_cast<uint16_t *>(out_bf16), rows,
                  cols, map);
  return launch(k_dequant_col<true>, grid, dim3(kThreads), s, c8, s8, alpha, static_cast<uint16_t *>(out_bf16), rows, cols,
                map);
}

int nvfp4_46_fake_quant(const void *x, const nvfp4_46_params *p, const float *alpha,
                        void *out_bf16, void *stream) {
  if (!alpha || !out_bf16) return NVFP4_ERR_NULL;
  int rc = check_params(x, p, true);
  if (rc != NVFP4_OK) return rc;
  const bool xf32 = p->x_dtype == NVFP4_X_F32;
  if (!aligned16(out_bf16)) return NVFP4_ERR_ALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (p->block2d) {
    Block2dArgs a{xf32, x, alpha, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr,
                  static_cast<uint16_t *>(out_bf16), p->rows, p->cols, p->sr_seed, s};
    return dispatch_block2d(a, p->rounding, p->select, kOutFake);
  }
  if (p->layout == NVFP4_ROWWISE) {
    FlatArgs a{xf32, static_cast<const uint4 *>(x), alpha, nullptr, nullptr, nullptr,
               static_cast<uint4 *>(out_bf16), nullptr, p->rows * p->cols / 16,
               (uint32_t)(p->cols / 16), p->sr_seed, p->rht_seed, s};
    return dispatch_flat(a, p->rounding, p->select, p->rht != 0, kOutFake);
  }
  TileArgs a{xf32, x, alpha, nullptr, nullptr, nullptr, nullptr,
             nullptr, nullptr, static_cast<uint16_t *>(out_bf16), p->rows, p->cols,
             p->sr_seed, p->rht_seed, s};
  return dispatch_tile(a, p->rounding, p->select, p->rht ? 4 : 3);
}

const char *nvfp4_46_status_string(int status) {
  switch (status) {
    case NVFP4_OK: return "ok";
    case NVFP4_ERR_NULL: return "a required pointer is NULL";
    case NVFP4_ERR_SHAPE: return "bad shape (dims must be positive, blocked axis a multiple of 16)";
    case NVFP4_ERR_ALIGN: return "buffer not 16-byte aligned";
    case NVFP4_ERR_PARAM: return "invalid parameter value";
    case NVFP4_ERR_UNSUPPORTED: return "unsupported combination of options";
    case NVFP4_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int nvfp4_46_debug_e2m1_rtn_range(uint32_t first_bits, int64_t n, void *out_u8, void *stream) {
  if (!out_u8) return NVFP4_ERR_NULL;
  if (n <= 0) return NVFP4_ERR_SHAPE;
  return launch(k_dbg_e2m1_rtn, dim3(grid_for(n, 8)), dim3(kThreads),
                static_cast<hipStream_t>(stream), first_bits, n, static_cast<uint8_t *>(out_u8));
}

int nvfp4_46_debug_e4m3_range(uint32_t first_bits, int64_t n, void *out_u8, void *stream) {
  if (!out_u8) return NVFP4_ERR_NULL;
  if (n <= 0) return NVFP4_ERR_SHAPE;
  return launch(k_dbg_e4m3, dim3(grid_for(n, 8)), dim3(kThreads),
                static_cast<hipStream_t>(stream), first_bits, n, static_cast<uint8_t *>(out_u8));
}

int nvfp4_46_debug_decode_tables(void *out_f32, void *stream) {
  if (!out_f32) return NVFP4_ERR_NULL;
  return launch(k_dbg_tables, dim3(1), dim3(256), static_cast<hipStream_t>(stream),
                static_cast<float *>(out_f32));
}

int nvfp4_46_debug_bf16_range(uint32_t first_bits, uint32_t stride, int64_t n, void *out_u16,
                              void *stream) {
  if (!out_u16) return NVFP4_ERR_NULL;
  if (n <= 0) return NVFP4_ERR_SHAPE;
  return launch(k_dbg_bf16, dim3(grid_for(n, 8)), dim3(kThreads),
                static_cast<hipStream_t>(stream), first_bits, stride, n,
                static_cast<uint16_t *>(out_u16));
}

int nvfp4_46_debug_e2m1_sr(const float *y, const uint32_t *words, int64_t n, void *out_u8,
                           void *out_fast_u8, void *stream) {
  if (!y || !words || !out_u8 || !out_fast_u8) return NVFP4_ERR_NULL;
  if (n <= 0) return NVFP4_ERR_SHAPE;
  return launch(k_dbg_e2m1_sr, dim3(grid_for(n, 8)), dim3(kThreads),
                static_cast<hipStream_t>(stream), y, words, n, static_cast<uint8_t *>(out_u8),
                static_cast<uint8_t *>(out_fast_u8));
}

int nvfp4_46_debug_philox(const uint32_t *ctr, uint32_t key0, uint32_t key1, int64_t n,
                          uint32_t *out, void *stream) {
  if (!ctr || !out) return NVFP4_ERR_NULL;
  if (n <= 0) return NVFP4_ERR_SHAPE;
  return launch(k_dbg_philox, dim3(grid_for(n, 8)), dim3(kThreads),
                static_cast<hipStream_t>(stream), ctr, key0, key1, n, out);
}

}  // extern "C"

#endif  // NVFP4_46_MAIN

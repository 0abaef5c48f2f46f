// NVFP4 x NVFP4 matrix product for gfx950: C = alpha_a * alpha_b * A . B^T with both operands
// in the quantizer's rowwise layout over the contraction axis (see include/nvfp4_46.h).
//
// gfx950's block-scaled FP4 matrix instructions take one power-of-two scale per 32 values;
// NVFP4 carries an E4M3 scale (three mantissa bits) per 16, so the operands are expanded on
// the way into the matrix unit instead: value(code) * value(scale) has at most six
// significant bits and lies in [2^-10, 2688], hence is exact in FP16, and the FP16 matrix
// instruction (v_mfma_f32_32x32x16_f16, fp32 accumulation) multiplies exact operands.  The
// only rounding is in the fp32 accumulation and in the final scaling.
//
// Data movement: the operands stay packed (4 bits per value) all the way into registers.
// A workgroup of four waves owns a 256 x 256 tile of C, each wave a 128 x 128 quarter
// (4 x 4 matrix-instruction tiles, 256 accumulator registers per lane).  Per chunk of 128
// contraction steps the workgroup copies 256 rows x 64 bytes of codes and 256 x 8 scale
// bytes of each operand into LDS with coalesced loads (the next chunk's loads are in flight
// while the current one is multiplied); a lane then reads 16 bytes (32 codes) per operand
// tile from LDS and expands them with v_cvt_scalef32_pk_f16_fp4 (x 256, exact) and one
// packed FP16 multiplication by the scale (times 2^-8, built from the scale byte by a
// shift).  Which eight contraction indices a lane feeds to a given matrix instruction is
// the same for A and for B, which is all the sum needs.
//
// Two kernels share this plan: k_gemm (the workgroup stages chunks through registers into
// shared LDS buffers; for K > 2^24, beyond the others' 32-bit offsets, and a ragged K where C is too long for a
// launch of smaller tiles) and k_gemm_dma (the workgroup fills a ring of LDS stages with asynchronous
// global -> LDS copies).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "block.hpp"
#include "codec.hpp"
#include "gemm_shapes.hpp"
#include "launch.hpp"
#include "layer.hpp"
#include "nvfp4_46.h"
#include "tensor.hpp"

namespace nvfp4_46 {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Which tile of C a workgroup takes.  Workgroups go to the eight dies in turn and each die has its
// own L2, so the tiles are put in an order -- strips `strip` tiles wide, each row by row -- of
// which every die takes one contiguous eighth: with strip_of() about a square of C, whose operand
// rows are the fewest that its L2 has to fetch.
struct TileAt {
  uint32_t m, n;
};
NV_DEV TileAt tile_of_workgroup(uint32_t tiles_m, uint32_t tiles_n, uint32_t strip) {
  const uint32_t tiles = tiles_m * tiles_n, xcd = blockIdx.x & 7u, seq = blockIdx.x >> 3;
  const uint32_t per = tiles >> 3, extra = tiles & 7u;
  const uint32_t tile = xcd * per + (xcd < extra ? xcd : extra) + seq;
  const uint32_t s = tile / (strip * tiles_m), left = tile - s * strip * tiles_m;
  const uint32_t width = tiles_n - s * strip < strip ? tiles_n - s * strip : strip;
  const uint32_t m = left / width;
  return TileAt{m, s * strip + (left - m * width)};
}

constexpr int kCodeRow = GK / 2 + 16;    // bytes per operand row in LDS: 64 of codes + 16 of padding,
                                         // so that 16 lanes reading 16 bytes from 16 rows hit 16
                                         // different bank groups (80 = 5 * 16, 5 coprime to 16)

// Eight codes (one 32-bit word) times one scale -> eight FP16 values, exactly.
// `sv` is the FP16 with the bit pattern (scale byte << 7), i.e. value(scale) * 2^-8 (also for
// the subnormal scale bytes); the conversion multiplies by 2^8.
NV_DEV h8 expand8(uint32_t word, _Float16 sv) {
  const h2 s = {sv, sv};
  const h2 p0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(word, 256.0f, 0) * s;
  const h2 p1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(word, 256.0f, 1) * s;
  const h2 p2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(word, 256.0f, 2) * s;
  const h2 p3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(word, 256.0f, 3) * s;
  return h8{p0.x, p0.y, p1.x, p1.y, p2.x, p2.y, p3.x, p3.y};
}

// LDS: two buffers (chunk c is multiplied out of one while chunk c + 1 is written into the
// other), each holding both operands' codes and scales.
struct GemmStage {
  uint8_t codes[2][GT * kCodeRow];   // [A, B][row][80]
  uint4 scales[2][GT];               // [A, B][row] -> the row's 8 scales as FP16 bit patterns
                                     // (byte << 7 = value * 2^-8), ready to multiply with
};
constexpr size_t kGemmLdsBytes = 2 * sizeof(GemmStage);

// What a lane holds of one half chunk (64 contraction steps): per operand tile 16 bytes of
// codes and the two scale bytes that go with them.
struct RawHalf {
  uint4 a[4], b[4];
  uint32_t sa[4], sb[4];
};
struct Frags {
  h8 a[4], b[4];
};

// KFULL: K is a multiple of 128, so every chunk is whole and scale rows are 8-byte aligned.
//
// The main loop is a software pipeline over "steps" of 16 contraction indices (8 per chunk):
// while the 16 matrix instructions of step s run, the lane expands the operands of step
// s + 1 (64 vector instructions, issued in the matrix instructions' shadow).  Per chunk:
//   step 1: read the second half's codes and scales from LDS;
//   step 5: write the next chunk (fetched from global memory one chunk earlier) into the
//           other LDS buffer and start fetching the chunk after it;
//   step 6: barrier (every wave has finished reading this buffer and writing the other),
//           then read the next chunk's first half from LDS;
//   step 7: expand the next chunk's first step.
// So the matrix unit is never left waiting for a barrier, an LDS read or an expansion.
template <bool KFULL, bool OUTF32>
__global__ __launch_bounds__(kGemmThreads) void k_gemm(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, int64_t K, uint32_t tiles_n, uint32_t sha,
    uint32_t shb) {
  extern __shared__ __align__(16) uint8_t lds_raw[];
  GemmStage *stage = reinterpret_cast<GemmStage *>(lds_raw);

  const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
  const uint32_t r = lane & 31u, g = lane >> 5;        // row within a 32-row tile, half of K
  const uint32_t wm = wave >> 1, wn = wave & 1u;       // the wave's quarter of the tile
  const uint32_t tile_m = blockIdx.x / tiles_n, tile_n = blockIdx.x - tile_m * tiles_n;
  const int64_t m0 = (int64_t)tile_m * GT, n0 = (int64_t)tile_n * GT;
  const int64_t row_codes = K / 2, row_scales = K / 16;

  // ---- global -> registers -> LDS.  Codes: 1024 16-byte pieces per operand and chunk,
  // four per thread (piece = row * 4 + unit, so four lanes read 64 contiguous bytes);
  // scales: thread t fetches row t's eight bytes.  Rows past the end of an operand re-read
  // its last row (their products are never stored).
  uint4 ga[4], gb[4];
  uint2 gsa, gsb;
  const uint32_t ld_row = t >> 2, ld_unit = t & 3u;
  auto clamp_row = [](int64_t row, int64_t n) { return row < n ? row : n - 1; };
  const uint8_t *pa[4], *pb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    pa[q] = codes_a + clamp_row(m0 + ld_row + 64 * q, M) * row_codes + ld_unit * 16;
    pb[q] = codes_b + clamp_row(n0 + ld_row + 64 * q, N) * row_codes + ld_unit * 16;
  }
  // a row's scale line: the row itself, or row / 16 for an operand quantized in 16x16 tiles
  const uint8_t *psa = scales_a + (clamp_row(m0 + t, M) >> sha) * row_scales;
  const uint8_t *psb = scales_b + (clamp_row(n0 + t, N) >> shb) * row_scales;
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      ga[q] = gb[q] = make_uint4(0, 0, 0, 0);
      if (KFULL || k0 + ld_unit * 32 < K) {
        ga[q] = *reinterpret_cast<const uint4 *>(pa[q] + k0 / 2);
        gb[q] = *reinterpret_cast<const uint4 *>(pb[q] + k0 / 2);
      }
    }
    if (KFULL) {
      gsa = *reinterpret_cast<const uint2 *>(psa + k0 / 16);
      gsb = *reinterpret_cast<const uint2 *>(psb + k0 / 16);
    } else {
      // two scale bytes (32 contraction steps) at a time; K is a multiple of 32
      uint32_t wa[4], wb[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        wa[q] = wb[q] = 0;
        if (k0 + 32 * q < K) {
          wa[q] = *reinterpret_cast<const uint16_t *>(psa + k0 / 16 + 2 * q);
          wb[q] = *reinterpret_cast<const uint16_t *>(psb + k0 / 16 + 2 * q);
        }
      }
      gsa = make_uint2(wa[0] | (wa[1] << 16), wa[2] | (wa[3] << 16));
      gsb = make_uint2(wb[0] | (wb[1] << 16), wb[2] | (wb[3] << 16));
    }
  };
  auto stash = [&](GemmStage &st) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t off = (ld_row + 64 * q) * kCodeRow + ld_unit * 16;
      *reinterpret_cast<uint4 *>(&st.codes[0][off]) = ga[q];
      *reinterpret_cast<uint4 *>(&st.codes[1][off]) = gb[q];
    }
    // scale bytes -> FP16 bit patterns, two per word
    auto widen = [](uint32_t two_bytes) { return ((two_bytes & 0xffu) << 7) | ((two_bytes & 0xff00u) << 15); };
    st.scales[0][t] = make_uint4(widen(gsa.x), widen(gsa.x >> 16), widen(gsa.y), widen(gsa.y >> 16));
    st.scales[1][t] = make_uint4(widen(gsb.x), widen(gsb.x >> 16), widen(gsb.y), widen(gsb.y >> 16));
  };

  // ---- LDS -> registers: 16 bytes (32 codes, two scale blocks) per operand tile and half
  const uint32_t a_row0 = wm * 128 + r, b_row0 = wn * 128 + r;
  auto read_half = [&](const GemmStage &st, int half, RawHalf &h) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t rowa = a_row0 + 32 * i, rowb = b_row0 + 32 * i;
      h.a[i] = *reinterpret_cast<const uint4 *>(&st.codes[0][rowa * kCodeRow + (2 * half + g) * 16]);
      h.b[i] = *reinterpret_cast<const uint4 *>(&st.codes[1][rowb * kCodeRow + (2 * half + g) * 16]);
      // the lane's two scales of this half (blocks 4*half + 2*g and + 1), one word
      const uint32_t *wa = reinterpret_cast<const uint32_t *>(&st.scales[0][rowa]);
      const uint32_t *wb = reinterpret_cast<const uint32_t *>(&st.scales[1][rowb]);
      h.sa[i] = wa[2 * half + g];
      h.sb[i] = wb[2 * half + g];
    }
  };
  // operands of step s (0..3) of a half: word s of the 16 bytes, scale byte s / 2
  auto expand = [&](const RawHalf &h, int s, Frags &f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t wa = s == 0 ? h.a[i].x : s == 1 ? h.a[i].y : s == 2 ? h.a[i].z : h.a[i].w;
      const uint32_t wb = s == 0 ? h.b[i].x : s == 1 ? h.b[i].y : s == 2 ? h.b[i].z : h.b[i].w;
      // the block's scale: low or high half of the pair read from LDS
      const h2 pa2 = __builtin_bit_cast(h2, h.sa[i]), pb2 = __builtin_bit_cast(h2, h.sb[i]);
      f.a[i] = expand8(wa, s < 2 ? pa2.x : pa2.y);
      f.b[i] = expand8(wb, s < 2 ? pb2.x : pb2.y);
    }
  };

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  auto mfma16 = [&](const Frags &f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
  };
  // ask the scheduler to issue four vector instructions behind every matrix instruction, and
  // the step's LDS / global accesses one at a time behind the first matrix instructions
  auto interleave = [&](int lds_reads, int lds_writes, int vmem_reads) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (q < lds_reads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (q < lds_writes) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      if (q < vmem_reads) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
    }
  };

  const int64_t nchunks = (K + GK - 1) / GK;
  RawHalf h0, h1;
  Frags f0, f1;
  fetch(0);
  stash(stage[0]);
  __syncthreads();
  fetch(nchunks > 1 ? GK : 0);
  read_half(stage[0], 0, h0);
  expand(h0, 0, f0);

  // one chunk; `last` = no chunk follows (nothing to write, read or expand ahead)
  auto chunk = [&](int64_t c, bool last) {
    GemmStage &cur = stage[c & 1], &nxt = stage[(c + 1) & 1];
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      Frags &fc = (st & 1) ? f1 : f0, &fn = (st & 1) ? f0 : f1;
      if (st == 1) read_half(cur, 1, h1);
      if (st == 5 && !last) {
        stash(nxt);
        const int64_t c2 = c + 2 < nchunks ? c + 2 : nchunks - 1;   // past the end: a harmless re-read
        fetch(c2 * GK);
      }
      if (st == 6) {
        // keep each step's instructions on their own side of the barrier
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        if (!last) read_half(nxt, 0, h0);
      }
      if (st < 7) expand(st < 3 ? h0 : h1, (st + 1) & 3, fn);
      else if (!last) expand(h0, 0, fn);
      mfma16(fc);
      interleave(st == 1 || (st == 6 && !last) ? 16 : 0, st == 5 && !last ? 10 : 0,
                 st == 5 && !last ? 10 : 0);
    }
  };
  for (int64_t c = 0; c + 1 < nchunks; ++c) chunk(c, false);
  chunk(nchunks - 1, true);

  // ---- epilogue: accumulator element v of tile (i, j) is C[32 i + 8 (v / 4) + 4 g + v % 4]
  // [32 j + r] within the wave's quarter
  const float scale = alpha_a[0] * alpha_b[0];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t col = n0 + wn * 128 + 32 * j + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = m0 + wm * 128 + 32 * i + 8 * (v / 4) + 4 * g + (v % 4);
        if (row < M && col < N) {
          const float c = acc[i][j][v] * scale;
          if (OUTF32)
            static_cast<float *>(out)[row * N + col] = c;
          else
            static_cast<uint16_t *>(out)[row * N + col] = (uint16_t)pack_bf16x2(c, 0.0f);
        }
      }
    }
}

// ----------------------------------------------------------------------------------------
// The same product with LDS filled by asynchronous global -> LDS loads (global_load_lds_dwordx4): no
// staging registers and no LDS write instructions.  Four waves, one per SIMD, hold 4 x 4 instruction tiles
// (128 x 128, 256 accumulators per lane) each and share a tile of C and the contraction axis in one of three ways
// (DmaShape): 256 x 256, 256 x 128 in two halves of K, 128 x 128 in four quarters.  Splitting K inside the
// workgroup keeps the largest wave tile, with the fewest expansions and LDS reads per matrix instruction,
// for products whose 256 x 256 tiles would leave compute units idle.  The waves copy each chunk together into a
// ring of NST stages: codes [BM + BN rows][U units of 16 bytes], then scales.
// A load instruction writes its 64 lanes' 16 (or 4) bytes to consecutive LDS addresses, so
// the LDS layout is plain row-major; to keep the later 16-byte reads of 16 lanes on 16
// different bank groups, position p of a row holds the row's unit p ^ swz(row).
// The copies are issued with inline assembly (the compiler then neither reorders LDS reads
// around them nor waits for all of them at every LDS read) and waited for with explicit
// s_waitcnt vmcnt: the kernel issues no other vector-memory loads inside the loop.
//
// Scales: K whole chunks (KFULL) 4 bytes per lane, U / 2 lanes per row; any other K (a multiple of
// 32) 2 bytes per lane, each pair in a word of its own, which asks nothing of the alignment of scale
// lines.  There the last chunk sticks out of the rows: the lanes past the end of K copy the row's last unit
// instead, and the scales they would meet count as zero.  K <= 2^24 (32-bit lane offsets).
//
// What bounds it: the chip's power for large products (8192 x 8192 x 8192: 778 us, 782 before the store went
// through LDS; builds with parts left out, timing only, of a version that took 788 to 826: 715 without the
// expansions, 690 without the scales' copies either, 655 matrix instructions alone; the vendor's FP16 product
// of the expanded operands 684; 1.7 GHz instead of 2.4).  For the others what comes before and after the loop:
// 1.5 to 2 us until the first chunk is there, 3 to 4 us of sums and stores (single stores of 2 columns straight from
// the accumulators, unrolled 128 times, took 9: one wave per SIMD issues them, cold in the instruction
// cache).  In BF16, us, this / what ran before: 8192 x 8192 x 1056 139 / 152, 4096 x 4096 x 2048 58 / 61,
// 2048 x 4096 x 4096 58 / 69.5, 1000 x 4096 x 4096 33 / 38.
// Expanding each operand once per workgroup into FP16 in LDS, which halves the expansions, takes
// 835 to 854 at 8192 x 8192 x 8192: a quarter more LDS traffic than the matrix instructions leave room for.

// M0 = LDS byte address of lane 0's piece; %1 = the lane's 32-bit byte offset (vector
// register), %2 = the 64-bit base address (scalar register pair).  M0 needs a wait state before a copy reads it.
#define NV_DMA16(lds_sgpr, voff, gbase)                                                       \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                          \
               :: "s"(lds_sgpr), "v"(voff), "s"(gbase) : "memory", "m0")
// as NV_DMA16, two bytes per lane, each into a 32-bit word of LDS
#define NV_DMA2(lds_sgpr, voff, gbase)                                                        \
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ushort %1, %2"                           \
               :: "s"(lds_sgpr), "v"(voff), "s"(gbase) : "memory", "m0")
// a copy by any of the instructions to the LDS address lds_sgpr + lds_imm
#define NV_COPY_TO(insn, lds_sgpr, lds_imm, voff, gbase)                                            \
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\t" insn " %1, %2"                                  \
               :: "s"(lds_sgpr), "v"(voff), "s"(gbase), "n"(lds_imm) : "memory", "m0", "scc")

// f(0), f(1), ..., f(N - 1) with the number as a constant, and the other way round
template <int N, typename F>
NV_DEV void each_number_down(F f) {
  if constexpr (N > 0) {
    f(std::integral_constant<int, N - 1>{});
    each_number_down<N - 1>(f);
  }
}
template <int N, typename F>
NV_DEV void each_number(F f) {
  if constexpr (N > 0) {
    each_number<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

template <typename S, bool KFULL, bool OUTF32>
__global__ __launch_bounds__(S::kThreads, 1) void k_gemm_dma(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, uint32_t K, uint32_t tiles_m, uint32_t tiles_n,
    uint32_t strip, uint32_t sha, uint32_t shb) {
  constexpr int WM = S::WM, WN = S::WN, KS = S::KS, HPW = S::HPW, NST = S::NST, U = S::U, T = S::T, W = S::kWaves;
  constexpr uint32_t STAGE = S::stage(KFULL);
  constexpr int NC = S::NC, NS = S::ns(KFULL), kCopies = NC + NS, STEPS = 4 * HPW;
  typedef uint32_t v4 __attribute__((ext_vector_type(4)));
  typedef float f4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) uint8_t lds_raw[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t r = lane & 31u, g = lane >> 5;
  const uint32_t kg = wave / (S::SM * S::SN), spatial = wave % (S::SM * S::SN);
  const uint32_t wm = spatial / S::SN, wn = spatial % S::SN;

  const TileAt at = tile_of_workgroup(tiles_m, tiles_n, strip);
  const int64_t m0 = (int64_t)at.m * S::BM, n0 = (int64_t)at.n * S::BN;
  const uint32_t row_codes = K / 2, row_scales = K / 16;
  const uint32_t rows_a = (uint32_t)(M - m0 < S::BM ? M - m0 : S::BM);     // rows the tile really has
  const uint32_t rows_b = (uint32_t)(N - n0 < S::BN ? N - n0 : S::BN);

  const float scale = alpha_a[0] * alpha_b[0];
  auto uniform = [](const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
  };
  const uint8_t *gca = uniform(codes_a + m0 * row_codes), *gcb = uniform(codes_b + n0 * row_codes);
  const uint8_t *gsa = uniform(scales_a + (m0 >> sha) * row_scales);
  const uint8_t *gsb = uniform(scales_b + (n0 >> shb) * row_scales);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw;

  auto swz_c = [](uint32_t row) { return (row / (16 / U)) & (U - 1u); };
  auto swz_s = [](uint32_t row) {
    return KFULL ? (U == 8 ? (row >> 4) & 1u : 0u) : ((row / (64 / U)) << 1) & (U - 1u);
  };
  // copies of a wave, numbered: n < NC codes, then scales; 64 / U (128 / U for KFULL's scales) rows each
  constexpr int RC = 64 / U, RS = KFULL ? 128 / U : 64 / U;
  constexpr int AC = S::BM / RC, AS = S::BM / RS;        // instructions that belong to A
  auto of_a = [&](int n) __attribute__((always_inline)) {
    const bool codes = n < NC;
    const int first = (codes ? n : n - NC) * W, cut = codes ? AC : AS;
    return first + W <= cut ? true : first >= cut ? false : first + (int)wave < cut;
  };
  // the lane's byte offset for copy n; units past `last` (the row's last one) give that one instead
  auto offset = [&](int n, uint32_t last) __attribute__((always_inline)) {
    const bool codes = n < NC, is_a = of_a(n);
    const uint32_t i = wave + W * (codes ? n : n - NC);
    const int per = codes ? U : KFULL ? U / 2 : U;       // lanes per row
    const uint32_t row = i * (64 / per) + lane / per, pos = lane % per;
    const uint32_t line = row - (is_a ? 0u : (uint32_t)S::BM), end = (is_a ? rows_a : rows_b) - 1;
    const uint32_t l = line < end ? line : end;
    uint32_t u = codes ? pos ^ swz_c(row) : pos ^ swz_s(row);
    if (!KFULL) u = u < last ? u : last;
    return codes ? l * row_codes + u * 16 : (l >> (is_a ? sha : shb)) * row_scales + u * (KFULL ? 4 : 2);
  };
  const uint32_t nchunks = (K + S::CK - 1) / S::CK;
  uint32_t off[kCopies];
  auto offsets = [&](uint32_t c) __attribute__((always_inline)) {
    const uint32_t left = (K - c * S::CK) / 32 - 1, last = left < U - 1u ? left : U - 1u;
#pragma unroll
    for (int n = 0; n < kCopies; ++n) off[n] = offset(n, last);
  };
  auto copy_one = [&](uint32_t c, uint32_t stage, auto copy) __attribute__((always_inline)) {
    constexpr int n = decltype(copy)::value;
    if constexpr (n < NC) {
      NV_COPY_TO("global_load_lds_dwordx4", lds0 + stage * STAGE + wave * 1024, n * W * 1024, off[n],
                   (of_a(n) ? gca : gcb) + c * (S::CK / 2));
    } else {
      const uint32_t to = lds0 + stage * STAGE + wave * 256;
      const uint8_t *base = (of_a(n) ? gsa : gsb) + c * (S::CK / 16);
      if constexpr (KFULL) NV_COPY_TO("global_load_lds_dword", to, S::kCodes + (n - NC) * W * 256, off[n], base);
      else NV_COPY_TO("global_load_lds_ushort", to, S::kCodes + (n - NC) * W * 256, off[n], base);
    }
  };

  struct Raw {
    v4 c[T];
    uint32_t s[T];
  } x;
  const uint32_t row_a = wm * (32 * WM) + r, row_b = S::BM + wn * (32 * WN) + r;
  auto read_tile = [&](uint32_t stage, int h, int i) __attribute__((always_inline)) {
    const uint32_t u = 2 * (kg * HPW + h) + g;
    const uint8_t *st = lds_raw + stage * STAGE, *sc = st + S::kCodes;
    const uint32_t row = i < WM ? row_a + 32 * i : row_b + 32 * (i - WM);
    x.c[i] = *reinterpret_cast<const v4 *>(st + row * (U * 16) + (u ^ swz_c(r)) * 16);
    x.s[i] = KFULL ? *reinterpret_cast<const uint16_t *>(sc + row * (U * 2) + (u ^ (swz_s(r) << 1)) * 2)
                   : *reinterpret_cast<const uint32_t *>(sc + row * (U * 4) + (u ^ swz_s(r)) * 4);
  };
  // k0: where the wave's piece begins
  auto expand_one = [&](int s, int i, uint32_t k0) __attribute__((always_inline)) {
    if (!KFULL && s == 0 && k0 + 32 * g >= K) x.s[i] = 0u;
    if (s == 0) x.s[i] = __builtin_amdgcn_perm(0u, x.s[i], 0x0c010c00u) << 7;
    const h2 pair = __builtin_bit_cast(h2, x.s[i]);
    return expand8(x.c[i][s], s < 2 ? pair.x : pair.y);
  };

  f32x16 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  // past the end: a harmless re-read, so that the waits below always count the same copies
  auto clamp_chunk = [&](uint32_t c) { return (uint32_t)__builtin_amdgcn_readfirstlane(c < nchunks ? c : nchunks - 1); };
  offsets(0);
#pragma unroll 1
  for (uint32_t p = 0; p < NST - 1; ++p) {
    if (!KFULL && p == nchunks - 1) offsets(p);
    each_number<kCopies>([&](auto copy) __attribute__((always_inline)) { copy_one(clamp_chunk(p), p, copy); });
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((NST - 2) * kCopies) : "memory");
  h8 f[2][T];
#pragma unroll
  for (int i = 0; i < T; ++i) read_tile(0, 0, i);
#pragma unroll
  for (int i = 0; i < T; ++i) f[0][i] = expand_one(0, i, kg * (64 * HPW));

  uint32_t stage = 0, freed = NST - 1;
  // Chunk c sits in stage c % NST.  A step is T units; unit u expands operand tile u for the next step beside its
  // matrix instructions of this one and carries the step's share of LDS reads and copies:
  //   all but the last two steps   start the wave's copies of chunk c + NST - 1, into the stage of chunk c - 1, which
  //                                every wave had read when it came to the barrier of chunk c - 1;
  //   the last step but one        waits until chunk c + 1 has landed and all waves' reads are back, meets the
  //                                other waves, and reads the first piece of chunk c + 1;
  //   step 2 of any other piece    reads the next piece of the chunk.
  // A tile's raw words are read into the registers whose last word has just been expanded.  The last chunk runs
  // the same code (what it reads ahead is not used): a copy of the loop without that cost more, cold in the
  // instruction cache, than it saved.
#pragma unroll 1
  for (uint32_t c = 0; c < nchunks; ++c) {
    const uint32_t nxt = stage + 1 == (uint32_t)NST ? 0u : stage + 1, ahead = c + NST - 1;
    const uint32_t from = clamp_chunk(ahead);
    if (!KFULL && ahead == nchunks - 1) offsets(ahead);
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      const int s = st & 3;
      if (st == STEPS - 2)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((NST - 2) * kCopies) : "memory");
#pragma unroll
      for (int u = 0; u < T; ++u) {
        constexpr int kSlots = (STEPS - 2) * T, kV = (8 * T + S::kTiles - 1) / S::kTiles;
        if (st < STEPS - 2)
          each_number<kCopies>([&](auto copy) __attribute__((always_inline)) {
            if (decltype(copy)::value * kSlots / kCopies == st * T + u) copy_one(from, freed, copy);
          });
        __builtin_amdgcn_sched_barrier(0);
        // expand for the next step, then (its last word gone) read the next piece
        const int h = st / 4;
        const uint32_t k0 = s == 3 ? (h == HPW - 1 ? (c + 1) * S::CK + kg * (64 * HPW) : c * S::CK + kg * (64 * HPW) + (h + 1) * 64) : 0u;
        f[(st + 1) & 1][u] = expand_one((s + 1) & 3, u, k0);
        if (s == 2) read_tile(h == HPW - 1 ? nxt : stage, h == HPW - 1 ? 0 : h + 1, u);
#pragma unroll
        for (int q = u * S::kTiles / T; q < (u + 1) * S::kTiles / T; ++q)
          acc[q / WN][q % WN] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[st & 1][WM + q % WN], f[st & 1][q / WN],
                                                                       acc[q / WN][q % WN], 0, 0, 0);
#pragma unroll
        for (int q = u * S::kTiles / T; q < (u + 1) * S::kTiles / T; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (q & 1) __builtin_amdgcn_sched_group_barrier(0x002, kV + 1, 0);
          else __builtin_amdgcn_sched_group_barrier(0x002, kV, 0);
        }
        if (s == 2) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    freed = stage;
    stage = nxt;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

  // ---- partial sums -> LDS -> C, a block of 32 rows per wave at a time: the operands were exchanged in the matrix
  // instruction, so four accumulator elements are neighbouring columns.  Then G columns (16 bytes) per lane, RPS
  // rows per turn of the workgroup, the KS parts added in order; two blocks in turn, so one barrier each.
  constexpr int G = OUTF32 ? 4 : 8, QG = S::BN / G, RPS = S::kThreads / QG, kRows = 32 * S::SM, E = kRows / RPS;
  static_assert(S::kThreads % QG == 0 && 32 % RPS == 0, "");
  const bool inside = rows_a == S::BM && rows_b == S::BN;
  const int64_t line = N * (OUTF32 ? 4 : 2);
  const uint32_t lr0 = t / QG, col0 = t % QG * G;
  char *const corner = static_cast<char *>(out) + (m0 + lr0) * line + (n0 + col0) * (OUTF32 ? 4 : 2);
#pragma unroll 1
  for (int i = 0; i < WM; ++i) {
    float *buf = reinterpret_cast<float *>(lds_raw + (i & 1) * S::kSums);
    float *to = buf + (kg * kRows + wm * 32 + r) * S::kPitch + wn * (32 * WN) + 4 * g;
#pragma unroll
    for (int ii = 0; ii < WM; ++ii)
      if (i == ii) {
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
          for (int v = 0; v < 16; v += 4)
            *reinterpret_cast<f4 *>(to + 32 * j + 2 * v) = f4{acc[ii][j][v], acc[ii][j][v + 1], acc[ii][j][v + 2], acc[ii][j][v + 3]};
        // (keeps the compiler from merging the blocks' writes behind copies of all 64 registers)
        asm volatile("; row block %0" :: "n"(ii));
      }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    f4 sum[E][G / 4];
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int h = 0; h < G / 4; ++h) {
          const f4 part = *reinterpret_cast<const f4 *>(buf + (k * kRows + e * RPS + lr0) * S::kPitch + col0 + 4 * h);
          sum[e][h] = k == 0 ? part : sum[e][h] + part;
        }
    // (lines of C start wherever N puts them)
    typedef f4 f4_anywhere __attribute__((aligned(4)));
    typedef v4 v4_anywhere __attribute__((aligned(2)));
    auto at_row = [&](int e) __attribute__((always_inline)) {
      return corner + (e * RPS / 32 * (32 * WM) + e * RPS % 32 + 32 * i) * line;
    };
    auto words_of = [&](int e) __attribute__((always_inline)) {
      const f4 x0 = sum[e][0] * scale, x1 = sum[e][G / 4 - 1] * scale;
      return v4{pack_bf16x2(x0.x, x0.y), pack_bf16x2(x0.z, x0.w), pack_bf16x2(x1.x, x1.y), pack_bf16x2(x1.z, x1.w)};
    };
    auto store = [&](int e) __attribute__((always_inline)) {
      if constexpr (OUTF32) *reinterpret_cast<f4_anywhere *>(at_row(e)) = sum[e][0] * scale;
      else *reinterpret_cast<v4_anywhere *>(at_row(e)) = words_of(e);
    };
    if (inside) {
#pragma unroll
      for (int e = 0; e < E; ++e) store(e);
    } else {
      // A tile that sticks out of C: lanes whose columns all exist store as ever.  Only where N is no multiple of G does
      // one lane per line have fewer, `left`, and stores them in pieces of a half, a quarter and an eighth (with a
      // branch for every column of every lane the last tile of a line, and with it the launch, took 3.5 us longer:
      // BF16 2816 x 4088 x 128 16.7 -> 13.2, 2816 x 4096 13.3; fp32 2799 x 3913 x 128 19.6 -> 17.2).
      const uint32_t left = rows_b > col0 ? rows_b - col0 : 0u;
      auto exists = [&](int e) { return e * RPS / 32 * (32 * WM) + e * RPS % 32 + 32 * i + lr0 < rows_a; };
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (left >= G && exists(e)) store(e);
      if (rows_b % G != 0) {
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (left - 1u < G - 1u && exists(e)) {
            typedef uint32_t v2_anywhere __attribute__((ext_vector_type(2), aligned(2)));
            typedef uint32_t word_anywhere __attribute__((aligned(2)));
            v4 w = OUTF32 ? __builtin_bit_cast(v4, sum[e][0] * scale) : words_of(e);
            char *o = at_row(e);
            if (left & (G / 2)) {
              *reinterpret_cast<v2_anywhere *>(o) = v2_anywhere{w.x, w.y};
              o += 8;
              w.x = w.z;
              w.y = w.w;
            }
            if (left & (G / 4)) {
              *reinterpret_cast<word_anywhere *>(o) = w.x;
              o += 4;
              w.x = w.y;
            }
            if (!OUTF32 && (left & 1)) *reinterpret_cast<uint16_t *>(o) = (uint16_t)w.x;
          }
      }
    }
  }
}

// ----------------------------------------------------------------------------------------
// k_gemm_tile: C in tiles of any of several shapes (TileShape), for the many products whose
// large tiles (k_gemm_dma's) would leave compute units idle.  A workgroup has SM x SN waves over its tile of C, each holding WM x WN instruction tiles
// (32 x 32), in KS copies that share the contraction axis: copy kg takes HPW pieces of 64 steps of
// every chunk, and the copies' partial tiles are added through LDS at the end, always in the same
// order.  Splitting the contraction axis inside the workgroup is what fills the chip when C is
// small, without a second pass or a place for partial sums.
//
// What bounds it.  A wave of 2 x 2 instruction tiles issues 8 vector instructions (the
// expansion, 4 cycles each) per matrix instruction (32 cycles): both pipes are equally busy and
// must run at once, which takes several waves per SIMD (the bare loop, no memory accesses: 208
// cycles per 4 matrix instructions with one wave per SIMD, 189 with two, 142 with four; the
// matrix pipe alone 128).  So the small tiles keep to 128 registers, and LDS leaves a compute unit four
// workgroups of Tile32 (eight waves each) and five of Tile64x32, but three of Tile64: its stages
// take 40 KiB, its partial sums 48.  (In two phases the sums fit 36 KiB and four workgroups a unit:
// 1536 x 4096 x 8192 113 -> 110 us, but 128 x 8192 x 2880 14.6 -> 15.4 and 300 x 2000 x 1056 7.7 -> 8.1, for
// the second exchange; not adopted.)  Waves of 4 x 2 expand less per matrix instruction (6 vector
// instructions) and hold 256 registers; they pay only where their larger tiles fill the chip.
//
// Chunks arrive by asynchronous global -> LDS copies, all waves of the workgroup together: codes
// 16 bytes and scale pairs 2 bytes per lane (a pair lands as one 32-bit word), which asks nothing
// of the alignment of scale lines, so K may be any multiple of 32.  Past the end of K a copy
// re-reads the row's last unit and the reader takes its scales as zero (those products are +-0).
// Unit u of LDS row r sits at position u ^ swz(r), so that the 16 (codes) or 64 (pairs) lanes
// of one LDS access pass hit all banks.  One barrier per chunk: it comes after the wait for the
// own copies of the chunk, so behind it the chunk is complete and the stage of the chunk before is
// free for the next copies.  K <= 2^24 (32-bit lane offsets).
//
// Small products spend as long before and after the loop as in it.  So the last chunk stands by itself: no copy
// is under way that the sums would wait for, and a copy of the tile whose piece of it is past K leaves the matrix unit to
// the others.  The sums go through LDS in pieces of 16 bytes, every copy adding up and storing an equal share of
// C (with a wave per 32 x 32 tile seven of Tile32's eight were idle meanwhile), and a tile inside C is stored without
// looking at its edges.  In a replayed graph, us, before / after: 64 x 1024 x 4096 7.1 / 6.4, 128 x 2000 x 1056 5.3 / 4.0,
// 128 x 4096 x 4096 10.3 / 9.1, 300 x 2000 x 1056 7.5 / 6.6, 2880 x 1440 x 1056 20.9 / 18.2, 192 x 4096 x 11008 30.7 / 26.6,
// 1000 x 4096 x 800 14.5 / 12.5; no change where the loop is all (1536 x 4096 x 8192 91).
template <typename S, bool KFULL, bool OUTF32, bool FIRST>
NV_DEV void gemm_tile(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, uint32_t K, uint32_t tiles_m, uint32_t tiles_n,
    uint32_t strip, uint32_t sha, uint32_t shb) {
  constexpr int WM = S::WM, WN = S::WN, KS = S::KS, HPW = S::HPW, NST = S::NST, U = S::U, T = S::T;
  typedef uint32_t v4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) uint8_t lds_raw[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t r = lane & 31u, g = lane >> 5;
  // (workgroups of one compute unit come a launch's turn apart; where K leaves copies without work in the last chunk they
  // differ in which SIMD those are on)
  const uint32_t turn = KFULL ? 0u : blockIdx.x / (uint32_t)kCus;
  const uint32_t kg = (wave / (S::SM * S::SN) + turn) % KS, spatial = wave % (S::SM * S::SN);
  const uint32_t wm = spatial / S::SN, wn = spatial % S::SN;

  const TileAt at = tile_of_workgroup(tiles_m, tiles_n, strip);
  const int64_t m0 = (int64_t)at.m * S::BM, n0 = (int64_t)at.n * S::BN;
  const uint32_t row_codes = K / 2, row_scales = K / 16;
  const uint32_t rows_a = (uint32_t)(M - m0 < S::BM ? M - m0 : S::BM);     // rows the tile really has
  const uint32_t rows_b = (uint32_t)(N - n0 < S::BN ? N - n0 : S::BN);
  const float scale = alpha_a[0] * alpha_b[0];

  auto uniform = [](const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
  };
  const uint8_t *gca = uniform(codes_a + m0 * row_codes), *gcb = uniform(codes_b + n0 * row_codes);
  // the tiles' first scales (FIRST: the 16 bytes that hold them, and how far they are into those)
  const int64_t at_a = (m0 >> sha) * row_scales, at_b = (n0 >> shb) * row_scales;
  const uint32_t into_a = FIRST ? (uint32_t)at_a & 15u : 0u, into_b = FIRST ? (uint32_t)at_b & 15u : 0u;
  const uint8_t *gsa = uniform(scales_a + (at_a - into_a)), *gsb = uniform(scales_b + (at_b - into_b));
  constexpr uint32_t kStage = FIRST ? S::kScaleBase : S::STAGE;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw;

  // 16 / U rows of codes, and 64 / U rows of pairs, fill the 256 bytes of all banks once
  auto swz_c = [](uint32_t row) { return (row / (16 / U)) & (U - 1u); };
  auto swz_s = [](uint32_t row) { return ((row / (64 / U)) << 1) & (U - 1u); };
  // copy instruction i moves the 64 / U LDS rows from i * 64 / U on; wave w issues i = w, w +
  // kWaves, ..., whose rows all have the same swizzle, so a lane copies units unit_c and pairs unit_s only.
  // A row past the end of its operand re-reads the last one (its products are never stored).
  static_assert(S::kCopies % S::kWaves == 0 && 2 * S::kWaves % U == 0, "one swizzle per lane");
  const uint32_t unit_c = lane % U ^ swz_c(wave * (64 / U) + lane / U);
  const uint32_t unit_s = lane % U ^ swz_s(wave * (64 / U) + lane / U);
  constexpr bool PIECES = KFULL && S::kPieces;            // scales 16 bytes per lane: P such pieces to a row and chunk
  constexpr int P = PIECES ? S::kPieces : 1;
  uint32_t off_c[S::NC], off_s[PIECES || FIRST ? 1 : S::NC];       // the lane's byte offsets at chunk 0
#pragma unroll
  for (int n = 0; n < S::NC; ++n) {
    const uint32_t i = wave + n * S::kWaves;
    const uint32_t row = i * (64 / U) + lane / U;
    const bool is_a = i * (64 / U) < (uint32_t)S::BM;
    const uint32_t line = row - (is_a ? 0u : (uint32_t)S::BM), last = (is_a ? rows_a : rows_b) - 1;
    const uint32_t l = line < last ? line : last;
    off_c[n] = l * row_codes + unit_c * 16;
    if constexpr (!PIECES && !FIRST) off_s[n] = (l >> (is_a ? sha : shb)) * row_scales + unit_s * 2;
  }
  // one copy instruction of each of the first kScaleCopies waves
  constexpr uint32_t kScaleCopiesA = S::BM * P / 64, kScaleCopies = S::ROWS * P / 64;
  const bool scales_of_a = wave < kScaleCopiesA;
  if constexpr (PIECES) {
    static_assert(S::BM * P % 64 == 0 && S::BN * P % 64 == 0 && kScaleCopies <= S::kWaves, "copies of one operand each");
    const uint32_t piece = (scales_of_a ? wave : wave - kScaleCopiesA) * 64 + lane, row = piece / P;
    const uint32_t last = (scales_of_a ? rows_a : rows_b) - 1, l = row < last ? row : last;
    off_s[0] = (l >> (scales_of_a ? sha : shb)) * row_scales + piece % P * 16;
  }
  auto copy_chunk = [&](uint32_t c, uint32_t stage) {
    const uint32_t lds = lds0 + stage * kStage;
    const uint32_t k0 = c * S::CK;
    // units past the end of K: the row's last one instead
    uint32_t past_c = 0, past_s = 0;
    if constexpr (!KFULL) {
      const uint32_t kc = k0 + unit_c * 32, ks = k0 + unit_s * 32;
      past_c = kc >= K ? (kc - (K - 32)) / 2 : 0u;
      past_s = ks >= K ? (ks - (K - 32)) / 16 : 0u;
    }
#pragma unroll
    for (int n = 0; n < S::NC; ++n) {
      const uint32_t i = wave + n * S::kWaves;
      const bool is_a = i * (64 / U) < (uint32_t)S::BM;
      const uint8_t *bc = (is_a ? gca : gcb) + k0 / 2, *bs = (is_a ? gsa : gsb) + k0 / 16;
      NV_DMA16(lds + i * 1024, off_c[n] - past_c, bc);
      if constexpr (!PIECES && !FIRST) NV_DMA2(lds + S::kScaleBase + i * 256, off_s[n] - past_s, bs);
    }
    if constexpr (PIECES)
      if (wave < kScaleCopies)
        NV_DMA16(lds + S::kScaleBase + wave * 1024, off_s[0], (scales_of_a ? gsa : gsb) + k0 / 16);
  };

  // FIRST: all scales of a tile, whose lines follow each other in memory, to LDS behind the stages
  const uint32_t first_a = NST * kStage, first_b = first_a + S::first_scales(S::BM, row_scales);
  auto copy_scales = [&](const uint8_t *from, uint32_t bytes, uint32_t to) {
    for (uint32_t i = wave * 1024; i < bytes; i += S::kWaves * 1024) {
      const uint32_t off = i + lane * 16;
      if (off + 16 <= bytes) {
        NV_DMA16(lds0 + to + i, off, from);
      } else {
        // an edge of C, in the middle of 16 bytes
        uint16_t last[7];
        auto place = [&](int j) { return off + 2 * j < bytes - 2 ? off + 2 * j : bytes - 2; };
        if (off < bytes) {
#pragma unroll
          for (int j = 0; j < 7; ++j) last[j] = *reinterpret_cast<const uint16_t *>(from + place(j));
#pragma unroll
          for (int j = 0; j < 7; ++j) *reinterpret_cast<uint16_t *>(lds_raw + to + place(j)) = last[j];
        }
      }
    }
  };
  // a lane's share of one piece: 32 codes and their two scales per operand tile (WM of A, WN of B)
  struct Raw {
    v4 c[T];
    uint32_t s[T];
  };
  const uint32_t row_a = wm * (32 * WM) + r, row_b = S::BM + wn * (32 * WN) + r;
  const uint32_t line_a = first_a + into_a + (row_a >> sha) * row_scales;
  const uint32_t line_b = first_b + into_b + ((row_b - S::BM) >> shb) * row_scales;
  auto read_piece = [&](uint32_t c, uint32_t stage, uint32_t h, Raw &x) {
    const uint32_t u = 2 * (kg * HPW + h) + g;
    const uint8_t *st = lds_raw + stage * kStage;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const uint32_t row = i < WM ? row_a + 32 * i : row_b + 32 * (i - WM);
      x.c[i] = *reinterpret_cast<const v4 *>(st + row * (U * 16) + (u ^ swz_c(r)) * 16);
      if constexpr (FIRST) {
        const uint32_t line = i < WM ? line_a + (32 * i >> sha) * row_scales : line_b + (32 * (i - WM) >> shb) * row_scales;
        x.s[i] = *reinterpret_cast<const uint16_t *>(lds_raw + line + (c * U + u) * 2);
      } else if constexpr (PIECES)
        x.s[i] = *reinterpret_cast<const uint16_t *>(st + S::kScaleBase + row * (16 * P) + u * 2);
      else
        x.s[i] = *reinterpret_cast<const uint32_t *>(st + S::kScaleBase + row * (U * 4) + (u ^ swz_s(r)) * 4);
    }
    if constexpr (!KFULL) {
      const uint32_t keep = c * S::CK + u * 32 < K ? 0xffffffffu : 0u;
#pragma unroll
      for (int i = 0; i < T; ++i) x.s[i] &= keep;
    }
  };
  auto expand_one = [&](Raw &x, int s, int i) {
    if (s == 0) x.s[i] = __builtin_amdgcn_perm(0u, x.s[i], 0x0c010c00u) << 7;
    const h2 pair = __builtin_bit_cast(h2, x.s[i]);
    return expand8(x.c[i][s], s < 2 ? pair.x : pair.y);
  };

  f32x16 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

  const uint32_t nchunks = (K + S::CK - 1) / S::CK;
  auto clamp_chunk = [&](uint32_t c) { return c < nchunks ? c : nchunks - 1; };
  if constexpr (S::kTiles <= 4) {
    // four waves per SIMD hide each other's LDS reads and expansions: plain order, few registers
    static_assert(S::kTiles > 4 || NST == 2, "every copy on its way belongs to the chunk that is waited for");
    auto multiply_piece = [&](uint32_t c, uint32_t stage, int h) {
      Raw x;
      read_piece(c, stage, h, x);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        h8 f[T];
#pragma unroll
        for (int i = 0; i < T; ++i) f[i] = expand_one(x, s, i);
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
          for (int j = 0; j < WN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[i], f[WM + j], acc[i][j], 0, 0, 0);
      }
    };
    copy_chunk(0, 0);
    if constexpr (FIRST) {
      copy_scales(gsa, into_a + (((rows_a - 1) >> sha) + 1) * row_scales, first_a);
      copy_scales(gsb, into_b + (((rows_b - 1) >> shb) + 1) * row_scales, first_b);
    }
    // chunk c is complete, and nobody reads the other stage, chunk c - 1's, any more
    auto wait_for_chunk = [] { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    for (uint32_t c = 0; c + 1 < nchunks; ++c) {
      wait_for_chunk();
      copy_chunk(c + 1, (c + 1) & 1);
#pragma unroll
      for (int h = 0; h < HPW; ++h) multiply_piece(c, c & 1, h);
    }
    // the last chunk by itself: no copy, which the sums would wait for, and nothing for copies whose pieces are past K
    wait_for_chunk();
#pragma unroll
    for (int h = 0; h < HPW; ++h)
      if (KFULL || (nchunks - 1) * S::CK + 64 * (kg * HPW + h) < K) multiply_piece(nchunks - 1, (nchunks - 1) & 1, h);
  } else {
#pragma unroll
    for (int p = 0; p < NST; ++p) copy_chunk(clamp_chunk(p), p);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((NST - 1) * 2 * S::NC) : "memory");
    // two waves per SIMD: a software pipeline over steps of 16 contraction indices, the next step's
    // operands expanded in the shadow of this step's matrix instructions
    Raw x, xn;
    h8 f[2][T];
    read_piece(0, 0, 0, x);
#pragma unroll
    for (int i = 0; i < T; ++i) f[0][i] = expand_one(x, 0, i);

    uint32_t stage = 0;
    for (uint32_t c = 0; c < nchunks; ++c) {
      const uint32_t nxt = stage + 1 == (uint32_t)NST ? 0u : stage + 1;
#pragma unroll
      for (int h = 0; h < HPW; ++h) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const bool sync = s == 2 && h == HPW - 1;
          if (s == 1 && h < HPW - 1) read_piece(c, stage, h + 1, xn);
          if (sync) {
            // every wave's reads of this stage are done and chunk c + 1 is complete
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((NST - 2) * 2 * S::NC) : "memory");
            read_piece(clamp_chunk(c + 1), nxt, 0, xn);
            copy_chunk(clamp_chunk(c + NST), stage);
            __builtin_amdgcn_sched_barrier(0);
          }
          Raw &src = s == 3 ? xn : x;
#pragma unroll
          for (int i = 0; i < T; ++i) f[(s + 1) & 1][i] = expand_one(src, (s + 1) & 3, i);
          if (s == 3) x = xn;
#pragma unroll
          for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[s & 1][i], f[s & 1][WM + j], acc[i][j], 0, 0, 0);
          constexpr int kV = (8 * T + S::kTiles - 1) / S::kTiles + 1;
#pragma unroll
          for (int q = 0; q < S::kTiles; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, kV, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      stage = nxt;
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");       // nothing may still be writing LDS

  // The copies' partial tiles, VW accumulators of a lane at a time: unit u belongs to copy u % KS, which adds the other
  // copies' to its own, in an order that depends on the tile only, and stores the sum.
  constexpr int VW = S::VW, kUnits = 16 / VW;
  typedef float Sums __attribute__((ext_vector_type(VW)));
  typedef Sums Part[kUnits][KS > 1 ? KS - 1 : 1][S::SM * S::SN][64];
  Part *part = reinterpret_cast<Part *>(lds_raw);
  auto sums_of = [&](int u) {
    Sums x;
#pragma unroll
    for (int i = 0; i < VW; ++i) x[i] = acc[u / kUnits / WN][u / kUnits % WN][u % kUnits * VW + i];
    return x;
  };
  typedef std::conditional_t<OUTF32, float, uint16_t> Out;
  const uint32_t row0 = wm * (32 * WM) + 4 * g, col0 = wn * (32 * WN) + r;
  Out *const c00 = static_cast<Out *>(out) + (m0 + row0) * N + n0 + col0;
  const bool whole = rows_a == (uint32_t)S::BM && rows_b == (uint32_t)S::BN;
#pragma unroll
  for (int e0 = 0; e0 < S::kTiles; e0 += S::PER) {
    constexpr int kLast = S::kTiles * kUnits;
    const int u0 = e0 * kUnits, u1 = u0 + S::PER * kUnits < kLast ? u0 + S::PER * kUnits : kLast;
    if (e0 > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    each_number<KS>([&](auto number) {
      constexpr int self = decltype(number)::value;
      if (kg != (uint32_t)self) return;
#pragma unroll
      for (int u = u0; u < u1; ++u)
        if (u % KS != self)
          part[(u - u0) / kUnits][u % kUnits][self - (self > u % KS ? 1 : 0)][spatial][lane] = sums_of(u);
    });
    if (KS > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    Sums sum[S::PER * kUnits / KS];
    each_number<KS>([&](auto number) {
      constexpr int self = decltype(number)::value;
      if (kg != (uint32_t)self) return;
#pragma unroll
      for (int u = u0 + self; u < u1; u += KS) {
        auto sums_from = [&](int copy) {
          return copy == self ? sums_of(u)
                              : part[(u - u0) / kUnits][u % kUnits][copy - (copy > self ? 1 : 0)][spatial][lane];
        };
        const int first = u / kUnits / S::kOwn;
        Sums x = sums_from(first);
#pragma unroll
        for (int copy = 0; copy < KS; ++copy)
          if (copy != first) x += sums_from(copy);
        sum[(u - u0) / KS] = x;
      }
    });
    auto store = [&](bool check) {
#pragma unroll
      for (int j = 0; j < (u1 - u0) / KS; ++j) {
        const uint32_t u = u0 + j * KS + kg, e = u / kUnits, v = u % kUnits * VW;
        const uint32_t row = 32 * (e / WN) + 8 * (v / 4) + v % 4, col = 32 * (e % WN);
#pragma unroll
        for (int i = 0; i < VW; ++i) {
          if (check && !(row0 + row + i < rows_a && col0 + col < rows_b)) continue;
          const float c = sum[j][i] * scale;
          Out *const at = c00 + (int64_t)(row + i) * N + col;
          if constexpr (OUTF32)
            *at = c;
          else
            *at = (uint16_t)pack_bf16x2(c, 0.0f);
        }
      }
    };
    if (whole)
      store(false);
    else
      store(true);
  }
}

template <typename S, bool KFULL, bool OUTF32>
__global__ __launch_bounds__(S::kThreads, S::kTiles > 8 ? 1 : S::kTiles > 4 ? 2 : 4) void k_gemm_tile(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, uint32_t K, uint32_t tiles_m, uint32_t tiles_n,
    uint32_t strip, uint32_t sha, uint32_t shb) {
  gemm_tile<S, KFULL, OUTF32, false>(
      codes_a, scales_a, alpha_a, codes_b, scales_b, alpha_b, out, M, N, K, tiles_m, tiles_n, strip,
      sha, shb);
}

// The same with all scales copied before the first chunk: S::scales_first() (125 registers).
template <typename S, bool OUTF32>
__global__ __launch_bounds__(S::kThreads, S::kTiles > 8 ? 1 : S::kTiles > 4 ? 2 : 4) void k_gemm_scales_first(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, uint32_t K, uint32_t tiles_m, uint32_t tiles_n,
    uint32_t strip, uint32_t sha, uint32_t shb) {
  gemm_tile<S, false, OUTF32, true>(
      codes_a, scales_a, alpha_a, codes_b, scales_b, alpha_b, out, M, N, K, tiles_m, tiles_n, strip,
      sha, shb);
}

// ----------------------------------------------------------------------------------------
// Few rows of A (a small batch of activations against a weight matrix; the entry point says
// how few).  The product
// is then bound by reading B once from HBM -- which is where four-bit operands pay on this
// chip: 0.5625 bytes per weight instead of 2 -- so the plan changes: every workgroup owns 32
// rows of B (32 columns of C) and all of A, and its waves split the contraction axis (wave w
// takes the chunks of 256 indices with chunk % waves == w); the partial tiles are added
// through LDS at the end in a fixed order.  A is re-read by every workgroup, but it is small
// and stays in L2.
//
// The matrix instruction wants one operand row per lane, but a load instruction whose 64
// lanes address 32 different rows is 64 separate 16-byte requests, and the kernel would be
// bound by their number.  So each wave copies its chunk with asynchronous global -> LDS loads
// in which eight neighbouring lanes fetch the 128 contiguous bytes of one row, into its own
// piece of LDS, and then reads it back a row per lane (16-byte unit u of a row sits at
// position u ^ ((row >> 1) & 7), which spreads 16 rows over 16 bank groups).  With one tile of
// A there is room for two such pieces per wave and the copy of the chunk after next runs
// while a chunk is multiplied; otherwise the next chunk's copy overlaps this chunk's
// arithmetic and the other waves' work.
// MT = number of 32-row tiles of A (1 or 2).  K must be a multiple of 256 and <= 2^24.
// Waves per workgroup and staging pieces per wave, for 1 and 2 tiles of A.  Four waves were
// fastest on every weight shape timed (8192 x 8192, 28672 x 8192, 8192 x 28672, 4096 x 4096;
// 2 to 10 waves and 1 to 4 pieces were tried): with one tile of A the workgroup then needs
// 72 KiB of LDS and two of them share a compute unit, so one's start and end overlap the
// other's stream.
constexpr int kSkinnyShape[2][2] = {{4, 2}, {4, 1}};
constexpr int skinny_waves(int mt) { return kSkinnyShape[mt - 1][0]; }
constexpr int skinny_stages(int mt) { return kSkinnyShape[mt - 1][1]; }
constexpr uint32_t skinny_rows(int mt) { return 32u + 32u * mt; }        // B rows, then A rows
constexpr uint32_t skinny_scale_rows(int mt) { return (skinny_rows(mt) + 63u) / 64u * 64u; }
constexpr uint32_t skinny_stage_bytes(int mt) {
  return skinny_rows(mt) * 128u + skinny_scale_rows(mt) * 16u;
}
constexpr size_t skinny_lds_bytes(int mt) {
  const size_t stages = (size_t)skinny_waves(mt) * skinny_stages(mt) * skinny_stage_bytes(mt);
  const size_t partials = (size_t)(skinny_waves(mt) - 1) * mt * 16 * 64 * sizeof(float);
  return stages > partials ? stages : partials;
}

static_assert(64 * skinny_waves(1) == kGemmThreads && 64 * skinny_waves(2) == kGemmThreads, "lanes_of");
static_assert(skinny_lds_bytes(1) <= 160 * 1024 && skinny_lds_bytes(2) <= 160 * 1024,
              "the stages must fit the LDS");

template <int MT, bool OUTF32>
__global__ __launch_bounds__(64 * skinny_waves(MT)) void k_gemm_skinny(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, int64_t K, uint32_t sha, uint32_t shb) {
  constexpr int W = skinny_waves(MT), NST = skinny_stages(MT);
  constexpr uint32_t ROWS = skinny_rows(MT), STAGE = skinny_stage_bytes(MT);
  constexpr int NC = ROWS / 8, NS = skinny_scale_rows(MT) / 64;   // copy instructions per chunk
  extern __shared__ __align__(16) uint8_t lds_raw[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t r = lane & 31u, g = lane >> 5;
  const int64_t n0 = (int64_t)blockIdx.x * 32;
  const int64_t row_codes = K / 2, row_scales = K / 16;
  const uint8_t *wl = lds_raw + wave * (NST * STAGE);
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw +
                            wave * (NST * STAGE);

  // ---- copy instructions.  Codes: instruction q moves rows 8q .. 8q+7 of the stage, lane l
  // the 16-byte unit (l & 7) ^ ((row >> 1) & 7) of row 8q + l / 8; rows 0-31 are B's, the rest
  // A's (rows past the end of an operand re-read its last row).  Scales: one lane per row.
  auto uniform = [](const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
  };
  const int64_t b_base = n0 < N ? n0 : N - 1;
  const uint8_t *gcb = uniform(codes_b + b_base * row_codes), *gca = uniform(codes_a);
  uint32_t oc[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const uint32_t row = 8 * q + (lane >> 3), unit = (lane & 7u) ^ ((row >> 1) & 7u);
    int64_t line;
    if (q < 4) line = b_base + row < N ? row : N - 1 - b_base;       // relative to b_base
    else line = (int64_t)(row - 32) < M ? row - 32 : M - 1;
    oc[q] = (uint32_t)(line * row_codes) + unit * 16;
  }
  const uint8_t *ps[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const uint32_t row = 64 * j + lane;
    if (row < 32) {
      const int64_t n = n0 + row < N ? n0 + row : N - 1;
      ps[j] = scales_b + (n >> shb) * row_scales;
    } else {
      const int64_t m = (int64_t)(row - 32) < M ? row - 32 : M - 1;
      ps[j] = scales_a + (m >> sha) * row_scales;
    }
  }
  auto copy_chunk = [&](int64_t c, uint32_t stage) {
    const uint32_t lds = lds_wave + stage * STAGE;
    const uint8_t *pb = gcb + c * (SK / 2), *pa = gca + c * (SK / 2);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      if (q < 4) NV_DMA16(lds + q * 1024, oc[q], pb);
      else NV_DMA16(lds + q * 1024, oc[q], pa);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const uint8_t *src = ps[j] + c * (SK / 16);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :: "s"(lds + ROWS * 128 + j * 1024), "v"(src) : "memory", "m0");
    }
  };
  constexpr int kCopies = NC + NS;

  // one chunk of one operand row as the lane holds it: 128 codes and their 8 scales, the
  // scales already as FP16 bit patterns (byte << 7), two per word
  struct Raw {
    uint4 c[4];
    uint32_t s[4];
  };
  const uint32_t swz = (r >> 1) & 7u;
  auto read_tile = [&](uint32_t stage, int u, Raw &x) {             // u = 0: B, 1..MT: tiles of A
    const uint8_t *st = wl + stage * STAGE;
    const uint32_t row = 32 * u + r;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      x.c[q] = *reinterpret_cast<const uint4 *>(st + row * 128 + (((4 * g + q) ^ swz) * 16));
    const uint2 sc = *reinterpret_cast<const uint2 *>(st + ROWS * 128 + row * 16 + 8 * g);
    x.s[0] = __builtin_amdgcn_perm(0u, sc.x, 0x0c010c00u) << 7;
    x.s[1] = __builtin_amdgcn_perm(0u, sc.x, 0x0c030c02u) << 7;
    x.s[2] = __builtin_amdgcn_perm(0u, sc.y, 0x0c010c00u) << 7;
    x.s[3] = __builtin_amdgcn_perm(0u, sc.y, 0x0c030c02u) << 7;
  };
  // the eight codes of matrix step s (0..15) of the chunk, expanded with their block's scale
  auto expand = [&](const Raw &x, int s) {
    const uint4 &q = x.c[s >> 2];
    const uint32_t w = (s & 3) == 0 ? q.x : (s & 3) == 1 ? q.y : (s & 3) == 2 ? q.z : q.w;
    const h2 pair = __builtin_bit_cast(h2, x.s[s >> 2]);          // blocks 2 (s / 4) and + 1
    return expand8(w, (s & 2) ? pair.y : pair.x);                  // block s / 2 of the lane's eight
  };

  f32x16 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;

  // The wave's chunks are wave, wave + W, ...  Copies are counted by hand (the kernel issues no
  // other vector-memory loads in the loop): before a stage is read, all but the copies
  // issued after it must have landed; before a stage is overwritten, its reads must be back.
  const int64_t nchunks = K / SK;
  int64_t c = wave;
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (c + W * p < nchunks) copy_chunk(c + W * p, p);
  uint32_t stage = 0;
  auto chunk = [&](auto after) {
    Raw rb, ra[MT];
    read_tile(stage, 0, rb);
#pragma unroll
    for (int i = 0; i < MT; ++i) read_tile(stage, 1 + i, ra[i]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    after();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const h8 fb = expand(rb, s);
#pragma unroll
      for (int i = 0; i < MT; ++i)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(expand(ra[i], s), fb, acc[i], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    c += W;
    stage = stage + 1 == (uint32_t)NST ? 0u : stage + 1;
  };
  while (c + W * NST < nchunks) {
    // all but the copies of the NST - 1 younger stages must have landed
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 1) * kCopies) : "memory");
    chunk([&] { copy_chunk(c + W * NST, stage); });
  }
  // the last NST chunks, with nothing left to copy (re-reading the last chunk instead, a quarter more copies at
  // K = 8192: 1 x 8192 x 8192 9.3 -> 9.0 us, 16 x 8192 x 8192 9.6 -> 9.2, 16 x 28672 x 8192 from memory 33.5 -> 31.9)
  each_number_down<NST>([&](auto p) {
    if (c + W * decltype(p)::value < nchunks) {
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"(decltype(p)::value * kCopies) : "memory");
      chunk([] {});
    }
  });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing may still be writing LDS
  __syncthreads();                                       // ... of any wave: the stages are reused

  // ---- add the waves' tiles in a fixed order (wave 0 collects), scale, store
  float (*part)[MT][16][64] = reinterpret_cast<float (*)[MT][16][64]>(lds_raw);
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) part[wave - 1][i][v][lane] = acc[i][v];
  }
  __syncthreads();
  if (wave == 0) {
    const float scale = alpha_a[0] * alpha_b[0];
    const int64_t col = n0 + r;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float sum = acc[i][v];
#pragma unroll
        for (int w = 0; w < W - 1; ++w) sum += part[w][i][v][lane];
        const int64_t row = 32 * i + 8 * (v / 4) + 4 * g + (v % 4);
        if (row < M && col < N) {
          const float cval = sum * scale;
          if (OUTF32)
            static_cast<float *>(out)[row * N + col] = cval;
          else
            static_cast<uint16_t *>(out)[row * N + col] = (uint16_t)pack_bf16x2(cval, 0.0f);
        }
      }
  }
}

// ----------------------------------------------------------------------------------------
// At most 16 rows of A (a decoding batch): the same plan with the 16x16x32 matrix instruction.
// A's tile is 16 rows, so half as much of A is copied, read back and expanded per workgroup,
// and the two 16-column halves of the workgroup's 32 columns of C share each expanded
// fragment of A; per 32 contraction indices a wave issues three expansions and two 4-pass
// matrix instructions where the 32-row plan issues four and two 8-pass ones.
//
// Stage layout per wave: rows 0-31 B, rows 32-47 A (128 code bytes each, 16-byte units
// swizzled as above), then 64 scale lines of 16 bytes (lines 48-63 repeat A's last row).
// Lane l holds row l % 16 of a tile and the 64 codes 64 g .. 64 g + 63 of the chunk,
// g = l / 16 (two 16-byte units); matrix step s (0..7) multiplies codes 64 g + 8 s .. + 7 of
// every lane group, the same for A and B, so which contraction indices meet in one
// instruction is again a permutation shared by both operands.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kSkinny16Rows = 48, kSkinny16Stage = kSkinny16Rows * 128 + 64 * 16;   // 7168
constexpr int kSkinny16Waves = 4, kSkinny16Stages = 2;
constexpr size_t kSkinny16LdsBytes = (size_t)kSkinny16Waves * kSkinny16Stages * kSkinny16Stage;
static_assert(64 * kSkinny16Waves == kGemmThreads, "lanes_of");
static_assert(kSkinny16LdsBytes <= 160 * 1024 && kSkinny16Stages >= 1, "stages must fit the LDS");
static_assert((size_t)(kSkinny16Waves - 1) * 2 * 4 * 64 * sizeof(float) <= kSkinny16LdsBytes,
              "the partial sums reuse the stages");

template <bool OUTF32>
__global__ __launch_bounds__(64 * kSkinny16Waves) void k_gemm_skinny16(
    const uint8_t *__restrict__ codes_a, const uint8_t *__restrict__ scales_a,
    const float *__restrict__ alpha_a, const uint8_t *__restrict__ codes_b,
    const uint8_t *__restrict__ scales_b, const float *__restrict__ alpha_b,
    void *__restrict__ out, int64_t M, int64_t N, int64_t K, uint32_t sha, uint32_t shb) {
  constexpr int W = kSkinny16Waves, NST = kSkinny16Stages;
  constexpr uint32_t ROWS = kSkinny16Rows, STAGE = kSkinny16Stage;
  constexpr int NC = ROWS / 8;                                     // code copies per chunk
  extern __shared__ __align__(16) uint8_t lds_raw[];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t rr = lane & 15u, g = lane >> 4;
  const int64_t n0 = (int64_t)blockIdx.x * 32;
  const int64_t row_codes = K / 2, row_scales = K / 16;
  const uint8_t *wl = lds_raw + wave * (NST * STAGE);
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw +
                            wave * (NST * STAGE);

  auto uniform = [](const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
  };
  const int64_t b_base = n0 < N ? n0 : N - 1;
  const uint8_t *gcb = uniform(codes_b + b_base * row_codes), *gca = uniform(codes_a);
  uint32_t oc[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const uint32_t row = 8 * q + (lane >> 3), unit = (lane & 7u) ^ ((row >> 1) & 7u);
    int64_t line;
    if (q < 4) line = b_base + row < N ? row : N - 1 - b_base;       // relative to b_base
    else line = (int64_t)(row - 32) < M ? row - 32 : M - 1;
    oc[q] = (uint32_t)(line * row_codes) + unit * 16;
  }
  const uint8_t *ps;
  if (lane < 32) {
    const int64_t n = n0 + lane < N ? n0 + lane : N - 1;
    ps = scales_b + (n >> shb) * row_scales;
  } else {
    const int64_t m = (int64_t)(lane - 32) < M ? lane - 32 : M - 1;
    ps = scales_a + (m >> sha) * row_scales;
  }
  auto copy_chunk = [&](int64_t c, uint32_t stage) {
    const uint32_t lds = lds_wave + stage * STAGE;
    const uint8_t *pb = gcb + c * (SK / 2), *pa = gca + c * (SK / 2);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      if (q < 4) NV_DMA16(lds + q * 1024, oc[q], pb);
      else NV_DMA16(lds + q * 1024, oc[q], pa);
    }
    const uint8_t *src = ps + c * (SK / 16);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :: "s"(lds + ROWS * 128), "v"(src) : "memory", "m0");
  };
  constexpr int kCopies = NC + 1;

  // a lane's share of one operand row for one chunk: 64 codes and the scales of their four
  // blocks as FP16 bit patterns (byte << 7), two per word
  struct Raw {
    uint4 c[2];
    uint32_t s[2];
  };
  auto read_tile = [&](uint32_t stage, uint32_t first_row, Raw &x) {
    const uint8_t *st = wl + stage * STAGE;
    const uint32_t row = first_row + rr, swz = (row >> 1) & 7u;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      x.c[q] = *reinterpret_cast<const uint4 *>(st + row * 128 + (((2 * g + q) ^ swz) * 16));
    const uint32_t sc = *reinterpret_cast<const uint32_t *>(st + ROWS * 128 + row * 16 + 4 * g);
    x.s[0] = __builtin_amdgcn_perm(0u, sc, 0x0c010c00u) << 7;
    x.s[1] = __builtin_amdgcn_perm(0u, sc, 0x0c030c02u) << 7;
  };
  auto expand = [&](const Raw &x, int s) {                         // matrix step s = 0..7
    const uint4 &q = x.c[s >> 2];
    const uint32_t w = (s & 3) == 0 ? q.x : (s & 3) == 1 ? q.y : (s & 3) == 2 ? q.z : q.w;
    const h2 pair = __builtin_bit_cast(h2, x.s[s >> 2]);            // blocks 4 g + 2 (s / 4), + 1
    return expand8(w, (s & 2) ? pair.y : pair.x);                    // block 4 g + s / 2
  };

  f32x4 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[j][v] = 0.0f;

  const int64_t nchunks = K / SK;
  int64_t c = wave;
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (c + W * p < nchunks) copy_chunk(c + W * p, p);
  uint32_t stage = 0;
  auto chunk = [&](auto after) {
    Raw ra, rb[2];
    read_tile(stage, 32, ra);
    read_tile(stage, 0, rb[0]);
    read_tile(stage, 16, rb[1]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    after();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const h8 fa = expand(ra, s);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, expand(rb[j], s), acc[j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    c += W;
    stage = stage + 1 == (uint32_t)NST ? 0u : stage + 1;
  };
  while (c + W * NST < nchunks) {
    // all but the copies of the NST - 1 younger stages must have landed
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 1) * kCopies) : "memory");
    chunk([&] { copy_chunk(c + W * NST, stage); });
  }
  // the last NST chunks, with nothing left to copy
  each_number_down<NST>([&](auto p) {
    if (c + W * decltype(p)::value < nchunks) {
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"(decltype(p)::value * kCopies) : "memory");
      chunk([] {});
    }
  });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing may still be writing LDS
  __syncthreads();                                       // ... of any wave: the stages are reused

  // ---- add the waves' tiles in a fixed order (wave 0 collects), scale, store
  float (*part)[2][4][64] = reinterpret_cast<float (*)[2][4][64]>(lds_raw);
  if (wave > 0) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave - 1][j][v][lane] = acc[j][v];
  }
  __syncthreads();
  if (wave == 0) {
    const float scale = alpha_a[0] * alpha_b[0];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float sum = acc[j][v];
#pragma unroll
        for (int w = 0; w < W - 1; ++w) sum += part[w][j][v][lane];
        const int64_t row = 4 * g + v, col = n0 + 16 * j + rr;
        if (row < M && col < N) {
          const float cval = sum * scale;
          if (OUTF32)
            static_cast<float *>(out)[row * N + col] = cval;
          else
            static_cast<uint16_t *>(out)[row * N + col] = (uint16_t)pack_bf16x2(cval, 0.0f);
        }
      }
  }
}

// ----------------------------------------------------------------------------------------
// Few values of x against a quantized weight, in one launch: tensor scale, rowwise round-to-nearest 4/6
// codes and the product, for at most 16 rows (FewRows says how many values).  Decoding spends its time in launches: the
// scale and codes of 4096 values take as long as those of 400,000, and the product waits for
// them.  Here every workgroup quantizes all of x for itself, a few blocks per lane, while its first chunks of B are
// on their way into LDS, and keeps the codes there; x and B come from memory once, and from the L2 for all
// workgroups but the first.  What bounds it: the launch, x's way (its maximum comes before anything else), then the
// quantizing (220 vector instructions per block; a lane has up to four, which take 4 us).  From Python, two calls / this:
// 1 x 512 x 512 11.5 / 5.3 us, 8 x 2048 x 2048 11.8 / 5.9, 4 x 4096 x 4096 10.9 / 6.7; gemm_shapes.hpp has both in a graph.
//
// The product's plan is k_gemm_skinny16's with eight waves: wave w takes the chunks of 256 indices with chunk % 8 == w,
// B through its own ring of stages (rows of 128 code bytes, 16-byte units swizzled, then the scales two bytes to a
// word: any K that is a multiple of 32), A's fragments straight from the codes in LDS, whose rows are padded to whole
// chunks with zeros and 16 bytes, for the banks.  Past the end of K the copies repeat a row's last unit and meet zeros.
template <int NT>
struct FewRows {
  static constexpr int kWaves = 8, kThreads = 64 * kWaves, NST = 2;
  static constexpr int kBlocks = 4;                          // blocks per lane at most
  static constexpr int COLS = 16 * NT, NC = COLS / 8;        // copies of codes, and of scales, per chunk
  static constexpr uint32_t STAGE = COLS * (128 + 32);
  static constexpr uint32_t padded(uint32_t K) { return (K + SK - 1) / SK * SK; }
  static constexpr uint32_t code_pitch(uint32_t K) { return padded(K) / 2 + 16; }
  static constexpr uint32_t scale_pitch(uint32_t K) { return padded(K) / 16 + 4; }
  static constexpr uint32_t lds(uint32_t M, uint32_t K) {
    return kWaves * NST * STAGE + M * (code_pitch(K) + scale_pitch(K));
  }
  // no size takes more: at most kFewValues values and as much padding, 16 bytes of code pitch and 4 of scale pitch as 16 rows have
  static constexpr uint32_t kMostLds = kWaves * NST * STAGE + (kFewValues + 16 * (SK - 32)) / 16 * 9 + 16 * 20;
  static_assert(kMostLds + sizeof(ScaleTable) + kWaves * sizeof(float) <= 160 * 1024, "the LDS of a compute unit");
};
static_assert(FewRows<1>::kBlocks * FewRows<1>::kThreads * 16 >= kFewValues, "a block per lane and turn");
static_assert(FewRows<2>::NST * FewRows<2>::STAGE >= 2 * 4 * 64 * sizeof(float), "a wave's sums fit its stages");

template <int NT>
__global__ __launch_bounds__(FewRows<NT>::kThreads) void k_few_rows(
    const uint4 *__restrict__ x, const uint8_t *__restrict__ codes_b, const uint8_t *__restrict__ scales_b,
    const float *__restrict__ alpha_b, uint16_t *__restrict__ out, uint32_t M, int64_t N, uint32_t K, uint32_t shb,
    float fp8_max) {
  typedef FewRows<NT> S;
  constexpr int W = S::kWaves, NST = S::NST, NC = S::NC, COLS = S::COLS;
  extern __shared__ __align__(16) uint8_t lds_raw[];
  __shared__ ScaleTable tab;
  __shared__ float wave_part[W];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t rr = lane & 15u, g = lane >> 4;
  // (the compiler's barrier would wait for the copies)
  auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

  // ---- x, and its maximum
  const uint32_t per_row = K / 16, nblocks = M * per_row;
  RawBlock<false> raw[S::kBlocks];
  PlainAmax<false> largest;
#pragma unroll
  for (int j = 0; j < S::kBlocks; ++j) {
    if (j * S::kThreads < nblocks) {                         // the same for all lanes
      const uint32_t k = t + j * S::kThreads;
      load_block<false>(x + 2 * (k < nblocks ? k : nblocks - 1), raw[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < S::kBlocks; ++j) {
    if (j * S::kThreads < nblocks) {
      largest.fold(raw[j].w[0]);
      largest.fold(raw[j].w[1]);
    }
  }
  float m = largest.value();
  // x is there before the first copy, and known to be: a wait for a register of it would wait for the copies too
  asm volatile("" : "+v"(m));
  __builtin_amdgcn_s_waitcnt(0x0f70);                        // vmcnt(0)

  // ---- copies of B
  auto uniform = [](const uint8_t *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const uint8_t *>(((uint64_t)hi << 32) | lo);
  };
  const int64_t n0 = (int64_t)blockIdx.x * COLS;
  const uint32_t row_codes = K / 2, row_scales = K / 16;
  const uint8_t *gcb = uniform(codes_b + n0 * row_codes), *gsb = uniform(scales_b + (n0 >> shb) * row_scales);
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds_raw +
                            wave * (NST * S::STAGE);
  uint32_t code_row[NC], code_unit[NC], scale_row[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const uint32_t row = 8 * q + (lane >> 3);
    const uint32_t line = n0 + row < N ? row : (uint32_t)(N - 1 - n0);        // relative to n0
    code_row[q] = line * row_codes;
    code_unit[q] = ((lane & 7u) ^ ((row >> 1) & 7u)) * 16u;
    scale_row[q] = (uint32_t)(((n0 + line) >> shb) - (n0 >> shb)) * row_scales;
  }
  auto copy_chunk = [&](uint32_t c, uint32_t stage) {
    const uint32_t lds = lds_wave + stage * S::STAGE;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const uint32_t at = c * (SK / 2) + code_unit[q], last = row_codes - 16u;
      NV_DMA16(lds + q * 1024, code_row[q] + (at < last ? at : last), gcb);
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const uint32_t at = c * (SK / 16) + (lane & 7u) * 2u, last = row_scales - 2u;
      NV_DMA2(lds + COLS * 128 + q * 256, scale_row[q] + (at < last ? at : last), gsb);
    }
  };
  constexpr int kCopies = 2 * NC;
  const uint32_t nchunks = (K + SK - 1) / SK;
  uint32_t c = wave;
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (c + W * p < nchunks) copy_chunk(c + W * p, p);

  // ---- scale and codes of x
  m = wave_max(m);
  if (lane == 0) wave_part[wave] = m;
  barrier();
#pragma unroll
  for (int w = 0; w < W; ++w) m = fmaxf(m, wave_part[w]);
  const float alpha = alpha_of(m, fp8_max);
  ScaleConsts sc = fill_scale_table(tab, alpha);
  barrier();
  take_reciprocals(tab, sc);
  const uint32_t code_pitch = S::code_pitch(K), scale_pitch = S::scale_pitch(K);
  uint8_t *const ca = lds_raw + W * NST * S::STAGE, *const sa = ca + M * code_pitch;
#pragma unroll
  for (int j = 0; j < S::kBlocks; ++j) {
    if (j * S::kThreads < nblocks) {
      const uint32_t k = t + j * S::kThreads;
      if (k < nblocks) {
        float v[16];
        const uint32_t u[16] = {};
        unpack16(raw[j], v);
        auto again = [&](float (&w)[16], uint32_t (&)[16]) { unpack16(raw[j], w); };
        const BlockResult r = quantize_block<kRTN, kSel46>(v, u, sc, tab, again);
        const uint32_t row = k / per_row, b = k - row * per_row;
        *reinterpret_cast<uint2 *>(ca + row * code_pitch + b * 8) = make_uint2(r.lo, r.hi);
        sa[row * scale_pitch + b] = (uint8_t)r.scale;
      }
    }
  }
  const uint32_t tail = S::padded(K) / 16 - per_row;          // blocks past the end of a row, at most 14
  if (t < M * tail) {
    const uint32_t row = t / tail, b = per_row + t - row * tail;
    *reinterpret_cast<uint2 *>(ca + row * code_pitch + b * 8) = make_uint2(0u, 0u);
    sa[row * scale_pitch + b] = 0;
  }
  barrier();

  // ---- the product: a lane's share of one operand row for one chunk, as in k_gemm_skinny16
  struct Raw {
    uint4 c[2];
    uint32_t s[2];
  };
  const uint32_t ra = rr < M ? rr : M - 1;
  auto read_a = [&](Raw &f) {
    const uint8_t *p = ca + ra * code_pitch + c * (SK / 2) + g * 32;
    f.c[0] = reinterpret_cast<const uint4 *>(p)[0];
    f.c[1] = reinterpret_cast<const uint4 *>(p)[1];
    const uint32_t s = *reinterpret_cast<const uint32_t *>(sa + ra * scale_pitch + c * (SK / 16) + g * 4);
    f.s[0] = __builtin_amdgcn_perm(0u, s, 0x0c010c00u) << 7;
    f.s[1] = __builtin_amdgcn_perm(0u, s, 0x0c030c02u) << 7;
  };
  auto read_b = [&](uint32_t stage, uint32_t row, Raw &f) {
    const uint8_t *st = lds_raw + (wave * NST + stage) * S::STAGE;
    const uint32_t swz = (row >> 1) & 7u;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      f.c[q] = *reinterpret_cast<const uint4 *>(st + row * 128 + (((2 * g + q) ^ swz) * 16));
    const uint2 s = *reinterpret_cast<const uint2 *>(st + COLS * 128 + row * 32 + g * 8);
    f.s[0] = __builtin_amdgcn_perm(0u, s.x, 0x0c010c00u) << 7;
    f.s[1] = __builtin_amdgcn_perm(0u, s.y, 0x0c010c00u) << 7;
  };
  auto expand = [&](const Raw &f, int s) {                         // matrix step s = 0..7
    const uint4 &q = f.c[s >> 2];
    const uint32_t w = (s & 3) == 0 ? q.x : (s & 3) == 1 ? q.y : (s & 3) == 2 ? q.z : q.w;
    const h2 pair = __builtin_bit_cast(h2, f.s[s >> 2]);
    return expand8(w, (s & 2) ? pair.y : pair.x);
  };
  f32x4 acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[j][v] = 0.0f;
  uint32_t stage = 0;
  auto chunk = [&](auto after) {
    Raw fa, fb[NT];
    read_a(fa);
#pragma unroll
    for (int j = 0; j < NT; ++j) read_b(stage, 16 * j + rr, fb[j]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    after();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const h8 a = expand(fa, s);
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, expand(fb[j], s), acc[j], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    c += W;
    stage = stage + 1 == (uint32_t)NST ? 0u : stage + 1;
  };
  while (c + W * NST < nchunks) {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((NST - 1) * kCopies) : "memory");
    chunk([&] { copy_chunk(c + W * NST, stage); });
  }
  each_number_down<NST>([&](auto p) {
    if (c + W * decltype(p)::value < nchunks) {
      asm volatile("s_waitcnt vmcnt(%0)" :: "n"(decltype(p)::value * kCopies) : "memory");
      chunk([] {});
    }
  });

  // ---- each wave's sums into its own (spent) stages; one lane per element adds them in the waves' order
  float *const own = reinterpret_cast<float *>(lds_raw + wave * (NST * S::STAGE));
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) own[(4 * j + v) * 64 + lane] = acc[j][v];
  barrier();
  const uint32_t e = t >> 6, j = e >> 2, v = e & 3u;
  if (e < 4 * NT) {
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w)
      sum += reinterpret_cast<const float *>(lds_raw + w * (NST * S::STAGE))[e * 64 + lane];
    const uint32_t row = 4 * g + v;
    const int64_t col = n0 + 16 * j + rr;
    if (row < M && col < N)
      out[row * N + col] = (uint16_t)pack_bf16x2(sum * (alpha * alpha_b[0]), 0.0f);
  }
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// The kernels compile side by side when this file is built in parts: NVFP4_46_GEMM_PART =
// 1..4 hold one instantiation of the staged kernel each (by far the slowest to compile),
// 5 the copy-based kernel, 6 the small-batch kernels and the kernel for smaller tiles, 0 the entry
// point; without the macro
// the file is one self-contained translation unit.
#ifndef NVFP4_46_GEMM_PART
#define NVFP4_46_GEMM_PART (-1)
#endif
#define NVFP4_46_GEMM_HAS(part) (NVFP4_46_GEMM_PART < 0 || NVFP4_46_GEMM_PART == (part))

struct GemmArgs {
  const uint8_t *codes_a, *scales_a;
  const float *alpha_a;
  const uint8_t *codes_b, *scales_b;
  const float *alpha_b;
  void *out;
  int64_t M, N, K;
  uint32_t sha, shb;     // scale rows are shared by 2^sha rows of A, 2^shb rows of B
  bool f32;              // C is fp32 instead of BF16
  hipStream_t stream;
};

struct FewRowsArgs {
  const uint4 *x;
  const uint8_t *codes_b, *scales_b;
  const float *alpha_b;
  uint16_t *out;
  int64_t M, N, K;
  uint32_t shb;
  float fp8_max;
  hipStream_t stream;
};

// Every run_* raises the kernel's dynamic LDS limit (most need more than the 64 KiB a
// kernel gets without asking), launches, and returns a status of the C ABI.  The limit belongs to the
// kernel and not to the call, so it is the same in every call: another thread's smaller one, set between
// this thread's two steps, would refuse the launch.
template <bool KFULL, bool OUTF32>
int run_gemm_staged(const GemmArgs &a);
template <typename S>
int run_gemm_dma(const GemmArgs &a);
int run_gemm_skinny(const GemmArgs &a);
template <typename S>
int run_gemm_tile(const GemmArgs &a);
int run_few_rows(const FewRowsArgs &a);

template <typename Kernel, typename... Args>
static int launch_with_lds_of(Kernel kernel, size_t most_lds_bytes, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s,
                              Args... args) {
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)most_lds_bytes) != hipSuccess) {
    return NVFP4_ERR_HIP;
  }
  return launch(kernel, grid, block, lds_bytes, s, args...);
}
// ... of a kernel that always has the same
template <typename Kernel, typename... Args>
static int launch_with_lds(Kernel kernel, dim3 grid, dim3 block, size_t lds_bytes, hipStream_t s,
                           Args... args) {
  return launch_with_lds_of(kernel, lds_bytes, grid, block, lds_bytes, s, args...);
}

// Strip width (in tiles) that makes an eighth of the tiles about square: h x w tiles of BM x BN with
// h w = tiles / 8 touch the fewest operand rows, BM h + BN w, at w = sqrt(tiles / 8 * BM / BN).
// Row by row / in strips: 1536 x 4096 x 8192 106 / 102 us, 8000 x 8000 x 2080 314 / 306, 768 x 4096
// x 8192 56 / 55.  Operands that fit the 4 MB of one die's L2 whole stay row by row (2880 x 1440 x
// 1056: 19.9 / 20.2).  (k_gemm_dma: no difference.)
template <int BM, int BN>
static uint32_t strip_of(const GemmArgs &a) {
  const double tm = (double)((a.M + BM - 1) / BM), tn = (double)((a.N + BN - 1) / BN);
  if ((double)(a.M + a.N) * (double)a.K * 0.5625 <= 4.0 * 1024 * 1024) return (uint32_t)tn;
  const double w = std::sqrt(tm * tn / 8.0 * BM / BN) + 0.5;
  return (uint32_t)(w < 1.0 ? 1.0 : w > tn ? tn : w);
}

static dim3 tile_grid(const GemmArgs &a) {
  const int64_t tiles_m = (a.M + GT - 1) / GT, tiles_n = (a.N + GT - 1) / GT;
  return dim3((uint32_t)(tiles_m * tiles_n));
}

template <bool KFULL, bool OUTF32>
int run_gemm_staged(const GemmArgs &a) {
  return launch_with_lds(k_gemm<KFULL, OUTF32>, tile_grid(a), dim3(kGemmThreads), kGemmLdsBytes,
                         a.stream, a.codes_a, a.scales_a, a.alpha_a, a.codes_b, a.scales_b,
                         a.alpha_b, a.out, a.M, a.N, a.K, (uint32_t)((a.N + GT - 1) / GT), a.sha,
                         a.shb);
}
#if NVFP4_46_GEMM_PART == 0
extern template int run_gemm_staged<false, false>(const GemmArgs &);
extern template int run_gemm_staged<false, true>(const GemmArgs &);
extern template int run_gemm_staged<true, false>(const GemmArgs &);
extern template int run_gemm_staged<true, true>(const GemmArgs &);
#elif NVFP4_46_GEMM_PART >= 1 && NVFP4_46_GEMM_PART <= 4
template int run_gemm_staged<((NVFP4_46_GEMM_PART - 1) / 2 != 0), ((NVFP4_46_GEMM_PART - 1) % 2 != 0)>(
    const GemmArgs &);
#endif

#if NVFP4_46_GEMM_HAS(5)
template <typename S>
int run_gemm_dma(const GemmArgs &a) {
  auto go = [&](auto kernel, bool kfull) {
    return launch_with_lds(kernel, dim3((uint32_t)tiles_of<S>(a.M, a.N)), dim3(S::kThreads), S::lds(kfull), a.stream,
                           a.codes_a, a.scales_a, a.alpha_a, a.codes_b, a.scales_b, a.alpha_b, a.out, a.M, a.N,
                           (uint32_t)a.K, (uint32_t)((a.M + S::BM - 1) / S::BM), (uint32_t)((a.N + S::BN - 1) / S::BN),
                           strip_of<S::BM, S::BN>(a), a.sha, a.shb);
  };
  if (a.K % S::CK == 0) return a.f32 ? go(k_gemm_dma<S, true, true>, true) : go(k_gemm_dma<S, true, false>, true);
  return a.f32 ? go(k_gemm_dma<S, false, true>, false) : go(k_gemm_dma<S, false, false>, false);
}
#endif
#if NVFP4_46_GEMM_PART == 0 || NVFP4_46_GEMM_PART == 5
#if NVFP4_46_GEMM_PART == 0
#define NVFP4_46_DMA extern template
#else
#define NVFP4_46_DMA template
#endif
NVFP4_46_DMA int run_gemm_dma<Dma256>(const GemmArgs &);
NVFP4_46_DMA int run_gemm_dma<Dma256x128>(const GemmArgs &);
NVFP4_46_DMA int run_gemm_dma<Dma128>(const GemmArgs &);
#endif

#if NVFP4_46_GEMM_HAS(6)
// Few rows of A: one workgroup per 32 columns of C, bound by streaming B.
int run_gemm_skinny(const GemmArgs &a) {
  auto go = [&](auto kernel, int mt) {
    return launch_with_lds(kernel, dim3((uint32_t)((a.N + 31) / 32)), dim3(64 * skinny_waves(mt)),
                           skinny_lds_bytes(mt), a.stream, a.codes_a, a.scales_a, a.alpha_a,
                           a.codes_b, a.scales_b, a.alpha_b, a.out, a.M, a.N, a.K, a.sha, a.shb);
  };
  if (a.M <= 16) {
    auto go16 = [&](auto kernel) {
      return launch_with_lds(kernel, dim3((uint32_t)((a.N + 31) / 32)), dim3(64 * kSkinny16Waves),
                             kSkinny16LdsBytes, a.stream, a.codes_a, a.scales_a, a.alpha_a,
                             a.codes_b, a.scales_b, a.alpha_b, a.out, a.M, a.N, a.K, a.sha, a.shb);
    };
    return a.f32 ? go16(k_gemm_skinny16<true>) : go16(k_gemm_skinny16<false>);
  }
  if (a.M <= 32) return a.f32 ? go(k_gemm_skinny<1, true>, 1) : go(k_gemm_skinny<1, false>, 1);
  return a.f32 ? go(k_gemm_skinny<2, true>, 2) : go(k_gemm_skinny<2, false>, 2);
}
#endif

#if NVFP4_46_GEMM_HAS(6)
int run_few_rows(const FewRowsArgs &a) {
  auto go = [&](auto kernel, auto shape) {
    typedef decltype(shape) S;
    return launch_with_lds_of(kernel, S::kMostLds, dim3((uint32_t)((a.N + S::COLS - 1) / S::COLS)), dim3(S::kThreads),
                              S::lds((uint32_t)a.M, (uint32_t)a.K), a.stream, a.x, a.codes_b, a.scales_b, a.alpha_b,
                              a.out, (uint32_t)a.M, a.N, (uint32_t)a.K, a.shb, a.fp8_max);
  };
  // at most one workgroup per compute unit, in the narrower of the two
  if ((a.N + 15) / 16 <= kCus) return go(k_few_rows<1>, FewRows<1>{});
  return go(k_few_rows<2>, FewRows<2>{});
}
#endif

#if NVFP4_46_GEMM_HAS(6)
template <typename S>
int run_gemm_tile(const GemmArgs &a) {
  auto go = [&](auto kernel) {
    return launch_with_lds(kernel, dim3((uint32_t)tiles_of<S>(a.M, a.N)), dim3(S::kThreads), S::LDS,
                           a.stream, a.codes_a, a.scales_a, a.alpha_a, a.codes_b, a.scales_b,
                           a.alpha_b, a.out, a.M, a.N, (uint32_t)a.K,
                           (uint32_t)((a.M + S::BM - 1) / S::BM),
                           (uint32_t)((a.N + S::BN - 1) / S::BN), strip_of<S::BM, S::BN>(a), a.sha,
                           a.shb);
  };
  if (a.K % S::CK == 0) return a.f32 ? go(k_gemm_tile<S, true, true>) : go(k_gemm_tile<S, true, false>);
  if constexpr (S::kFirst)
    if (S::scales_first(a.K)) return a.f32 ? go(k_gemm_scales_first<S, true>) : go(k_gemm_scales_first<S, false>);
  return a.f32 ? go(k_gemm_tile<S, false, true>) : go(k_gemm_tile<S, false, false>);
}
#endif
#if NVFP4_46_GEMM_PART == 0
#define NVFP4_46_TILE(S) extern template int run_gemm_tile<S>(const GemmArgs &);
#elif NVFP4_46_GEMM_PART == 6
#define NVFP4_46_TILE(S) template int run_gemm_tile<S>(const GemmArgs &);
#endif
#ifdef NVFP4_46_TILE
NVFP4_46_TILE(Tile32)
NVFP4_46_TILE(Tile64x32)
NVFP4_46_TILE(Tile64)
NVFP4_46_TILE(Tile64Long)
NVFP4_46_TILE(Tile128)
NVFP4_46_TILE(Tile256x128)
#endif

}  // namespace nvfp4_46

#if NVFP4_46_GEMM_PART <= 0

using namespace nvfp4_46;

// (see layer.hpp)
extern "C" int nvfp4_46_few_rows(const void *x, float fp8_max, const void *codes_b, const void *scales_b,
                                 const float *alpha_b, int64_t M, int64_t N, int64_t K, uint32_t flags, void *out,
                                 void *stream) {
  if (!x || !codes_b || !scales_b || !alpha_b || !out) return NVFP4_ERR_NULL;
  if (M <= 0 || N <= 0 || K <= 0 || K % 32 != 0) return NVFP4_ERR_SHAPE;
  if (flags & ~(uint32_t)NVFP4_GEMM_B_TILE_SCALES) return NVFP4_ERR_PARAM;
  if ((flags & NVFP4_GEMM_B_TILE_SCALES) && N % 16 != 0) return NVFP4_ERR_SHAPE;
  if (!aligned16(x) || !aligned16(codes_b) || !aligned16(scales_b) || !aligned16(out)) return NVFP4_ERR_ALIGN;
  if (!(fp8_max > 0.0f) || !(fp8_max <= 448.0f)) return NVFP4_ERR_PARAM;
  if (!few_rows_in_one_launch(M, N, K)) return NVFP4_ERR_UNSUPPORTED;
  return run_few_rows(FewRowsArgs{static_cast<const uint4 *>(x), static_cast<const uint8_t *>(codes_b),
                                  static_cast<const uint8_t *>(scales_b), alpha_b, static_cast<uint16_t *>(out), M, N, K,
                                  (flags & NVFP4_GEMM_B_TILE_SCALES) ? 4u : 0u, fp8_max,
                                  static_cast<hipStream_t>(stream)});
}

extern "C" int nvfp4_46_gemm(const void *codes_a, const void *scales_a, const float *alpha_a,
                             const void *codes_b, const void *scales_b, const float *alpha_b,
                             int64_t M, int64_t N, int64_t K, uint32_t out_dtype, uint32_t flags,
                             void *out, void *stream) {
  if (!codes_a || !scales_a || !alpha_a || !codes_b || !scales_b || !alpha_b || !out)
    return NVFP4_ERR_NULL;
  if (M <= 0 || N <= 0 || K <= 0 || (K % 32) != 0) return NVFP4_ERR_SHAPE;
  if (M > (int64_t)1 << 31 || N > (int64_t)1 << 31 || K > (int64_t)1 << 31 ||
      M * K > (int64_t)1 << 40 || N * K > (int64_t)1 << 40 || M * N > (int64_t)1 << 40)
    return NVFP4_ERR_SHAPE;
  if (out_dtype > NVFP4_OUT_F32 || flags > (NVFP4_GEMM_A_TILE_SCALES | NVFP4_GEMM_B_TILE_SCALES))
    return NVFP4_ERR_PARAM;
  if (((flags & NVFP4_GEMM_A_TILE_SCALES) && (M % 16) != 0) ||
      ((flags & NVFP4_GEMM_B_TILE_SCALES) && (N % 16) != 0))
    return NVFP4_ERR_SHAPE;
  if (!aligned16(codes_a) || !aligned16(scales_a) || !aligned16(codes_b) || !aligned16(scales_b) ||
      !aligned16(out))
    return NVFP4_ERR_ALIGN;
  const int64_t tiles_m = (M + GT - 1) / GT, tiles_n = (N + GT - 1) / GT;
  if (tiles_m * tiles_n > (int64_t)1 << 30) return NVFP4_ERR_SHAPE;
  const GemmArgs a{static_cast<const uint8_t *>(codes_a), static_cast<const uint8_t *>(scales_a),
                   alpha_a, static_cast<const uint8_t *>(codes_b),
                   static_cast<const uint8_t *>(scales_b), alpha_b, out, M, N, K,
                   (flags & NVFP4_GEMM_A_TILE_SCALES) ? 4u : 0u,
                   (flags & NVFP4_GEMM_B_TILE_SCALES) ? 4u : 0u, out_dtype == NVFP4_OUT_F32,
                   static_cast<hipStream_t>(stream)};
  switch (choose_gemm(M, N, K, a.f32)) {
    case kGemmStaged:
      return (K % GK) == 0 ? (a.f32 ? run_gemm_staged<true, true>(a) : run_gemm_staged<true, false>(a))
                           : (a.f32 ? run_gemm_staged<false, true>(a) : run_gemm_staged<false, false>(a));
    case kGemmDma: return run_gemm_dma<Dma256>(a);
    case kGemmDma256x128: return run_gemm_dma<Dma256x128>(a);
    case kGemmDma128: return run_gemm_dma<Dma128>(a);
    case kGemmSkinny: return run_gemm_skinny(a);
    case kGemmTile32: return run_gemm_tile<Tile32>(a);
    case kGemmTile64x32: return run_gemm_tile<Tile64x32>(a);
    case kGemmTile64: return run_gemm_tile<Tile64>(a);
    case kGemmTile64Long: return run_gemm_tile<Tile64Long>(a);
    case kGemmTile128: return run_gemm_tile<Tile128>(a);
    default: return run_gemm_tile<Tile256x128>(a);
  }
}

#endif

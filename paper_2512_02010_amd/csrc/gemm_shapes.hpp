// Host side of the matrix product: the tile shapes of its kernels and which kernel a product takes.
// Plain C++ without HIP, so that the choice and the budgets can be checked where there is no GPU.
#pragma once

#include <cstddef>
#include <cstdint>

namespace nvfp4_46 {

constexpr int GT = 256;                  // k_gemm: rows of A (and of B) per workgroup tile
constexpr int GK = 128;                  // ... and contraction steps per chunk
constexpr int SK = 256;                  // k_gemm_skinny, k_gemm_skinny16: contraction steps per chunk
constexpr int64_t kCus = 256;

// k_gemm_tile's shapes (described at the kernel).
template <int WM_, int WN_, int SM_, int SN_, int KS_, int HPW_, int NST_>
struct TileShape {
  static constexpr int WM = WM_, WN = WN_, SM = SM_, SN = SN_, KS = KS_, HPW = HPW_, NST = NST_;
  static constexpr int kWaves = SM * SN * KS, kThreads = 64 * kWaves;
  static constexpr int BM = 32 * WM * SM, BN = 32 * WN * SN, ROWS = BM + BN;
  static constexpr int CK = 64 * KS * HPW;                // contraction steps per chunk
  static constexpr int U = CK / 32;                       // 16-byte units of codes (= scale pairs) per row
  static constexpr int kCopies = ROWS * U / 64;           // copy instructions per chunk, codes (and scales)
  static constexpr int NC = (kCopies + kWaves - 1) / kWaves;
  static constexpr uint32_t kScaleBase = ROWS * U * 16, STAGE = ROWS * U * 20;
  // Where K is whole chunks, scales are copied in pieces of 16 bytes, this many to a row and chunk, else (0) two bytes
  // per lane: an eighth of the copy instructions, which the waves of 64 x 64 tiles would otherwise spend as many on as
  // on codes (us, two bytes / 16: 200 x 4096 x 4096 13.7 / 12.9, 512 x 2048 x 1024 5.9 / 5.6, 3000 x 3000 x 1024 25.3 /
  // 24.6, 192 x 4096 x 11264 24.9 / 23.8).  32 x 32 and 64 x 32 tiles are slower with it (64 x 1024 x 4096 6.4 / 6.7, 128 x
  // 4096 x 4096 9.8 / 10.0: one wave's copy of 32 lines, for which all wait), 128 x 128 no faster (1000 x 4096 x 768
  // 10.6 / 10.6); and where lines begin anywhere, two pieces to a row, 300 x 2000 x 1056 takes 7.4, not 6.5.
  static constexpr int kPieces = WM * WN == 4 && SM * SN == 1 && CK % 256 == 0 ? CK / 256 : 0;
  static constexpr int T = WM + WN, kTiles = WM * WN;
  // 64 x 64 tiles: where K is no whole number of chunks but all scales of both tiles fit the LDS beside the stages, which is
  // up to K = 2016, they are copied there before the first chunk, as one run of memory: `rows` lines, which may begin 14
  // bytes into the first 16 (us, two bytes per lane and chunk / this: 2880 x 1440 x 1056 17.4 / 16.3, 575 x 2048 x 1056
  // 9.1 / 8.5, 900 x 1600 x 2016 12.4 / 11.4, 1000 x 1000 x 1312 7.4 / 7.2).  Not below four chunks (501 x 1333 x 736 5.5 /
  // 5.7: an edge's last bytes have a latency of their own), nor in the smaller tiles (128 x 2000 x 1056 4.15 / 4.15, 100 x
  // 3000 x 544 4.2 / 4.3); 128 x 128 has no registers for it.
  static constexpr uint32_t first_scales(int rows, uint32_t row_scales) { return (rows * row_scales + 31) & ~15u; }
  static constexpr bool kFirst = WM * WN == 4 && SM * SN == 1 && KS == 4;
  static constexpr bool scales_first(int64_t K) {
    return kFirst && K % CK != 0 && K >= 4 * CK && K <= 8192 &&
           NST * kScaleBase + first_scales(BM, (uint32_t)K / 16) + first_scales(BN, (uint32_t)K / 16) + 2 * U <= LDS;
  }
  // partial sums of the KS groups: each owns kOwn instruction tiles, exchanged in PH phases
  static constexpr int kOwn = KS == 1 ? kTiles : kTiles >= KS ? kTiles / KS : 1;
  static constexpr int VW = kTiles * 4 >= KS ? 4 : 2;      // accumulators of a lane that go together
  static constexpr int kPartialTile = (KS - 1) * SM * SN * 4096;
  static constexpr int kPerPhaseMax = KS == 1 ? kTiles : 160 * 1024 / kPartialTile;
  static constexpr int PER = kPerPhaseMax < kTiles ? kPerPhaseMax : kTiles;
  static constexpr int LDS_STAGES = NST * STAGE, LDS_PART = KS == 1 ? 0 : PER * kPartialTile;
  static constexpr int LDS = LDS_STAGES > LDS_PART ? LDS_STAGES : LDS_PART;
  static_assert(ROWS * U % 64 == 0 && BM % (64 / U) == 0 && U <= 16, "a copy instruction stays within one operand");
  static_assert(LDS <= 160 * 1024, "the stages must fit the LDS");
  static_assert(kTiles % KS == 0 || KS % kTiles == 0, "kOwn");
  static_assert(kTiles * (16 / VW) % KS == 0, "as many units for every copy");
  static_assert((NST - 1) * 2 * NC < 63, "vmcnt counts to 63");
};

// The shapes of k_gemm_tile that are in use.  (Timed against these: 64 x 64 with three stages, 128
// x 64 and 128 x 128 in two copies, 32 x 64, 32 x 32 in four copies, 256 x 256.)
using Tile32 = TileShape<1, 1, 1, 1, 8, 1, 2>;         // 32 x 32, 8 waves, each an eighth of K
using Tile64x32 = TileShape<2, 1, 1, 1, 4, 1, 2>;      // 64 x 32, 4 waves
using Tile64 = TileShape<2, 2, 1, 1, 4, 1, 2>;         // 64 x 64, 4 waves; three workgroups per CU
using Tile64Long = TileShape<2, 2, 1, 1, 8, 1, 2>;     // 64 x 64, 8 waves
using Tile128 = TileShape<2, 2, 2, 2, 4, 1, 2>;        // 128 x 128, 16 waves
using Tile256x128 = TileShape<4, 2, 2, 2, 2, 1, 4>;    // 256 x 128, 8 waves

// k_gemm_dma's shapes (described at the kernel): four waves of WM x WN instruction tiles, SM x SN of them over the
// tile of C and KS along the contraction axis, each taking HPW pieces of 64 steps of a chunk; NST stages.
template <int WM_, int WN_, int SM_, int SN_, int KS_, int HPW_, int NST_>
struct DmaShape {
  static constexpr int WM = WM_, WN = WN_, SM = SM_, SN = SN_, KS = KS_, HPW = HPW_, NST = NST_;
  static constexpr int kWaves = SM * SN * KS, kThreads = 64 * kWaves;
  static constexpr int BM = 32 * WM * SM, BN = 32 * WN * SN, ROWS = BM + BN;
  static constexpr int CK = 64 * KS * HPW, U = CK / 32, T = WM + WN, kTiles = WM * WN;
  // bytes of a stage: codes, then 2 (K whole chunks) or 4 bytes per pair of scales
  static constexpr uint32_t kCodes = ROWS * U * 16;
  static constexpr uint32_t stage(bool kfull) { return kCodes + ROWS * U * (kfull ? 2 : 4); }
  // copy instructions per wave and chunk: codes and scales
  static constexpr int NC = ROWS * U / 64 / kWaves;
  static constexpr int ns(bool kfull) { return ROWS * U / (kfull ? 128 : 64) / kWaves; }
  // a block of 32 rows per wave of the partial sums, on its way through LDS to the store; two of them in turn
  static constexpr int kPitch = BN + 4;
  static constexpr uint32_t kSums = KS * SM * 32 * kPitch * 4;
  static constexpr uint32_t lds(bool kfull) {
    return NST * stage(kfull) > 2 * kSums ? NST * stage(kfull) : 2 * kSums;
  }
  static_assert(ROWS * U % (128 * kWaves) == 0 && BM % (128 / U) == 0, "a copy instruction stays within one operand");
  static_assert(lds(false) <= 160 * 1024 && lds(true) <= 160 * 1024, "the stages must fit the LDS");
  static_assert((NST - 2) * (NC + ns(false)) < 63, "vmcnt counts to 63");
};
using Dma256 = DmaShape<4, 4, 2, 2, 1, 2, 4>;          // 256 x 256, each wave a quarter of it
using Dma256x128 = DmaShape<4, 4, 2, 1, 2, 1, 5>;      // 256 x 128, two waves per half of K
using Dma128 = DmaShape<4, 4, 1, 1, 4, 1, 4>;          // 128 x 128, each wave a quarter of K

constexpr int64_t tiles_of(int64_t M, int64_t N, int BM, int BN) {
  return ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
}
template <typename S>
constexpr int64_t tiles_of(int64_t M, int64_t N) { return tiles_of(M, N, S::BM, S::BN); }

enum GemmKernel {
  kGemmStaged, kGemmDma, kGemmSkinny, kGemmTile32, kGemmTile64x32, kGemmTile64, kGemmTile64Long,
  kGemmTile128, kGemmTile256x128, kGemmDma256x128, kGemmDma128
};

// How evenly tiles of BM x BN divide over whole turns of one workgroup per compute unit ...
inline double turns_filled(int64_t M, int64_t N, int BM, int BN) {
  const int64_t tiles = tiles_of(M, N, BM, BN);
  return (double)tiles / (double)((tiles + kCus - 1) / kCus * kCus);
}
// ... and how much of them there is to do: what tiles of 64 x 64 would cover of C over what these do.
// 64 x 28672 has 224 tiles of 256 x 128, which fill a turn to 87 %, but hold 64 of 256 rows each (at
// K = 8192 110 us, in 64 x 64 tiles 45).  64 x 64 is the measure because that is the other choice, with
// padding of its own: 196 rows pad to 256 in either (196 x 29536 x 4096: 63 in 256 x 128, 72 in 64 x 64).
inline double tiles_covered(int64_t M, int64_t N, int BM, int BN) {
  return (double)tiles_of<Tile64>(M, N) * Tile64::BM * Tile64::BN /
         ((double)tiles_of(M, N, BM, BN) * BM * BN);
}
template <typename S>
inline bool fills_chip(int64_t M, int64_t N, double turns) {
  return turns_filled(M, N, S::BM, S::BN) >= turns && tiles_covered(M, N, S::BM, S::BN) >= 0.8;
}
// Both in one figure: the share of the chip that is busy with what exists.
template <typename S>
inline double chip_filled(int64_t M, int64_t N) {
  return turns_filled(M, N, S::BM, S::BN) * tiles_covered(M, N, S::BM, S::BN);
}

// Which kernel: times in us, BF16 out, on one card, M x N x K; operands as the calls before left
// them (all in the memory-side cache), or B from memory where it says so.  `f32`: C is fp32, not BF16.
inline GemmKernel fastest_gemm(int64_t M, int64_t N, int64_t K, bool f32) {
  if (K > ((int64_t)1 << 24)) return kGemmStaged;       // 32-bit lane offsets of the others' copies

  // Few rows of A against a large weight: the kernels that stream B, one workgroup per 32 columns.
  // Up to 32 rows always (16 x 8192 x 8192: 9.5, in 32 x 32 tiles 11.6; 32 x 8192 x 28672: 29.6 /
  // 33.6; B from memory, 16 x 28672 x 8192: 32 / 40, 32 x 28672 x 8192: 40 / 43, 32 x 4096 x 4096 7.9 / 8.6; but 17 to 32
  // rows along a short K, or with all operands in the memory-side cache, are as fast or faster in tiles: 32 x 4096 x
  // 4096 6.8 / 6.5, 32 x 2048 x 1024 4.0 / 3.6, 32 x 512 x 256 3.8 / 3.0); from 33 to 64 rows
  // only between the widths whose 32 x 32 tiles are at most one per compute unit (64 x 4096 x 4096:
  // 9.6, tiles 6.6) and those that fill the chip in 64 x 64 tiles (B from memory, 33 / 64 x 28672 x
  // 8192: 52 / 57, tiles 46 / 46; 33 / 64 x 128256 x 4096: 108 / 120, tiles 89 / 93; between them
  // 64 x 8192 x 8192: 17 / 22); with up to 48 rows and narrower weights where the stream is long,
  // which the tiles' one workgroup per compute unit does not keep up with (B from memory, 33 / 48 / 64
  // rows x 4096 x 28672: 38 / 39 / 45, tiles 41; 33 x 2048 x 53248: 65 / 73; but 33 x 4096 x 8192: 15.1 /
  // 14.3).
  const int64_t t32 = tiles_of<Tile32>(M, N), t64 = tiles_of<Tile64>(M, N);
  const bool stream_64 = t32 > kCus || (M <= 48 && N * K > ((int64_t)1 << 25));
  if ((K % SK) == 0 && (M <= 32 || (M <= 64 && t64 <= kCus && stream_64))) return kGemmSkinny;

  // The largest tiles (the fewest expansions and copies per product) that leave little of the chip idle, padding
  // counted as idle.  k_gemm_dma's three shapes (the shape / what would run else):
  //   256 x 256 from 62 %: 6144 x 6400 x 1056 (78 %) 104 / 108, 2816 x 4096 x 4064 (69 %) 93 / 107, x 32 12.8 / 15.6,
  //   8192 x 8192 x 96 44 / 62; 3000 x 3000 x 1024 (56 %) 29.6 / 26.3;
  //   256 x 128 from 62 % of one turn, 72 % of several: 2048 x 4096 x 4096 63 / 68.5, 1536 x 4096 x 4096 (75 %) 52 / 56,
  //   6798 x 880 x 4160 (73 %) 55 / 63, 192 x 28672 x 8192 (66 %) 101 / 103, 1024 x 5000 x 1024 (62 %) 15.2 / 16.3, but the
  //   shorter K of 996 x 5232 x 704 (64 %) 16.2 / 15.1 in 64 x 64; 3388 x 1408 x 2304 (60 %) 29.9 / 28.0, 4798 x 912 x 768
  //   (59 %) 15.4 / 13.2; three turns: 8324 x 1925 x 256 (66 %) 30 / 22 and 6496 x 2681 x 256 (70 %) 31 / 22;
  //   128 x 128 from 70 % of one turn and a K whose quarters outlast their sum's way through LDS: 1000 x 4096 x 4096
  //   33.5 / 36.6, 768 x 4096 x 4096 (75 %) 28.7 / 30.0, 128 x 28672 x 8192 (87 %) 56 / 68; 575 x 4526 x 4352 (63 %)
  //   29.8 / 29.6; 1000 x 4096 x 1024 13.5 / 13.2 and x 256 9.3 / 7.4; two turns and more 3000 x 3000 x 1024 35 / 27.
  // They store 16 bytes per lane, which takes a quarter longer (3 to 5 us of one turn) where the lines of C do not
  // begin at multiples of 16 bytes.  The smaller two shapes are then ahead of k_gemm_tile, which stores column by
  // column, only along a longer K (2048 x 4095: K = 32 13.2 / 11.1, 256 15.3 / 12.5, 640 20.3 / 17.9; 1654 x 4428 x 128
  // 12.7 / 10.5; 128 x 128: 4055 x 738 x 1536, fp32, 19 % longer).
  const bool skewed = N * (f32 ? 4 : 2) % 16 != 0, one_turn = tiles_of<Dma256x128>(M, N) <= kCus;
  if (chip_filled<Dma256>(M, N) >= 0.62) return kGemmDma;
  if (chip_filled<Dma256x128>(M, N) >= (one_turn ? 0.62 : 0.72) && !(one_turn && skewed && K < 1024))
    return kGemmDma256x128;
  if (K >= (skewed ? 2048 : 1024) && tiles_of<Dma128>(M, N) <= kCus && chip_filled<Dma128>(M, N) >= 0.7)
    return kGemmDma128;
  // ... and k_gemm_tile's: 256 x 128 from 80 % (2048 x 3072 x 4096, 75 %: 57, in 64 x 64 tiles 56), 128 x 128 from 87 %
  // (1000 x 4096 x 800: 12.0, in 64 x 64 13.3; 2048 x 3072 x 4096, 75 %: 62), both only where they cover 80 % of it (192 x
  // 28672 x 8192, 75 %: 116 in 256 x 128, 103 in 64 x 64).
  if (fills_chip<Tile256x128>(M, N, 0.8)) return kGemmTile256x128;
  if (fills_chip<Tile128>(M, N, 0.87)) return kGemmTile128;
  // Small products: the smallest tiles that are at most one per compute unit (64 x 1024 x 4096:
  // 6.3 in 32 x 32, 8.9 in 64 x 32, 11.9 in 64 x 64; 128 x 4096 x 4096: 10.1 / 9.4 / 12.5; 200 x
  // 4096 x 4096: 16.2 / 14.3 / 13.0); 32 rows or columns would leave larger tiles half empty (B from
  // memory, 16 x 28672 x 8256: 40 / 54 / 49, and 124 in 256 x 128).  Along a long K two tiles of
  // 32 x 32 per compute unit still beat fewer larger ones (B from memory, 65 x 5120 x 8192: 18 / 24 /
  // 26; 128 x 4096 x 28672: 59 / 74 / 83; 256 x 2048 x 28672: 59 / 72 / 82; with K no whole number of their chunks 256 x
  // 2048 x 11008 26 / 29 too; not from memory 128 x 4096 x 4096 10.1 / 9.4).
  const int64_t t64x32 = tiles_of<Tile64x32>(M, N);
  const bool two_of_32 = K >= 8192 && (K % Tile32::CK == 0 || t64x32 > kCus);
  if (M <= 32 || t32 <= (two_of_32 ? 2 : 1) * kCus) return kGemmTile32;
  if (N <= 32 || t64x32 <= kCus) return kGemmTile64x32;
  // 64 x 64 tiles, at most one per compute unit: along a long K in eight copies, since four waves wait
  // for most of every chunk (four / eight copies, B from memory, 128 x 8192 x 8192: 29.1 / 24.9; 192 x
  // 4096 x 11008: 32.6 / 28.7; 128 x 8192 x 28672: 89 / 78).  Their chunks are twice as long, and a shorter
  // K leaves the last one emptier, which costs less since the empty pieces are left out (141 x 4652 x 4352: 15.4 / 13.7).
  if (K >= 8192 && t64 <= kCus) return kGemmTile64Long;
  return kGemmTile64;
}

constexpr int kGemmThreads = 256;        // k_gemm, k_gemm_dma, k_gemm_skinny and k_gemm_skinny16
inline int64_t lanes_of(GemmKernel kernel, int64_t M, int64_t N) {
  switch (kernel) {
    case kGemmSkinny: return (N + 31) / 32 * kGemmThreads;
    case kGemmTile32: return tiles_of<Tile32>(M, N) * Tile32::kThreads;
    case kGemmTile64x32: return tiles_of<Tile64x32>(M, N) * Tile64x32::kThreads;
    case kGemmTile64: return tiles_of<Tile64>(M, N) * Tile64::kThreads;
    case kGemmTile64Long: return tiles_of<Tile64Long>(M, N) * Tile64Long::kThreads;
    case kGemmTile128: return tiles_of<Tile128>(M, N) * Tile128::kThreads;
    case kGemmTile256x128: return tiles_of<Tile256x128>(M, N) * Tile256x128::kThreads;
    case kGemmDma256x128: return tiles_of<Dma256x128>(M, N) * Dma256x128::kThreads;
    case kGemmDma128: return tiles_of<Dma128>(M, N) * Dma128::kThreads;
    default: return tiles_of(M, N, GT, GT) * kGemmThreads;
  }
}

// A launch holds fewer than 2^32 lanes: where one row or column of C is that long, the kernels of the
// fewest lanes per element take it.
inline GemmKernel choose_gemm(int64_t M, int64_t N, int64_t K, bool f32) {
  const GemmKernel fastest = fastest_gemm(M, N, K, f32);
  if (lanes_of(fastest, M, N) >> 32 == 0) return fastest;
  return (K % GK) == 0 && K <= ((int64_t)1 << 24) ? kGemmDma : kGemmStaged;
}

// Up to which size x and its product with a quantized weight take one launch (k_few_rows): as far as it is not behind the
// two launches in a replayed graph (us, two launches / one: 1 x 512 x 512 5.8 / 3.9, 8 x 2048 x 2048 7.8 / 5.6, 12 x 2048
// x 8192 7.8 / 7.4, 14 x 2048 x 8192 8.2 / 8.1 but 16 x 2048 x 8192 8.0 / 8.7; 7 x 4096 x 4096 9.1 / 8.1, 1 x 8192 x 8192
// 12.4 / 9.5), and one workgroup per compute unit (1 x 2048 x 28672: 10.7 / 16.0).  Called one by one the two launches
// take 11 to 12 us at all these sizes, the one 5 to 9.
constexpr int64_t kFewValues = 28672, kFewColumns = 32 * kCus;
inline bool few_rows_in_one_launch(int64_t M, int64_t N, int64_t K) {
  return M <= 16 && M * K <= kFewValues && N <= kFewColumns;
}
}  // namespace nvfp4_46

// Host side of the quantizer: up to which size a tensor takes the small-tensor kernels.  Plain C++
// without HIP, so that the rules can be checked where there is no GPU.
#pragma once

#include <cstdint>

namespace nvfp4_46 {

// Times in us per call in a replayed graph of 200 calls on tensors of their own, BF16 / FP32; x in the
// memory-side cache, or in memory (a first read).  A launch costs the host 2.7 to 3.3 us besides.
//
// Tensor scale in one workgroup (k_scale_small):
//           in the cache                          in memory
//   KiB     one       with scratch  three         one         with scratch  three
//   128     3.0/2.8   3.5/3.5       5.4/5.4       4.3/4.2     4.2/4.2       6.1/6.0
//   160     4.1/3.9   3.7/3.7       5.6/5.6       5.7/5.6     4.3/4.2       6.1/6.1
//   256     4.2/3.8   3.8/3.8       6.0/5.9       6.5/6.3     4.3/4.2       6.4/6.4
//   512     6.6/6.1   3.9/3.8       6.8/6.6       11.1/10.6   4.4/4.3       7.2/7.1
//   768     8.9/8.2   4.0/3.9       7.3/7.2       15.5/14.9   4.5/4.4       7.9/7.8
//   1024    11.2/10.4 4.1/3.9       7.9/7.9       19.9/19.2   4.5/4.4       8.6/8.5
// With a workspace it replaces one launch by one: as far as it is ahead in the cache and not behind in memory.
// Without, it replaces three, which the host pays for: as far as it is not behind when called one by one with x
// in the cache (us per call among others from Python, BF16: 512 KiB 6.5 / 11.1, 768 KiB 8.9 / 8.7 to 11.4, 896 KiB
// 9.9 / 8.8 to 12, 1 MiB 11.2 / 11.2; first read from memory 10.7 / 9.5, 15.2 / 8.5, 17.3 / 10.1 and 19.8 / 9.9;
// programs that replay graphs have a workspace).
// On the default stream, without a workspace, it replaces one launch on lent words, which costs the host 0.2 to 0.5 us more.
// Such calls come one by one and have others after them that the host is busy
// with while the one workgroup reads, so what counts is the whole pass (us among others from Python, BF16, one workgroup /
// lent words; fp32 is within 0.5 of it):
//   KiB     scale, codes, values    scale, fake-quant   scale, both orientations   scale alone
//   256     15.2 / 15.7             9.1 / 9.3           12.0 / 12.2                4.2 / 4.6
//   384     15.2 / 15.7             9.3 / 9.3           12.0 / 12.2                4.5 / 4.5
//   512     15.2 / 15.8             9.7 / 9.1           11.9 / 12.2                5.5 / 4.6
//   640     15.1 / 15.5             10.0 / 9.3          12.1 / 12.4                6.4 / 4.6
//   768     15.0 / 15.4             11.3 / 9.3          12.9 / 12.2                7.2 / 4.5
enum class ScratchWords { kNone, kLent, kWorkspace };
constexpr bool scale_in_one_workgroup(int64_t bytes, ScratchWords words) {
  return bytes <= (int64_t)(words == ScratchWords::kWorkspace ? 128 : words == ScratchWords::kLent ? 512 : 768) << 10;
}

// Scale and rowwise codes in one launch (k_scale_quantize_small), against codes in a launch of their
// own after the scale in one launch (with scratch words) or as above (without: one workgroup to 768 KiB, then three):
//           in the cache                           in memory
//   KiB     one       with scratch  without        one        with scratch  without
//   256     5.8/5.3   7.1/6.7       7.4/6.7        6.2/5.8    7.8/7.4       10.0/9.4
//   320     6.9/6.6   7.3/6.8       8.6/8.0        7.3/7.1    7.9/7.4       11.7/11.4
//   384     7.0/6.7   7.3/6.8       8.8/8.0        7.4/7.1    8.0/7.5       12.4/11.8
//   448     8.0/7.6   7.3/6.9       9.8/9.3        8.4/8.1    8.0/7.5       14.0/13.9
//   512     8.1/7.7   7.3/6.9       10.0/9.0       8.5/8.1    8.1/7.5       14.8/13.8
//   768     10.4/9.9  7.5/7.0       12.5/11.4      10.9/10.3  8.2/7.7       19.5/18.9
//   896     11.6/10.8 7.6/7.1       11.0/10.4      12.0/11.3  8.3/7.8       11.9/11.4
// As far as it is ahead in both columns.  The library's own scratch words on the default stream count as none
// here: such calls come one by one, where a second launch costs the host more than the reading (us per call from Python,
// BF16 512 KiB: one launch 8.5, two 10.8).  (FP32 ended at 256 KiB and the calls without scratch words at 512 while a
// workgroup quantized 1024 blocks.)
constexpr bool scale_and_codes_in_one_launch(int64_t bytes, bool has_scratch) {
  return bytes <= (int64_t)(has_scratch ? 384 : 768) << 10;
}

// Tensor scale after the columnwise transform (k_amax_rht_col): whether a lane takes 4 bytes of each of a block's sixteen rows
// instead of 16, for so many words of 4 bytes in a sixteenth of the rows.  A lane's columns follow each other, so 4 where
// those are still no more than two waves per SIMD, in fp32 a little less (us in a replayed graph, 16 / 4 bytes, BF16 256 x
// 512 5.5 / 4.65, 736 x 1024 5.75 / 4.65, 1344 x 2208 5.8 / 5.2, 1008 x 4096 5.85 / 5.5, 2048 x 2048 6.2 / 5.9, 2048 x 4096 6.25 /
// 6.8, 4096 x 4096 7.5 / 9.0; fp32 736 x 1024 5.0 / 4.5, 480 x 4096 and 1920 x 1024 5.15 / 5.0, 1024 x 2048 and 256 x 8192
// 5.1 / 5.3, 4096 x 4096 14.8 / 16.4; 8 bytes lie between).
constexpr bool scale_by_words(int64_t words, bool xf32) {
  return words <= (int64_t)(xf32 ? 15 : 16) << 13;
}

}  // namespace nvfp4_46

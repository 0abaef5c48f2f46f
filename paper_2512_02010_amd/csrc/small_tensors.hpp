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
//   128     3.0/2.9   4.5/4.5       5.3/5.4       4.3/4.2     5.1/5.0       6.1/6.1
//   160     4.1/3.9   4.6/4.6       5.7/5.6       5.7/5.6     5.1/5.0       6.2/6.1
//   256     4.2/3.9   4.8/4.7       6.1/6.0       6.5/6.2     5.1/5.1       6.4/6.4
//   512     6.6/6.1   4.8/4.8       6.6/6.6       10.9/10.5   5.2/5.1       7.1/7.0
//   768     8.9/8.3   4.9/4.8       7.2/7.1       15.2/14.7   5.2/5.1       7.7/7.7
//   1024    11.2/10.4 4.9/4.8       7.7/7.7       19.6/18.7   5.2/5.1       8.3/8.3
// With scratch words it replaces one launch by one: as far as it is ahead in both columns.  Without,
// it replaces three, which the host pays for: as far as it is not behind when called one by one with x
// in the cache (us per call among others: 512 KiB 7.0 / 10.7, 768 KiB 9.3 / 10.7, 1 MiB 11.8 / 10.8; first
// read from memory 11.1 / 10.6, 15.5 / 10.8 and 20.1 / 10.8; programs that replay graphs have scratch words).
constexpr bool scale_in_one_workgroup(int64_t bytes, bool has_scratch) {
  return bytes <= (int64_t)(has_scratch ? 128 : 768) << 10;
}

// Scale and rowwise codes in one launch (k_scale_quantize_small), against codes in a launch of their
// own after the scale in one (with scratch words) or three launches (without):
//           in the cache                           in memory
//   KiB     one       with scratch  without        one        with scratch  without
//   256     6.9/6.7   7.9/7.5       9.1/8.7        7.8/8.1    8.4/8.0       9.7/9.2
//   320     8.0/7.8   7.9/7.5       9.2/8.9        8.8/9.4    8.4/8.0       9.8/9.4
//   384     8.1/8.1   8.0/7.5       9.4/9.0        9.1/9.6    8.5/8.0       10.0/9.5
//   512     9.5/9.4   8.1/7.6       9.8/9.3        10.4/11.1  8.6/8.1       10.4/9.9
//   768     11.8/11.5 8.2/7.7       10.5/10.0      12.7/13.2  8.7/8.2       11.2/10.7
constexpr bool scale_and_codes_in_one_launch(int64_t bytes, bool xf32, bool has_scratch) {
  return bytes <= (int64_t)(!has_scratch ? 512 : xf32 ? 256 : 384) << 10;
}

}  // namespace nvfp4_46

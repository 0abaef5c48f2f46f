// How a tensor of BF16 or fp32 values arrives in registers: blocks of sixteen, the largest magnitude, Eq. (1).
#pragma once

#include "codec.hpp"

namespace nvfp4_46 {

NV_DEV uint4 load_stream(const uint4 *p) { return *p; }
NV_DEV void unpack16(const uint4 &w0, const uint4 &w1, float (&v)[16]) {
  const uint32_t w[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    v[2 * j] = bf16_lo(w[j]);
    v[2 * j + 1] = bf16_hi(w[j]);
  }
}

// A block as it arrives from memory: two 128-bit pieces of BF16 or four of fp32.
template <bool XF32>
struct RawBlock {
  static constexpr int kPieces = XF32 ? 4 : 2;
  uint4 w[kPieces];
};
template <bool XF32>
NV_DEV void load_block(const uint4 *p, RawBlock<XF32> &r) {
#pragma unroll
  for (int j = 0; j < RawBlock<XF32>::kPieces; ++j) r.w[j] = load_stream(p + j);
}
template <bool XF32>
NV_DEV void unpack16(const RawBlock<XF32> &r, float (&v)[16]) {
  if constexpr (XF32) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[4 * j] = u2f(r.w[j].x);
      v[4 * j + 1] = u2f(r.w[j].y);
      v[4 * j + 2] = u2f(r.w[j].z);
      v[4 * j + 3] = u2f(r.w[j].w);
    }
  } else {
    unpack16(r.w[0], r.w[1], v);
  }
}

NV_DEV float wave_max(float m) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  return m;
}

// Eq. (1): alpha = amax / (6 * fp8_max); an all-zero tensor gets alpha = 1.
NV_DEV float alpha_of(float amax, float fp8_max) {
  return (amax == 0.0f) ? 1.0f : amax / (6.0f * fp8_max);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Largest magnitude, compared as integers (15 bits of a BF16 value, 31 of an fp32 value).
template <bool XF32>
struct PlainAmax {
  u16x2 acc = {0, 0};
  uint32_t acc32 = 0;
  NV_DEV void fold(const uint4 &w) {
    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (XF32) {
        const uint32_t m = ww[j] & 0x7fffffffu;
        acc32 = m > acc32 ? m : acc32;
      } else {
        uint32_t m = ww[j] & 0x7fff7fffu;
        acc = __builtin_elementwise_max(acc, *reinterpret_cast<u16x2 *>(&m));
      }
    }
  }
  NV_DEV float value() const {
    return u2f(XF32 ? acc32 : (uint32_t)(acc.x > acc.y ? acc.x : acc.y) << 16);
  }
};

}  // namespace nvfp4_46

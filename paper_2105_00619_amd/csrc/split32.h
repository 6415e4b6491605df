// fp32 operands on the 16-bit matrix cores.
//
// A float is the sum of three bf16 values (8 + 8 + 8 bits of its 24): plane 0 is the value rounded to bf16, plane 1 what
// that leaves, rounded, plane 2 what the two leave, exact but for its last rounding (2^-27 of the value).  The product of
// two floats is then the six products of planes whose indices add up to at most two; the three left out are below 2^-26 of
// it.  The 16-bit MFMAs multiply exactly and add in fp32, so a sum carries the error of its fp32 additions -- of six per 16
// products, where the fp32 MFMA makes eight -- and six of them take 192 cycles of a SIMD for what the fp32 instruction
// does in 512: registers only, on normally distributed values (the clock follows the power), 296 TFLOP/s of fp32 products
// against 155.  Measured in the layers (us, fp32 MFMA -> this): 3x3, 64 -> 64 channels at 1 048 576 pixels forward and data gradient
// 706 -> 446 (173 TFLOP/s), weight gradient 797 -> 367 (211); 128 -> 128 at 262 144 515 -> 420 and 719 -> 387; strided 64 -> 128
// 260 -> 245, 227 -> 195 and 570 -> 435.
//
// The 16-bit MFMA drops what lies eight or more bits below the last one of its largest term, towards minus infinity: a sum of 400
// MFMAs is too low by 6e-8 of the results' deviation, one over a million pixels by 3.3e-6, each by as much.  So half of a sum is
// made with one operand negated: forward and data gradient in a second accumulator, a weight gradient in every other pixel range
// and, for the ranges' own sake, from wgrad_flip on, where the accumulators are negated with it (mean error of a weight gradient
// of 64 -> 64 channels over 1 048 576 pixels -3.3e-6 of its deviation -> 5e-9, over 4 194 304 -1.2e-5 -> -2e-8, root mean square
// 3.5e-6 -> 1.0e-6 and 1.3e-5 -> 1.9e-6, on the fp32 MFMA 1.2e-6 and 2.3e-6; in the same time).
//
// Not finite: a value beyond the largest bf16, an infinity or a NaN makes planes that are not finite, and every sum with it
// a NaN.  A block that finds such a sum when its tile is done makes the tile again -- forward and data gradient on the fp32 MFMA,
// weight gradients as chains of multiply-adds, pixel by pixel -- so that infinities and NaNs come out as from fp32 arithmetic.
// (Two 64 -> 64 layers at 1 048 576 pixels, one infinity in the images: 7.1 ms a step, 2.5 without it.  As a chain per such output,
// one thread each, it was 95 ms.)
#pragma once
#include "dev_common.h"

namespace oseq {

// two floats -> their three planes, each a pair of bf16 in one register
__device__ __forceinline__ void split32_pair(float a, float b, uint32_t (&p)[3]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    p[q] = __builtin_bit_cast(uint32_t, from_f32x2<bf16_t>(a, b));
    if (q < 2) {
      const uint32_t lo = p[q] << 16, hi = p[q] & 0xffff0000u;
      a -= __builtin_bit_cast(float, lo);
      b -= __builtin_bit_cast(float, hi);
    }
  }
}

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

// four floats -> their three planes, 8 bytes each
__device__ __forceinline__ void split32(const Chunk& c, u32x2_t (&p)[3]) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  const f32x4 v = __builtin_bit_cast(f32x4, c);
  uint32_t lo[3], hi[3];
  split32_pair(v[0], v[1], lo);
  split32_pair(v[2], v[3], hi);
#pragma unroll
  for (int q = 0; q < 3; ++q) { p[q][0] = lo[q]; p[q][1] = hi[q]; }
}

// the depth tile of n from which on a weight gradient's operand is negated: what is dropped goes with the size of the sum, which
// grows with the square root of the tiles, so 5/8 of them drop as much as the rest (n^1.5 / 2)
__device__ __forceinline__ int wgrad_flip(int n) { return n * 5 / 8; }
// c, negated where sign is the sign bit; zero where ok is false (one three-operand instruction a value)
__device__ __forceinline__ Chunk signed_chunk(const Chunk& c, bool ok, uint32_t sign) {
  const uint32_t keep = ok ? ~0u : 0u;
  Chunk r;
#pragma unroll
  for (int k = 0; k < 4; ++k) r[k] = (c[k] & keep) ^ sign;
  return r;
}

}  // namespace oseq

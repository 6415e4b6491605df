// Division of 32-bit numbers by a number fixed at launch, as a multiplication.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define OSEQ_FASTDIV_FN __host__ __device__ __forceinline__
#else
#define OSEQ_FASTDIV_FN inline
#endif

namespace oseq {

// floor(m / d) for every m < 2^32 and 1 <= d <= 2^31: the upper part of m * ceil(2^63 / d).  The rounding of the factor adds
// less than m / 2^63 < 1 / d to the quotient, and the product of 95 bits is taken in two halves, so nothing wraps.  (In 64 bits
// with a factor of 2^48 the product wraps as soon as the quotient reaches 2^16, e.g. an image index of a large batch.)
struct FastDiv {
  uint64_t magic; uint32_t d;
  OSEQ_FASTDIV_FN uint32_t div(uint32_t m) const {
    const uint64_t lo = ((uint64_t)(uint32_t)magic * m) >> 32;
    return (uint32_t)(((uint64_t)(uint32_t)(magic >> 32) * m + lo) >> 31);
  }
};
inline FastDiv make_fastdiv(uint32_t d) { FastDiv f; f.d = d; f.magic = (((uint64_t)1 << 63) + d - 1) / d; return f; }

}  // namespace oseq

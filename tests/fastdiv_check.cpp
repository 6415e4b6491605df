// Host check of csrc/fastdiv.h: the quotient for divisors and numbers around every power of two and around multiples of the
// divisor, among them quotients on both sides of 2^16 and divisor 1, and for a fixed pseudo-random set.  Prints the number of
// pairs compared, or the first wrong one.
#include <cstdio>

#include "fastdiv.h"

static uint64_t pairs = 0;
static bool check(uint32_t m, uint32_t d) {
  ++pairs;
  if (oseq::make_fastdiv(d).div(m) == m / d) return true;
  std::printf("wrong: %u / %u gives %u\n", m, d, oseq::make_fastdiv(d).div(m));
  return false;
}

int main() {
  uint64_t state = 88172645463325252ull;
  auto next = [&] { state ^= state << 13; state ^= state >> 7; state ^= state << 17; return state; };
  for (int b = 0; b <= 31; ++b)
    for (int o = -2; o <= 2; ++o) {
      const int64_t d64 = ((int64_t)1 << b) + o;
      if (d64 < 1 || d64 > (int64_t)1 << 31) continue;
      const uint32_t d = (uint32_t)d64;
      for (int e = 0; e <= 32; ++e)
        for (int64_t p = -3; p <= 3; ++p) {
          const int64_t edge = ((int64_t)1 << e) + p;
          if (edge >= 0 && edge < (int64_t)1 << 32 && !check((uint32_t)edge, d)) return 1;
          const unsigned __int128 mult = (unsigned __int128)(edge < 0 ? 0 : edge) * d;  // the quotient is near 2^e
          for (int s = -1; s <= 1; ++s)
            if (mult < ((unsigned __int128)1 << 32) && !check((uint32_t)mult + s, d)) return 1;
        }
    }
  for (int i = 0; i < 4000000; ++i) {
    const uint32_t d = (uint32_t)(next() >> (33 + next() % 31)) + 1;
    if (!check((uint32_t)(next() >> 32), d > (1u << 31) ? 1u << 31 : d)) return 1;
  }
  std::printf("ok %llu\n", (unsigned long long)pairs);
  return 0;
}

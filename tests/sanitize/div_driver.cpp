// The kernels' divisions by launch constants (cci_div.hpp) against the
// language's, over the ranges the launchers accept.
#include <cstdio>
#include <cstdlib>

#include "../../paper_1910_11971_amd/csrc/cci_div.hpp"

static void check(uint32_t n, uint32_t d) {
  uint32_t r = 0;
  const uint32_t q = cci::divmod(n, cci::make_div(d), r);
  if (q != n / d || r != n % d) {
    printf("%u / %u: %u rest %u\n", n, d, q, r);
    exit(1);
  }
}

int main() {
  // k-steps of a tap (Cin / 32, C = taps * Cin <= 2^24): first and last step of every tap
  for (uint32_t taps = 1; taps <= 32; ++taps)
    for (uint32_t steps = 1; steps <= (1u << 19) / taps; ++steps)
      for (uint32_t t = 0; t < taps; ++t) {
        check(t * steps, steps);
        check(t * steps + steps - 1, steps);
      }
  // any 32-bit numerator: around multiples of small, odd, power-of-two and large divisors
  for (uint64_t d : {1ull, 2ull, 3ull, 7ull, 49ull, 56ull * 56, 65535ull, 65536ull, 65537ull, 1ull << 24, (1ull << 31) - 1, 1ull << 31})
    for (uint64_t k = 0; k < 4096; ++k) {
      const uint64_t top = 0xffffffffull / d, m = (k % 2 ? top - k / 2 % (top + 1) : k / 2 % (top + 1)) * d;
      for (int64_t e : {-1, 0, 1})
        if (static_cast<int64_t>(m) + e >= 0 && m + e <= 0xffffffffull) check(static_cast<uint32_t>(m + e), static_cast<uint32_t>(d));
    }
  for (int32_t d = 1; d <= 64; ++d)
    for (uint32_t n = 0; n <= 64; ++n)
      if (cci::small_div(n, cci::make_small_div(d)) != n / static_cast<uint32_t>(d)) {
        printf("small %u / %d\n", n, d);
        return 1;
      }
  printf("div driver ok\n");
  return 0;
}

// Divisions by launch constants as multiplications (host and device).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cci {

// Division by a launch constant d: with m = floor(2^32 / d) (all ones for d =
// 1) the high half of n m is n / d or one less, for every 32-bit n.
struct Div {
  uint32_t d, m;
};
inline Div make_div(int64_t d) {
  return Div{static_cast<uint32_t>(d), d > 1 ? static_cast<uint32_t>((uint64_t(1) << 32) / static_cast<uint64_t>(d)) : ~0u};
}
__host__ __device__ inline uint32_t divmod(uint32_t n, const Div v, uint32_t& rem) {
  const uint32_t q = static_cast<uint32_t>(static_cast<uint64_t>(n) * v.m >> 32), r = n - q * v.d;
  rem = r >= v.d ? r - v.d : r;
  return r >= v.d ? q + 1 : q;
}

// The same without a correction for small numbers: n / d for n, d <= 64.
inline uint32_t make_small_div(int32_t d) { return (1u << 16) / static_cast<uint32_t>(d) + 1; }
__host__ __device__ inline uint32_t small_div(uint32_t n, uint32_t m) { return n * m >> 16; }

}  // namespace cci

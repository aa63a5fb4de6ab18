// Outputs over their kept columns alone, for the kernels that multiply
// expanded tiles.  There a dropped weight is a zero that is multiplied, so an
// infinity or NaN of X makes every output of its row NaN; on the sparse-MAC
// kernels it reaches the outputs that keep its column.  A product that AUTO
// takes from the sparse-MAC kernels keeps their results (ProductArgs::
// kept_only): a finite sum has met no such value (infinity times zero and
// all that follows is NaN), so only the non-finite sums are formed again, by
// a whole wave each, from the packed rows.
#pragma once

#include "cci_device.hpp"

namespace cci {

// Sum of output o of row n over its kept columns, lanes over the columns (n
// and o wave-uniform).  P: the kernel's parameters (bf16 X [N][C], or NHWC
// with CONV; packed vals and idx [O / G][K][C]).
template <bool CONV, typename P>
__device__ __forceinline__ float kept_sum(const P& p, int32_t K, int32_t n, int32_t o) {
  const int32_t lane = static_cast<int32_t>(threadIdx.x) & 63;
  const int32_t g = o / p.G, slot = o - g * p.G;
  int32_t img = 0, ih0 = 0, iw0 = 0;
  if constexpr (CONV) {
    uint32_t rem, ow;
    img = static_cast<int32_t>(divmod(static_cast<uint32_t>(n), p.fd_howo, rem));
    ih0 = static_cast<int32_t>(divmod(rem, p.fd_wo, ow)) * p.sh - p.ph;
    iw0 = static_cast<int32_t>(ow) * p.sw - p.pw;
  }
  float s = 0.0f;
#pragma unroll 1
  for (int32_t c0 = 0; c0 < p.C; c0 += 64) {  // (the same trips for every lane)
    const int32_t c = c0 + lane;
    if (c < p.C) {
      int64_t at = static_cast<int64_t>(n) * p.C + c;
      bool in = true;
      if constexpr (CONV) {
        const int32_t t = c / p.Cin, kh = t / p.KW, ih = ih0 + kh, iw = iw0 + t - kh * p.KW;
        in = ih >= 0 && ih < p.H && iw >= 0 && iw < p.W;
        at = ((static_cast<int64_t>(img) * p.H + ih) * p.W + iw) * p.Cin + (c - t * p.Cin);
      }
      const float x = in ? bf16_to_f32(p.X[at]) : 0.0f;
#pragma unroll 1
      for (int32_t k = 0; k < K; ++k) {
        const int64_t q = (static_cast<int64_t>(g) * K + k) * p.C + c;
        if ((K == p.G ? k : static_cast<int32_t>(p.idx[q])) == slot) s = __builtin_fmaf(bf16_to_f32(p.vals[q]), x, s);
      }
    }
    // a NaN, or infinities of both signs, settle the sum: inputs full of them
    // end after a trip or two
    if (__any(s != s) || (__any(s == __builtin_inff()) && __any(s == -__builtin_inff()))) return __builtin_nanf("");
  }
#pragma unroll
  for (int off = 32; off >= 1; off /= 2) s += __shfl_xor(s, off, 64);
  return s;
}

// Replaces the non-finite ones of the lane's eight sums y (row n, outputs o ..
// o + 7; not live: no outputs).  All lanes of the wave call it together.
template <bool CONV, typename P>
__device__ __forceinline__ void keep_kept(float (&y)[8], const P& p, int32_t K, int32_t n, int32_t o, bool live) {
  uint32_t bad = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) bad |= (__float_as_uint(y[e]) & 0x7f800000u) == 0x7f800000u ? 1u << e : 0u;
  if (!live) bad = 0;
  const int32_t lane = static_cast<int32_t>(threadIdx.x) & 63;
#pragma unroll 1
  for (uint64_t lanes = __ballot(bad != 0); lanes != 0; lanes &= lanes - 1) {
    const int src = __builtin_ctzll(lanes);
    const int32_t sn = __builtin_amdgcn_readlane(n, src), so = __builtin_amdgcn_readlane(o, src);
#pragma unroll 1
    for (uint32_t bits = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(bad), src)); bits != 0;
         bits &= bits - 1) {
      const int e = __builtin_ctz(bits);
      const float s = kept_sum<CONV>(p, K, sn, so + e);
#pragma unroll
      for (int f = 0; f < 8; ++f) y[f] = lane == src && f == e ? s : y[f];
    }
  }
}

}  // namespace cci
